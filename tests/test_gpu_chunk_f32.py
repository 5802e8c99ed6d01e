"""fp32 inputs on the matrix-core chunk form (SWILA_ALGO_AUTO for J <= 4, J * Dk <=
256 on small grids) against the token-by-token scan and the fp64 oracle, in the
plain, temporal, gated and gated temporal forms.  Its products keep all 24 bits of
their operands (three bf16 parts each), so both forms differ from the oracle by
fp32 rounding: 1e-7 to 8e-7 (2-norm) measured over lengths of 17 to 4096.  The bound
is 3e-6, 2^-18: two of the three parts alone would leave 4e-6 and more."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import NAMES, to_device

pytestmark = pytest.mark.gpu

TOL = 3e-6


def _rel(x, y):
    return np.linalg.norm(x - y) / max(np.linalg.norm(y), 1e-30)


def _run(form, inp, tmp, dec, algo):
    import torch
    import paper_2609_39034_amd as sw
    dev = to_device(inp, "f32")
    args = [dev[n] for n in NAMES]
    cu = lambda x: None if x is None else torch.from_numpy(x).cuda()
    gates = dict(gate_k_logit=cu(tmp["gk"]), gate_q_logit=cu(tmp["gq"]), prior_in=cu(tmp["prior"]))
    if form == "plain":
        out = sw.forward(*args, dev["state"], resp=True, algo=algo)
    elif form == "temporal":
        out = sw.forward_temporal(*args, gates["gate_k_logit"], gates["gate_q_logit"], dev["state"],
                                  gates["prior_in"], resp=True, algo=algo)
    else:
        out = sw.forward_gated(*args, cu(dec), dev["state"], resp=True, algo=algo,
                               **(gates if form == "gated_temporal" else {}))
    torch.cuda.synchronize()
    return [x.cpu().numpy().astype(np.float64) for x in out]


def _check(form, B, H, T, Dk, Dv, J, std, mean, prior, seed, same=False, v_at=(), tol=TOL):
    inp = workloads.iid_inputs(B, H, T, Dk, Dv, J, dtype="f32", seed=seed, state_std=std)
    tmp = workloads.temporal_inputs(B, H, T, Dv, J, dtype="f32", seed=seed, prior_state=prior)
    dec = workloads.gated_inputs(B, H, T, Dk, J, dtype="f32", seed=seed, mean=mean)["decay"]
    for t in v_at:
        inp["v"][:, t] = np.sign(inp["v"][:, t]) * np.float32(13.5)
    a, r = _run(form, inp, tmp, dec, "auto"), _run(form, inp, tmp, dec, "recurrent")
    if same:
        for x, y in zip(a, r):
            assert np.array_equal(x, y)
        return
    kw = {}
    if "temporal" in form:
        kw.update(gate_k_logit=tmp["gk"], gate_q_logit=tmp["gq"], prior_in=tmp["prior"])
    if "gated" in form:
        kw.update(decay_logit=dec)
    ref = oracle.forward(*(inp[n] for n in NAMES), inp["state"], want_resp=True, **kw)
    names = ("o", "state", "prior", "resp") if "temporal" in form else ("o", "state", "resp")
    for name, x, y in zip(names, a, r):
        print(form, name, _rel(x, y), _rel(x, ref[name]))
        assert _rel(x, y) <= tol and _rel(x, ref[name]) <= tol, name


FORMS = ["plain", "temporal", "gated", "gated_temporal"]


# every J and Dk the rule takes, both column blocks (16 output dims from 256 blocks
# on), lengths around the chunk edges, gates from nearly open to past the factorised
# Gram products
@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("B,H,T,Dk,Dv,J,std,mean,prior", [
    (1, 2, 37, 64, 64, 4, 0.1, 2.0, True), (1, 1, 8, 64, 16, 4, 0.0, 2.0, False),
    (2, 1, 16, 32, 16, 2, 0.0, 1.0, True), (1, 3, 17, 128, 32, 2, 0.2, 2.0, False),
    (1, 2, 33, 16, 128, 1, 0.3, 2.0, True), (2, 2, 47, 32, 64, 3, 0.1, 0.0, True),
    (1, 2, 49, 128, 16, 1, 0.1, 2.0, False), (1, 1, 64, 64, 32, 3, 0.1, 3.0, True),
    (16, 16, 19, 16, 16, 4, 0.1, 2.0, True), (8, 32, 18, 64, 16, 2, 0.1, 2.0, False),
    (1, 2, 40, 64, 32, 4, 0.2, -4.0, True), (1, 2, 50, 128, 16, 2, 0.2, -3.0, True),
    # lengths from which AUTO takes the chunk form (the two meet later with fewer components)
    (1, 3, 31, 128, 32, 2, 0.2, 2.0, False), (1, 2, 127, 128, 16, 1, 0.1, 2.0, False),
    (16, 16, 24, 64, 16, 2, 0.1, 2.0, False), (1, 2, 95, 64, 16, 1, 0.1, -3.0, True),
])
def test_chunk_matches_token_scan(form, B, H, T, Dk, Dv, J, std, mean, prior):
    _check(form, B, H, T, Dk, Dv, J, std, mean, prior, 1500 + T + Dk + J)


@pytest.mark.parametrize("form", ["plain", "gated"])
@pytest.mark.parametrize("at", [(0,), (15,), (16, 31), (33,)])
def test_rerun_with_the_maximum_subtracted(form, at):
    """|delta| of 13 to 14 puts the sum over j below 2^-100.  A rounding of delta
    (2^-24 of it, three of them with the prediction's and the square's) moves
    e^{-delta^2/2} by delta^2 times as much: 196 * 3 * 2^-24 = 3.5e-5 of r."""
    _check(form, 1, 2, 34, 64, 32, 4, 0.1, 2.0, True, 1550, v_at=at, tol=3.5e-5)


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("B,H,T,Dk,Dv,J", [
    (1, 2, 20, 128, 16, 4), (1, 2, 20, 64, 16, 8),       # J * Dk > 256, J > 4
    (1, 2, 7, 64, 16, 4), (1, 2, 31, 32, 16, 1),         # T * J < 32
    (17, 16, 18, 16, 16, 2), (33, 32, 9, 16, 16, 4),     # larger grids
])
def test_other_calls_keep_the_token_scan(form, B, H, T, Dk, Dv, J):
    _check(form, B, H, T, Dk, Dv, J, 0.1, 2.0, True, 1570 + J, same=True)


# what is not finite at one token leaves the tokens before it as they are, also
# those of its own chunk, and every other output dim
@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("name,value", [("v", np.nan), ("v", np.inf), ("beta_logit", np.nan)])
def test_not_finite_reaches_later_tokens_only(form, name, value):
    B, H, T, Dk, Dv, J, at = 1, 2, 45, 32, 16, 4, 23
    inp = workloads.iid_inputs(B, H, T, Dk, Dv, J, dtype="f32", seed=1590, state_std=0.1)
    tmp = workloads.temporal_inputs(B, H, T, Dv, J, dtype="f32", seed=1590, prior_state=True)
    dec = workloads.gated_inputs(B, H, T, Dk, J, dtype="f32", seed=1590, mean=2.0)["decay"]
    inp[NAMES[2] if name == "v" else NAMES[3]][0, at, 1, ..., 5] = value
    a, r = _run(form, inp, tmp, dec, "auto"), _run(form, inp, tmp, dec, "recurrent")
    o, want = a[0], np.isfinite(r[0])
    assert want[:, :at].all() and want[:, :, 0].all() and not want[0, at:, 1, 5].any()
    assert np.array_equal(np.isfinite(o), want)
    assert _rel(o[want], r[0][want]) <= TOL
    assert np.array_equal(np.isfinite(a[1]), np.isfinite(r[1]))


# the same for every component count (J = 3 has a padding lane in each dim) and for the
# first dim of a block, which idle lanes might read
@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("J", [1, 2, 3])
@pytest.mark.parametrize("dim", [0, 8, 15])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_not_finite_stays_in_its_dim(form, J, dim, value):
    B, H, T, Dk, Dv, at = 1, 2, 45, 32, 16, 23
    inp = workloads.iid_inputs(B, H, T, Dk, Dv, J, dtype="f32", seed=1595, state_std=0.1)
    tmp = workloads.temporal_inputs(B, H, T, Dv, J, dtype="f32", seed=1595, prior_state=True)
    dec = workloads.gated_inputs(B, H, T, Dk, J, dtype="f32", seed=1595, mean=2.0)["decay"]
    inp["v"][0, at, 1, dim] = value
    a, r = _run(form, inp, tmp, dec, "auto"), _run(form, inp, tmp, dec, "recurrent")
    want = np.ones(a[0].shape, bool)
    want[0, at:, 1, dim] = False
    assert np.array_equal(np.isfinite(r[0]), want)   # (the token scan)
    assert np.array_equal(np.isfinite(a[0]), want)
    assert _rel(a[0][want], r[0][want]) <= TOL
    assert np.array_equal(np.isfinite(a[1]), np.isfinite(r[1]))
