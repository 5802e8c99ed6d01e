"""Gated Temporal SwiLA on the matrix-core chunk form (SWILA_ALGO_AUTO for bf16
inputs, J <= 4, J * Dk <= 256) against the token-by-token scan and the fp64
oracle.  Both evaluate the recurrence with fp32-grade arithmetic (the chunk
form's products take three bf16 parts of each fp32 operand), so the state, r and
the priors agree to a few 1e-7 of their size (2-norm; 4e-7 measured against the
oracle over lengths of 17 to 4096): the bound is 2e-6.  o is bf16 in both: a value
that sits on a rounding boundary may round either way, and neighbouring bf16
values (8 significant bits) lie up to 2^-7 of their size apart."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import NAMES, to_device

pytestmark = pytest.mark.gpu

TOL, TOL_O = 2e-6, 2.0 ** -7


def _inputs(B, H, T, Dk, Dv, J, seed, std, mean, prior):
    inp = workloads.iid_inputs(B, H, T, Dk, Dv, J, dtype="bf16", seed=seed, state_std=std)
    tmp = workloads.temporal_inputs(B, H, T, Dv, J, dtype="bf16", seed=seed, prior_state=prior)
    dec = workloads.gated_inputs(B, H, T, Dk, J, dtype="bf16", seed=seed, mean=mean)["decay"]
    return inp, tmp, dec


def _gpu(inp, tmp, dec, algo, **kw):
    import torch
    import paper_2609_39034_amd as sw
    dev = to_device(inp, "bf16")
    bf = lambda x: torch.from_numpy(x).to("cuda", torch.bfloat16)
    p = None if tmp["prior"] is None else torch.from_numpy(tmp["prior"]).cuda()
    out = sw.forward_gated(*(dev[n] for n in NAMES), bf(dec), dev["state"], gate_k_logit=bf(tmp["gk"]),
                           gate_q_logit=bf(tmp["gq"]), prior_in=p, resp=True, algo=algo, **kw)
    torch.cuda.synchronize()
    return [x.float().cpu().numpy().astype(np.float64) for x in out]


def _rel(x, y):
    return np.linalg.norm(x - y) / max(np.linalg.norm(y), 1e-30)


def _check(case, tol=TOL, **kw):
    a, r = _gpu(*case, "auto", **kw), _gpu(*case, "recurrent", **kw)
    inp, tmp, dec = case
    ref = oracle.forward(*(inp[n] for n in NAMES), inp["state"], want_resp=True, decay_logit=dec,
                         gate_k_logit=tmp["gk"], gate_q_logit=tmp["gq"], prior_in=tmp["prior"])
    for name, x, y, z in zip(("o", "state", "prior", "resp"), a, r,
                             (ref["o"], ref["state"], ref["prior"], ref["resp"])):
        if name == "o":
            scale = np.maximum(np.abs(y), 1e-3 * np.abs(y).max())
            assert np.max(np.abs(x - y) / scale) <= TOL_O * 1.01, name
            assert _rel(x, z) <= 3e-3
        else:
            print(name, _rel(x, y), _rel(x, z))
            assert _rel(x, y) <= tol and _rel(x, z) <= tol, name


# every J and Dk the rule takes, both column blocks (DB = 16 from 256 blocks on),
# lengths around the chunk edges, gates from nearly open to past the factorised
# Gram products
@pytest.mark.parametrize("B,H,T,Dk,Dv,J,std,mean,prior", [
    (1, 2, 37, 64, 64, 4, 0.1, 2.0, True), (1, 1, 1, 64, 16, 4, 0.0, 2.0, False),
    (2, 1, 16, 32, 16, 2, 0.0, 1.0, True), (1, 3, 17, 128, 32, 2, 0.2, 2.0, False),
    (1, 2, 33, 16, 128, 1, 0.3, 2.0, True), (2, 2, 47, 32, 64, 3, 0.1, 0.0, True),
    (1, 2, 49, 128, 16, 1, 0.1, 2.0, False), (1, 1, 64, 64, 32, 3, 0.1, 3.0, True),
    (8, 16, 35, 16, 32, 4, 0.1, 2.0, True), (16, 16, 18, 64, 16, 2, 0.1, 2.0, False),
    (1, 2, 40, 64, 32, 4, 0.2, -4.0, True), (1, 2, 50, 128, 16, 2, 0.2, -3.0, True),
    # lengths from which AUTO takes the chunk form (the two meet later with fewer components)
    (1, 1, 6, 64, 16, 4, 0.0, 2.0, False), (1, 3, 31, 128, 32, 2, 0.2, 2.0, False),
    (1, 2, 127, 128, 16, 1, 0.1, 2.0, False), (16, 16, 24, 64, 16, 2, 0.1, 2.0, False),
    (2, 2, 8, 32, 64, 3, 0.1, 0.0, True), (1, 2, 95, 64, 16, 1, 0.1, -3.0, True),
])
def test_chunk_matches_token_scan(B, H, T, Dk, Dv, J, std, mean, prior):
    _check(_inputs(B, H, T, Dk, Dv, J, 1300 + T + Dk + J, std, mean, prior))


@pytest.mark.parametrize("at", [(0,), (15,), (16, 31), (33,)])
def test_rerun_with_the_maximum_subtracted(at):
    """|delta| of 13 to 14 at the given tokens puts the sum over j below 2^-100.
    There a rounding of delta (2^-24 of it, three of them with the prediction's and
    the square's) moves e^{-delta^2/2} by delta^2 times as much: 196 * 3 * 2^-24 =
    3.5e-5 of r, in either form."""
    case = _inputs(1, 2, 34, 64, 32, 4, 1350, 0.1, 2.0, True)
    rng = np.random.default_rng(1351)
    for t in at:
        v = case[0]["v"][:, t]
        case[0]["v"][:, t] = workloads.round_bf16(np.sign(v) * rng.uniform(13.0, 14.0, v.shape))
    _check(case, tol=3.5e-5)


def test_chained_calls_and_float_output():
    """Two calls over the parts equal one over the whole (split inside a chunk),
    with o in fp32."""
    import torch
    case = _inputs(1, 2, 45, 64, 32, 4, 1360, 0.1, 2.0, True)
    inp, tmp, dec = case
    whole = _gpu(*case, "auto", out_dtype=torch.float32)
    cut = 21
    part = lambda d, sl: {n: (x if x is None or n in ("state", "prior") else np.ascontiguousarray(x[:, sl]))
                          for n, x in d.items()}
    first = _gpu(part(inp, slice(0, cut)), part(tmp, slice(0, cut)), np.ascontiguousarray(dec[:, :cut]),
                 "auto", out_dtype=torch.float32)
    i2, t2 = part(inp, slice(cut, None)), part(tmp, slice(cut, None))
    i2["state"], t2["prior"] = first[1].astype(np.float32), first[2].astype(np.float32)
    second = _gpu(i2, t2, np.ascontiguousarray(dec[:, cut:]), "auto", out_dtype=torch.float32)
    assert _rel(np.concatenate([first[0], second[0]], 1), whole[0]) <= TOL
    assert _rel(second[1], whole[1]) <= TOL and _rel(second[2], whole[2]) <= TOL


@pytest.mark.parametrize("B,H,T,Dk,Dv,J,chunk", [
    (1, 2, 1, 64, 16, 4, False), (1, 2, 5, 64, 16, 4, False), (1, 2, 7, 32, 16, 3, False),
    (1, 2, 17, 64, 32, 2, False), (1, 2, 17, 64, 64, 1, False), (1, 2, 64, 128, 16, 1, False),
    (17, 16, 40, 64, 16, 1, False), (33, 16, 20, 16, 16, 2, False), (33, 16, 32, 16, 16, 4, False),
    (1, 2, 32, 64, 16, 4, True), (1, 2, 48, 64, 16, 1, True), (33, 16, 144, 64, 16, 4, True),
])
def test_auto_takes_the_faster_form(B, H, T, Dk, Dv, J, chunk):
    """Short calls, and large grids of few components or short keys, on the token scan (its
    result to the bit); the others on the chunk form (other roundings)."""
    case = _inputs(B, H, T, Dk, Dv, J, 1380 + T + J, 0.1, 2.0, True)
    same = all(np.array_equal(x, y) for x, y in zip(_gpu(*case, "auto"), _gpu(*case, "recurrent")))
    assert same != chunk


def test_other_shapes_keep_the_token_scan():
    """J * Dk > 256 and J = 8: AUTO gives the token scan's result to the bit."""
    for Dk, J in ((128, 4), (64, 8)):
        case = _inputs(1, 2, 20, Dk, 16, J, 1370 + J, 0.1, 2.0, True)
        for x, y in zip(_gpu(*case, "auto"), _gpu(*case, "recurrent")):
            assert np.array_equal(x, y)
