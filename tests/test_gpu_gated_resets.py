"""Gated SwiLA with gates that are closed hard or altogether (decay logits of -50 to
-inf, a reset of the state) at the first, a middle and the last token of a chunk of
16, in every form that runs chunk by chunk: fp32 inputs, bf16 inputs with and without
the temporal priors, and the bf16 kernel for J = 4, Dk = 128.  The gates after a
closed one still count, to the precision of the form's products: 3e-6 of the state
and outputs (2-norm) with three bf16 parts to an operand, as for open gates, and
2^-14 with two (a product is good to about 2^-16 of its size)."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import NAMES, to_device, torch_dtype

pytestmark = pytest.mark.gpu

FORMS = [
    # dtype, temporal, Dk, J
    ("f32", False, 64, 4), ("f32", True, 32, 3), ("f32", False, 128, 1),
    ("bf16", True, 64, 4), ("bf16", True, 16, 2),
    ("bf16", False, 64, 4), ("bf16", False, 128, 3), ("bf16", False, 128, 4),
]


def _rel(x, y):
    return np.linalg.norm(x - y) / max(np.linalg.norm(y), 1e-30)


def _check(dtype, temporal, Dk, J, close):
    import torch
    import paper_2609_39034_amd as sw
    B, H, T, Dv = 1, 3, 127 if (Dk, J) == (128, 1) else 43, 16   # (a length that AUTO gives the chunk form)
    inp = workloads.iid_inputs(B, H, T, Dk, Dv, J, dtype=dtype, seed=1700 + Dk + J, state_std=0.2)
    dec = workloads.gated_inputs(B, H, T, Dk, J, dtype=dtype, seed=1700, mean=2.0)["decay"]
    close(dec)
    dev = to_device(inp, dtype)
    cu = lambda x: torch.from_numpy(x).to("cuda", torch_dtype(dtype))
    kw, okw = {}, {}
    if temporal:
        tmp = workloads.temporal_inputs(B, H, T, Dv, J, dtype=dtype, seed=1700, prior_state=True)
        kw = dict(gate_k_logit=cu(tmp["gk"]), gate_q_logit=cu(tmp["gq"]),
                  prior_in=torch.from_numpy(tmp["prior"]).cuda())
        okw = dict(gate_k_logit=tmp["gk"], gate_q_logit=tmp["gq"], prior_in=tmp["prior"])
    out = sw.forward_gated(*(dev[n] for n in NAMES), cu(dec), dev["state"], resp=True,
                           out_dtype=torch.float32, **kw)
    torch.cuda.synchronize()
    ref = oracle.forward(*(inp[n] for n in NAMES), inp["state"], decay_logit=dec, want_resp=True, **okw)
    tol = 3e-6 if dtype == "f32" or temporal else 2.0 ** -14
    for name, x in zip(("o", "state", "prior", "resp") if temporal else ("o", "state", "resp"), out):
        e = _rel(x.cpu().numpy().astype(np.float64), ref[name])
        print(dtype, temporal, Dk, J, name, e)
        assert e <= tol, (name, e)


@pytest.mark.parametrize("dtype,temporal,Dk,J", FORMS)
@pytest.mark.parametrize("logit", [-50.0, -1e4, -1e9, float(np.finfo(np.float32).min), -np.inf])
@pytest.mark.parametrize("at", [0, 3, 15, 21, 42])
def test_closed_gate(dtype, temporal, Dk, J, logit, at):
    """One key index of one component of head 0, every second key index of the last
    component of head 1, and every gate of head 2 closed at token ``at``."""
    if dtype == "bf16":
        logit = max(logit, -3.3e38) if np.isfinite(logit) else logit   # (finite in bf16)

    def close(dec):
        dec[0, at, 0, 0, 5] = logit
        dec[0, at, 1, J - 1, ::2] = logit
        dec[0, at, 2] = logit
    _check(dtype, temporal, Dk, J, close)


@pytest.mark.parametrize("dtype,temporal,Dk,J", FORMS)
def test_gates_closed_in_a_row(dtype, temporal, Dk, J):
    """Closed gates at neighbouring tokens and across a chunk edge."""
    def close(dec):
        dec[0, 14:18, 0] = -np.inf
        dec[0, 4, 1] = -np.inf
        dec[0, 5:9, 1, :, 1::2] = -60.0
        dec[0, 30, 2, 0] = -1e9
        dec[0, 31, 2, 0, 3] = -np.inf
    _check(dtype, temporal, Dk, J, close)
