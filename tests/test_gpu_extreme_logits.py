"""Key- and query-prior logits at the limits of fp32 (masks of the type's lowest value, on
one component, all but one, or all of them; the largest value; -inf on some) on every
form that takes fp32 inputs: the chunk form (which AUTO takes here) gives what the
token-by-token scan gives.  Logits of 2.4e38 and more overflow when they are multiplied
by log2(e).  (Where all components of a column are that large, both forms lose the
errors beside them, as lk - delta^2 / 2 does in 64 bits too.)"""
import numpy as np
import pytest

import workloads
from gpu_helpers import NAMES, to_device

pytestmark = pytest.mark.gpu

LOW, HIGH = float(np.finfo(np.float32).min), float(np.finfo(np.float32).max)
MASKS = {
    "one": lambda x: x.__setitem__((slice(None), 0), LOW),
    "all but one": lambda x: x.__setitem__((slice(None), slice(1, None)), LOW),
    "all": lambda x: x.__setitem__(slice(None), LOW),
    "all high": lambda x: x.__setitem__(slice(None), HIGH),
    "one high": lambda x: x.__setitem__((slice(None), 1), HIGH),
    "two, different": lambda x: (x.__setitem__(slice(None), LOW), x.__setitem__((slice(None), 1), 0.8 * LOW)),
    "infinite": lambda x: x.__setitem__((slice(None), 0), -np.inf),
}


@pytest.mark.parametrize("form", ["plain", "gated", "temporal", "gated_temporal"])
@pytest.mark.parametrize("which", list(MASKS))
@pytest.mark.parametrize("J", [2, 3, 4])
def test_masks(form, which, J):
    import torch
    import paper_2609_39034_amd as sw
    B, H, T, Dk, Dv = 1, 2, 37, 32, 16
    inp = workloads.iid_inputs(B, H, T, Dk, Dv, J, dtype="f32", seed=1900 + J, state_std=0.1)
    tmp = workloads.temporal_inputs(B, H, T, Dv, J, dtype="f32", seed=1900, prior_state=True)
    dec = workloads.gated_inputs(B, H, T, Dk, J, dtype="f32", seed=1900, mean=2.0)["decay"]
    for n in NAMES[4:6]:                # tokens 5 and 16 .. 18 of head 1
        for t in (5, 16, 17, 18):
            MASKS[which](np.moveaxis(inp[n][0, t, 1], 0, 0)[None])
    dev = to_device(inp, "f32")
    cu = lambda x: torch.from_numpy(x).cuda()
    kw = {}
    if "temporal" in form:
        kw = dict(gate_k_logit=cu(tmp["gk"]), gate_q_logit=cu(tmp["gq"]), prior_in=cu(tmp["prior"]))
    args = [dev[n] for n in NAMES]
    res = []
    for algo in ("recurrent", "auto"):
        if "gated" in form:
            out = sw.forward_gated(*args, cu(dec), dev["state"], resp=True, algo=algo, **kw)
        elif form == "temporal":
            out = sw.forward_temporal(*args, kw["gate_k_logit"], kw["gate_q_logit"], dev["state"],
                                      kw["prior_in"], resp=True, algo=algo)
        else:
            out = sw.forward(*args, dev["state"], resp=True, algo=algo)
        torch.cuda.synchronize()
        res.append([x.cpu().numpy().astype(np.float64) for x in out])
    for i, (x, y) in enumerate(zip(*res)):
        assert np.isfinite(x).all()
        e = np.linalg.norm(x - y) / np.linalg.norm(x)
        print(form, which, J, i, e)
        assert e <= 3e-6, (i, e)
