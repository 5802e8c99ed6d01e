"""The chunk scan takes its helper waves from the grid: five a block while a compute unit
gets one block, two, one or none where two or more share it.  A head's result must not
depend on that: the same heads run alone (five) and inside grids on either side of the
lines, with and without responsibilities (whose buffer decides for J = 3), and the
backward's recompute likewise.  Every variant does the same arithmetic; the bound is
fp32 rounding, 2^-20 of the largest value."""
import numpy as np
import pytest

import workloads
from gpu_helpers import NAMES, to_device

pytestmark = pytest.mark.gpu


def _close(x, y):
    assert np.abs(x - y).max() <= 2.0 ** -20 * np.abs(y).max()


GRIDS = [
    # J, Dk, Dv, heads (16 columns a block: one block a head, and so on)
    (1, 64, 16, 257), (1, 16, 16, 769), (1, 32, 16, 770), (1, 128, 16, 300),
    (1, 16, 32, 258), (1, 64, 32, 513), (2, 32, 16, 259), (2, 64, 16, 520),
    (3, 16, 16, 511), (3, 16, 16, 512), (3, 32, 16, 515), (4, 32, 16, 130), (1, 16, 64, 514),
]


@pytest.mark.parametrize("temporal", [False, True])
@pytest.mark.parametrize("J,Dk,Dv,heads", GRIDS)
def test_head_independent_of_grid(J, Dk, Dv, heads, temporal):
    import torch
    import paper_2609_39034_amd as sw
    T = 37
    inp = workloads.iid_inputs(heads, 1, T, Dk, Dv, J, dtype="bf16", seed=1700 + J, state_std=0.2)
    tmp = workloads.temporal_inputs(heads, 1, T, Dv, J, dtype="bf16", seed=1700, prior_state=True)
    dev = to_device(inp, "bf16")
    gates = [torch.from_numpy(tmp[n]).to("cuda", torch.bfloat16) for n in ("gk", "gq")]
    prior = torch.from_numpy(tmp["prior"]).cuda()

    def run(sel, resp):
        args = [dev[n][sel].contiguous() for n in NAMES]
        st = dev["state"][sel].contiguous()
        if temporal:
            out = sw.forward_temporal(*args, *(g[sel].contiguous() for g in gates), st,
                                      prior[sel].contiguous(), out_dtype=torch.float32, resp=resp)
        else:
            out = sw.forward(*args, st, out_dtype=torch.float32, resp=resp)
        torch.cuda.synchronize()
        return [x.cpu().numpy() for x in out]

    whole, kept = run(slice(None), False), run(slice(None), True)
    for h in (0, heads // 2, heads - 1):
        alone = run(slice(h, h + 1), True)
        for x, y in zip(whole, alone):
            _close(x[h:h + 1], y)
        for x, y in zip(kept, alone):
            _close(x[h:h + 1], y)


@pytest.mark.parametrize("J,Dk,Dv,heads", [(1, 64, 16, 257), (1, 32, 32, 300), (3, 16, 16, 512), (2, 32, 16, 259)])
def test_gradients_independent_of_grid(J, Dk, Dv, heads):
    import torch
    import paper_2609_39034_amd as sw
    T = 37
    inp = workloads.iid_inputs(heads, 1, T, Dk, Dv, J, dtype="bf16", seed=1710 + J, state_std=0.2)
    dev = to_device(inp, "bf16")
    go = torch.from_numpy(np.random.default_rng(1710).standard_normal((heads, T, 1, Dv))).to("cuda", torch.bfloat16)
    run = lambda sel: [x.cpu().numpy() for x in sw.backward(
        *(dev[n][sel].contiguous() for n in NAMES), dev["state"][sel].contiguous(), go[sel].contiguous())]
    whole = run(slice(None))
    for h in (0, heads - 1):
        for x, y in zip(whole, run(slice(h, h + 1))):
            _close(x[h:h + 1], y)
