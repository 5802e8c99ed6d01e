"""The token-by-token scan picks its key rows per lane from the grid size: 4 on
grids under 256 blocks, 16 (J <= 4) on larger ones.  A head's result must not
depend on which layout its batch gets.  The same heads run alone (small grid)
and inside a 256-head batch (large grid); both must match the fp64 oracle to the
fp32 bar, and each other to fp32 rounding.
"""
import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import NAMES, head_rel_err, to_device

pytestmark = pytest.mark.gpu


def _run(inp, gated_decay=None):
    import torch
    import paper_2609_39034_amd as sw
    dev = to_device(inp, "f32")
    if gated_decay is None:
        res = sw.forward(*(dev[n] for n in NAMES), dev["state"], algo="recurrent")
    else:
        dec = torch.from_numpy(np.ascontiguousarray(gated_decay)).cuda()
        res = sw.forward_gated(*(dev[n] for n in NAMES), dec, dev["state"], algo="recurrent")
    torch.cuda.synchronize()
    return [x.cpu().numpy().astype(np.float64) for x in res[:2]]


@pytest.mark.parametrize("gated", [False, True])
def test_head_independent_of_layout(gated):
    B, H, T, D, J = 16, 16, 23, 64, 4          # 256 heads: 16 rows per lane
    big = workloads.iid_inputs(B, H, T, D, D, J, dtype="f32", seed=901, state_std=0.2)
    dec = workloads.gated_inputs(B, H, T, D, J, dtype="f32", seed=901)["decay"] if gated else None
    o_big, s_big = _run(big, dec)
    for b, h in [(0, 0), (7, 9), (15, 15)]:
        one = {n: big[n][b:b + 1, :, h:h + 1].copy() for n in NAMES}   # one head: 4 rows per lane
        one["state"] = big["state"][b:b + 1, h:h + 1].copy()
        d1 = dec[b:b + 1, :, h:h + 1].copy() if gated else None
        o1, s1 = _run(one, d1)
        ref = oracle.forward(*(one[n] for n in NAMES), one["state"], decay_logit=d1)
        eo_big = head_rel_err(o_big[b:b + 1, :, h:h + 1], ref["o"], "o")
        eo_one = head_rel_err(o1, ref["o"], "o")
        es_one = head_rel_err(s1, ref["state"], "state")
        ediff = head_rel_err(o1, o_big[b:b + 1, :, h:h + 1], "o")
        sdiff = head_rel_err(s1, s_big[b:b + 1, h:h + 1], "state")
        print("head (%d,%d): o big %.2e one %.2e, state one %.2e, one vs big o %.2e state %.2e"
              % (b, h, eo_big, eo_one, es_one, ediff, sdiff))
        assert eo_big <= 1e-4 and eo_one <= 1e-4 and es_one <= 1e-4
        assert ediff <= 1e-5 and sdiff <= 1e-5
