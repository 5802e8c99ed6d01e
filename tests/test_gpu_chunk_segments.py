"""The chunk scan's chunks of 16 tokens in two segments (tokens 0 to 11, then 12
to 15): sequence lengths around every boundary, and a softmax sum outside the
fp32 range at each end of either segment, whose tokens then run again with the
maximum subtracted.  Bar as in test_gpu_parity.py: max |gpu - oracle| / max
|oracle| <= 2e-2 per (b, h) for bf16 inputs, and 1e-3 for the fp32 state and
responsibilities (products of fp32 values split into bf16 high parts and
residuals are good to about 2^-16; a token's coefficient that misses one of its
updates is off by whole percents)."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import NAMES, TOL_BF16, head_rel_err, to_device

pytestmark = pytest.mark.gpu

TOL_STATE = 1e-3


def _run(inp, tmp=None):
    import torch
    import paper_2609_39034_amd as sw
    dev = to_device(inp, "bf16")
    args = [dev[n] for n in NAMES]
    if tmp is None:
        o, s, r = sw.forward(*args, dev["state"], resp=True, algo="chunk")
        ref = oracle.forward(*(inp[n] for n in NAMES), inp["state"], want_resp=True)
    else:
        gk, gq = (torch.from_numpy(tmp[n]).to("cuda", torch.bfloat16) for n in ("gk", "gq"))
        o, s, p, r = sw.forward_temporal(*args, gk, gq, dev["state"],
                                         torch.from_numpy(tmp["prior"]).cuda(), resp=True)
        ref = oracle.forward(*(inp[n] for n in NAMES), inp["state"], want_resp=True,
                             gate_k_logit=tmp["gk"], gate_q_logit=tmp["gq"], prior_in=tmp["prior"])
    torch.cuda.synchronize()
    o, s, r = (x.float().cpu().numpy() for x in (o, s, r))
    assert head_rel_err(o, ref["o"], "o") <= TOL_BF16
    assert head_rel_err(s, ref["state"], "state") <= TOL_STATE
    assert head_rel_err(r, ref["resp"], "resp") <= TOL_STATE
    if tmp is not None:
        assert np.abs(p.cpu().numpy() - ref["prior"]).max() <= TOL_STATE


@pytest.mark.parametrize("T", [1, 11, 12, 13, 16, 17, 28, 29, 32, 33, 47, 49, 80, 81])
@pytest.mark.parametrize("Dk,Dv,J", [(16, 16, 1), (32, 32, 3), (64, 16, 4), (128, 8 * 2, 8)])
def test_lengths(T, Dk, Dv, J):
    inp = workloads.iid_inputs(1, 2, T, Dk, Dv, J, dtype="bf16", seed=900 + T, state_std=0.2)
    _run(inp)


# B * H * Dv / DB at 512 blocks and more: the variant without helper waves
@pytest.mark.parametrize("B,H,T,Dk,Dv,J", [(16, 16, 37, 16, 32, 2), (8, 16, 29, 64, 64, 1)])
def test_no_helper_waves(B, H, T, Dk, Dv, J):
    _run(workloads.iid_inputs(B, H, T, Dk, Dv, J, dtype="bf16", seed=950 + T, state_std=0.2))


@pytest.mark.parametrize("temporal", [False, True])
@pytest.mark.parametrize("at", [(0,), (11,), (12,), (15,), (5, 14), (16, 27), (28, 31), (39,)])
def test_rerun_of_a_segment(at, temporal):
    """|delta| of 13 to 14 at the given tokens puts the sum over j below 2^-100."""
    inp = workloads.iid_inputs(1, 2, 40, 64, 32, 4, dtype="bf16", seed=970, state_std=0.1)
    rng = np.random.default_rng(971)
    for t in at:
        v = inp["v"][:, t]
        inp["v"][:, t] = workloads.round_bf16(np.sign(v) * rng.uniform(13.0, 14.0, v.shape))
    _run(inp, workloads.temporal_inputs(1, 2, 40, 32, 4, dtype="bf16", seed=970, prior_state=True)
         if temporal else None)
