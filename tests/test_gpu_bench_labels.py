"""The form that bench.py names for a line is the one that runs: where it names a chunk
form, AUTO's state differs in its last bits from the token-by-token scan's; where it
names that scan, the two are the same call.  Also that the source it names holds the
kernel it names."""
import os
import re

import numpy as np
import pytest

import bench
import workloads
from gpu_helpers import NAMES, to_device, torch_dtype

CSRC = os.path.join(bench.ROOT, "paper_2609_39034_amd", "csrc")
KINDS = ["forward", "temporal", "gated"]


def _code(name, seen):
    text = open(os.path.join(CSRC, name)).read()
    for inc in re.findall(r'^\s*#include\s+"([^"]+)"', text, re.M):
        if inc not in seen and os.path.exists(os.path.join(CSRC, inc)):
            seen.add(inc)
            text += _code(inc, seen)
    return text


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("cfg", [1, 2, 3, 5])
def test_source_holds_the_kernel(cfg, kind):
    _, kernel, source = bench.scan_kernel(kind, workloads.CONFIGS[cfg], "auto")
    assert re.search(r"__global__[^;{]*\b%s\(" % kernel, _code(source, set()))


@pytest.mark.gpu
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("cfg", [1, 2, 5])
def test_auto_runs_the_form_named(cfg, kind):
    import torch
    import paper_2609_39034_amd as sw
    c = workloads.CONFIGS[cfg]
    B, H, Dk, Dv, J = (c[x] for x in ("B", "H", "Dk", "Dv", "J"))
    T = min(c["T"], 256)
    tdt = torch_dtype(c["dtype"])
    dev = to_device(workloads.iid_inputs(B, H, T, Dk, Dv, J, dtype=c["dtype"], seed=71), c["dtype"])
    args = [dev[n] for n in NAMES]

    def run(algo):
        if kind == "forward":
            return sw.forward(*args, dev["state"], algo=algo)[1]
        if kind == "gated":
            dec = workloads.gated_inputs(B, H, T, Dk, J, dtype=c["dtype"], seed=71)["decay"]
            return sw.forward_gated(*args, torch.from_numpy(dec).to("cuda", tdt), dev["state"],
                                    algo=algo)[1]
        tmp = workloads.temporal_inputs(B, H, T, Dv, J, dtype=c["dtype"], seed=71)
        gates = [torch.from_numpy(tmp[n]).to("cuda", tdt) for n in ("gk", "gq")]
        return sw.forward_temporal(*args, *gates, dev["state"], algo=algo)[1]

    chunk = bench.scan_kernel(kind, c, "auto")[0]
    auto, token = (run(a).cpu().numpy() for a in ("auto", "recurrent"))
    assert np.array_equal(auto, token) != chunk
