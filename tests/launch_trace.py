"""The kernel launches of a call, from torch's profiler: which kernel ran, with
how many workgroups of how many threads and how much dynamic LDS."""
import json
import os
import tempfile
from collections import namedtuple

import pytest

Launch = namedtuple("Launch", "kernel groups threads lds")


def launches(run):
    """The library's launches while ``run()`` is called, in order."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        run()
        torch.cuda.synchronize()
    fd, path = tempfile.mkstemp(suffix=".json")
    os.close(fd)
    try:
        prof.export_chrome_trace(path)
        with open(path) as fh:
            events = json.load(fh)["traceEvents"]
    finally:
        os.remove(path)
    calls = sorted((e for e in events if e.get("name") == "hipLaunchKernel" and "kernel" in e.get("args", {})),
                   key=lambda e: e["ts"])
    out = []
    for e in calls:
        a = e["args"]
        # "void lbm::(anonymous namespace)::k_node<0, false>(lbm::StepArgs)" -> "k_node<0, false>"
        name = a["kernel"].replace("(anonymous namespace)::", "").split("(")[0].split("::")[-1]
        gx, gy, gz = a["grid"]
        out.append(Launch(name, gx * gy * gz, a["block"][0], a["shared memory"]))
    if not out:
        pytest.skip("the profiler records no launches here")
    return out
