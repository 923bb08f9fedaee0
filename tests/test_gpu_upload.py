"""Inputs from pinned host memory: one kernel copies a whole group's points up
to a size, a copy per agent beyond.  Frames on both sides of that size, with
empty and single-point inputs and with agents whose inputs are on the device,
leave the canvases that device inputs leave, bit for bit."""

import copy
import time

import numpy as np
import pytest
import torch

import synth
from paper_2608_08330_amd import rtcc as R
from tests.helpers import make_ctx

pytestmark = pytest.mark.gpu

# points of the agents; sums on both sides of 24,576 for one, 40,000 (131,072 SERIAL) per agent of a group whose
# input is in host memory
COUNTS = [(0, 1, 257), (24576, 24577, 3), (40001, 40000, 39999), (40001, 40000, 40000), (131073, 131072, 131072)]


# with graphs, more than six branches released apart copy whatever the size
@pytest.mark.parametrize("agents,graphs", [(3, 0), (8, 1)], ids=("eager", "graphs"))
@pytest.mark.parametrize("serial", (False, True), ids=("streams", "serial"))
@pytest.mark.parametrize("group", (False, True), ids=("each", "group"))
def test_host_inputs_equal_device_inputs(group, serial, agents, graphs):
    cfg = copy.deepcopy(synth.config("t_max"))
    cfg.update(K=agents, n_points=100)
    fr = synth.make_frame(cfg, 5)
    rng = np.random.default_rng(9)
    box = (cfg["x_range"], cfg["y_range"], cfg["z_range"], (0.0, 1.0))
    kw = dict(use_graphs=graphs)
    if serial:
        kw["exec"] = R.RTCC_EXEC_SERIAL
    with make_ctx(cfg, fr, max_points=max(map(max, COUNTS)), **kw) as ctx:
        for counts in COUNTS:
            counts = counts + (100, 0, 2000, 7, 300)[:agents - 3]
            print("upload: %s" % (counts,), flush=True)
            pts = [np.stack([rng.uniform(r[0], r[1], n) for r in box], 1).astype(np.float32) for n in counts]
            dev = [torch.from_numpy(p).cuda() if len(p) else torch.zeros((1, 4), device="cuda") for p in pts]
            torch.cuda.synchronize()
            got = []
            for where in ("device", "host", "mixed"):
                ev = [dict(agent=k, device=1, points=dev[k].data_ptr(), n=counts[k], pose=fr["poses"][k], arrival_t=0.0)
                      if where == "device" or (where == "mixed" and k == 1) else
                      dict(agent=k, points=pts[k], pose=fr["poses"][k], arrival_t=0.0) for k in range(agents)]
                R.rtcc_begin_frame(ctx, time.monotonic() - 1.0)
                for part in ([ev] if group else [[e] for e in ev]):
                    R.rtcc_release_branches(ctx, part)
                R.rtcc_join_and_detect(ctx)
                got.append([R.rtcc_get_tensor(ctx, R.RTCC_T_CANVAS, k, np.uint8) for k in range(agents)])
            for other in got[1:]:
                for a, b in zip(got[0], other):
                    assert np.array_equal(a, b)
