"""Node times read right behind a join: the join returns when its last kernel
(the selection, or the export of a frame without suppression) has handed over
the result, and the times are there whatever the event behind it has done."""

import copy
import time

import numpy as np
import pytest

import synth
from paper_2608_08330_amd import rtcc as R
from tests.helpers import make_ctx, run_frame

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap", (0, 512), ids=("no_nms", "nms"))
def test_node_times_right_behind_the_join(cap):
    cfg = copy.deepcopy(synth.config("t_max"))
    cfg["nms_max_candidates"] = cap
    fr = synth.make_frame(cfg, 3)
    with make_ctx(cfg, fr, node_timing=1) as ctx:
        for _ in range(100):
            run_frame(ctx, fr)
            assert (R.rtcc_node_times(ctx)[-4:-1] > 0.0).all()  # fusion, head, decode


@pytest.mark.parametrize("group", (False, True), ids=("each", "group"))
def test_the_input_node_is_the_launch_that_runs(group):
    """The inputs of a group are read by one kernel, with node times as without:
    every member's input node, measured on the group's stream, is over before
    its pillar stage and spans the same launch."""
    cfg = copy.deepcopy(synth.config("t_max"))
    fr = synth.make_frame(cfg, 3)
    with make_ctx(cfg, fr, node_timing=1) as ctx:
        for _ in range(20):
            if group:
                R.rtcc_begin_frame(ctx, time.monotonic() - 1.0)
                R.rtcc_release_branches(ctx, [dict(agent=k, points=p, pose=fr["poses"][k], arrival_t=0.0)
                                              for k, p in enumerate(fr["points"])])
                R.rtcc_join_and_detect(ctx)
            else:
                run_frame(ctx, fr)
            h2d = R.rtcc_node_times(ctx)[:-4].reshape(cfg["K"], -1)[:, 0]
            assert (h2d > 0.0).all()
            if group:  # recorded one after the other, on one stream
                assert (np.diff(h2d) <= 0.0).all(), h2d
