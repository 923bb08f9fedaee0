"""Node times read right behind a join: the join returns when its last kernel
(the selection, or the export of a frame without suppression) has handed over
the result, and the times are there whatever the event behind it has done."""

import copy

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
