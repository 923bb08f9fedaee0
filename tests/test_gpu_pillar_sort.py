"""The pillar sort at sizes off the common path, bit-exact against the
oracle (pillar cells, counts and the points each pillar feeds to the
point-feature net): an agent with three agents' clouds (586 point blocks
over 128 tiles of cells), and an agent with 15,000,000 points on 4,096
cells, where each of the two tiles holds far more points than the tile
sort keeps in registers and every pillar is over the cap."""

import sys
import time

import numpy as np
import pytest

import synth
from oracle import network as N
from paper_2608_08330_amd import rtcc as R
from tests.helpers import check_members, make_ctx, run_frame

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _check_pillars(ctx, cfg, points, agent):
    pil = N.pillars(N.cell_ids(points, cfg), cfg["max_pts"])
    cells = R.rtcc_get_tensor(ctx, R.RTCC_T_PILLAR_CELLS, agent, np.int32)
    counts = R.rtcc_get_tensor(ctx, R.RTCC_T_PILLAR_COUNTS, agent, np.int32)
    assert np.array_equal(cells, pil["cells"].astype(np.int32)), agent
    assert np.array_equal(counts, pil["counts"].astype(np.int32)), agent
    check_members(ctx, cfg, points, agent)


def test_many_point_blocks_over_many_tiles():
    # c5 geometry (128 tiles); agent 0 holds three agents' clouds, 586 point
    # blocks
    cfg = synth.config("c5")
    fr = synth.make_frame(cfg)
    big = np.ascontiguousarray(np.concatenate(fr["points"][:3]))
    fr["points"] = [big] + fr["points"][1:]
    _say("c5 with %d points in agent 0" % len(big))
    with make_ctx(cfg, fr, max_points=len(big)) as ctx:
        run_frame(ctx, fr)
        _check_pillars(ctx, cfg, big, 0)
        _check_pillars(ctx, cfg, fr["points"][1], 1)


def test_fifteen_million_points_on_two_tiles():
    # c1 geometry (2 tiles of cells, 4,096 cells); 15,000,000 points in
    # agent 0: 29,297 point blocks, 7.5 million points per tile
    cfg = synth.config("c1")
    fr = synth.make_frame(cfg)
    n = 15_000_000
    rng = np.random.default_rng(11)
    big = np.empty((n, 4), np.float32)
    big[:, 0] = rng.uniform(cfg["x_range"][0], cfg["x_range"][1], n)
    big[:, 1] = rng.uniform(cfg["y_range"][0], cfg["y_range"][1], n)
    big[:, 2] = rng.uniform(cfg["z_range"][0], cfg["z_range"][1], n)
    big[:, 3] = rng.uniform(0.0, 1.0, n)
    fr["points"] = [big] + fr["points"][1:]
    _say("c1 with %d points in agent 0" % n)
    with make_ctx(cfg, fr, max_points=n) as ctx:
        run_frame(ctx, fr)
        _check_pillars(ctx, cfg, big, 0)
        _check_pillars(ctx, cfg, fr["points"][1], 1)


# (H, W) cells and points: one block per agent up to 8,192 points and 16,384
# cells or 4,096 points and 65,536 cells (half the points for a group), tiles of
# 512 cells up to 131,072 cells and of 2,048 above
@pytest.mark.parametrize("grid,n", [
    ((1, 1), 40), ((3, 5), 0), ((3, 5), 1), ((128, 128), 1024), ((128, 129), 1025), ((127, 129), 16384),
    ((256, 256), 16384), ((256, 256), 16385), ((128, 128), 8192), ((128, 128), 8193),
    ((128, 129), 4096), ((128, 129), 4097), ((256, 256), 4096), ((256, 257), 4096),
    ((128, 129), 2048), ((128, 129), 2049),
    ((256, 257), 1023), ((11, 5958), 5000), ((512, 1), 513),
    ((256, 512), 20000), ((257, 511), 20000), ((2, 70001), 30000),
])
def test_sizes_at_the_edges_of_the_paths(grid, n):
    cfg = synth.config("c1")
    H, W = grid
    cfg.update(K=2, n_points=max(n, 1), pillar=0.5, x_range=(0.0, 0.5 * W), y_range=(0.0, 0.5 * H))
    rng = np.random.default_rng(H * 1000003 + W * 101 + n)
    _say("%d x %d cells, %d points" % (H, W, n))
    clouds = []
    for k in range(2):
        p = np.empty((n, 4), np.float32)
        # two thirds spread (some outside), the rest crowded into a few cells
        p[:, 0] = rng.uniform(-0.3, 0.5 * W + 0.3, n)
        p[:, 1] = rng.uniform(-0.3, 0.5 * H + 0.3, n)
        m = n // 3
        p[:m, 0] = 0.5 * rng.integers(max(0, W - 3), W, m) + 0.2
        p[:m, 1] = 0.5 * rng.integers(max(0, H - 2), H, m) + 0.2
        p[:, 2] = rng.uniform(cfg["z_range"][0], cfg["z_range"][1], n)
        p[:, 3] = rng.uniform(0.0, 1.0, n)
        clouds.append(p[rng.permutation(n)])
    fr = dict(points=clouds, poses=np.zeros((2, 3)), weights=synth.make_weights(synth.config("c1")))
    with make_ctx(cfg, fr, max_points=max(n, 1)) as ctx:
        for points, group in ((clouds, False), (clouds[::-1], False), (clouds, True)):
            if group:
                R.rtcc_begin_frame(ctx, time.monotonic() - 1.0)
                R.rtcc_release_branches(ctx, [dict(agent=k, points=p, pose=fr["poses"][k], arrival_t=0.0)
                                              for k, p in enumerate(points)])
                R.rtcc_join_and_detect(ctx)
            else:
                run_frame(ctx, fr, points=points)
            for k in range(2):
                _check_pillars(ctx, cfg, points[k], k)
                canvas = R.rtcc_get_tensor(ctx, R.RTCC_T_CANVAS, k, np.float32).reshape(H * W, -1)
                pil = N.pillars(N.cell_ids(points[k], cfg), cfg["max_pts"])
                pw = N.prepared_weights(cfg, fr["weights"])
                ref = N.pfn_canvas(points[k], pil, pw["pfn_w"], pw["pfn_b"], cfg)
                assert np.max(np.abs(canvas - ref.reshape(H * W, -1)), initial=0.0) <= 1e-5
