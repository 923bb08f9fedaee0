"""The 3x3 convolutions whose K slices run side by side in one block: every
channel width (two slices, four, four of two chunks), both strides, float32
and bf16, on grids with ragged tiles, one map per launch (two-row tiles) and
eight maps per launch (the larger tiles, and the halo tilings that sum the
same slices).  Every layer elementwise against the oracle convolution of its
GPU input, and the group launch bit for bit equal to separate launches (the
tiles sum in the same order).  The upsamplings of the same networks (one launch
for all stages, or one each) likewise."""

import copy

import numpy as np
import pytest

import synth
from oracle import network as N
from paper_2608_08330_amd import rtcc as R
from tests.helpers import check_conv_layers, make_ctx, run_frame

pytestmark = pytest.mark.gpu

# (name, precision, c_pfn, stages, up_channels, (H, W) cells)
SHAPES = [
    ("widths", "bf16", 64, ((2, 128, 2), (2, 256, 2)), 128, (45, 61)),       # 2, 4 and 4 x 2 slices
    ("edges", "bf16", 64, ((1, 64, 2),), 0, (2, 15)),                        # below one tile
    ("one_row", "bf16", 128, ((2, 64, 2),), 128, (1, 33)),
    ("narrow", "bf16", 64, ((1, 96, 1), (2, 32, 1)), 128, (67, 131)),        # 96 channels: no 64-channel tiles
    ("deep_entry", "bf16", 256, ((2, 96, 1), (1, 64, 1)), 64, (66, 127)),    # stride 2 at 256 channels
    ("upsample", "bf16", 64, ((1, 64, 1), (2, 128, 1), (2, 256, 1)), 128, (35, 53)),  # x1, x2, x4 with a crop
    ("wide_up", "bf16", 64, ((2, 128, 1), (2, 256, 1)), 256, (30, 46)),      # two blocks of 128 output channels
    # eight maps: more blocks than the one-group upsampling takes, 64 / 128 / 256 input channels
    ("many_up", "bf16", 64, ((1, 64, 1), (2, 128, 1), (2, 256, 1)), 128, (197, 203)),
    # ... and two blocks of 128 output channels; eight maps: one group per block, four
    ("some_wide_up", "bf16", 64, ((1, 64, 1), (2, 256, 1)), 256, (150, 170)),
    ("many_wide_up", "bf16", 64, ((1, 64, 1), (2, 256, 1)), 256, (170, 190)),
    # one map: 888 blocks, which run all at once with two wavefronts each; eight: the three groups of a pixel in one block
    ("up_384", "bf16", 64, ((1, 64, 1),), 384, (135, 140)),
    ("fp32", "fp32", 64, ((2, 32, 2),), 32, (47, 95)),
    # group launches by the halo tilings: 8 rows of 16 pixels, strides 1 and 2 ...
    ("halo", "bf16", 128, ((2, 256, 2), (2, 256, 1)), 128, (90, 100)),
    ("fp32_128", "fp32", 128, ((1, 128, 1), (2, 128, 1)), 64, (47, 95)),
    ("fp32_64", "fp32", 64, ((1, 64, 1), (2, 128, 1)), 64, (130, 131)),
    # ... 4 rows
    ("halo4", "bf16", 256, ((1, 128, 1),), 0, (40, 60)),
]


def _config(precision, c_pfn, stages, up, grid):
    cfg = copy.deepcopy(synth.config("t_max"))
    H, W = grid
    cfg.update(K=8, n_points=900, precision=precision, c_pfn=c_pfn, stages=stages, up_channels=up, fusion="max",
               x_range=(-0.2 * W, 0.2 * W), y_range=(-0.2 * H, 0.2 * H), pillar=0.4, logit_threshold=1.0)
    return cfg


def _frame(cfg):
    rng = np.random.default_rng(17)
    pts = []
    for k in range(cfg["K"]):
        p = np.empty((cfg["n_points"] - 7 * k, 4), np.float32)
        for c, r in enumerate((cfg["x_range"], cfg["y_range"], cfg["z_range"], (0.0, 1.0))):
            p[:, c] = rng.uniform(r[0], r[1], len(p))
        pts.append(p)
    w = {}
    for name, shape, fan in synth.network_layers(cfg):
        w[name] = (rng.standard_normal(shape) * (0.1 if fan is None else np.sqrt(2.0 / fan))).astype(np.float32)
    poses = np.zeros((cfg["K"], 3))
    poses[1:, 0] = 0.3
    return dict(points=pts, poses=poses, weights=w)


def _run(ctx, fr, group):
    if not group:
        return run_frame(ctx, fr)
    import time
    R.rtcc_begin_frame(ctx, time.monotonic() - 1.0)
    R.rtcc_release_branches(ctx, [dict(agent=k, points=p, pose=fr["poses"][k], arrival_t=0.0)
                                  for k, p in enumerate(fr["points"])])
    return R.rtcc_join_and_detect(ctx)


@pytest.mark.parametrize("name,precision,c_pfn,stages,up,grid", SHAPES, ids=[s[0] for s in SHAPES])
def test_slices_against_the_oracle_and_between_batch_sizes(name, precision, c_pfn, stages, up, grid):
    print("conv slices: %s" % name, flush=True)
    cfg = _config(precision, c_pfn, stages, up, grid)
    fr = _frame(cfg)
    pw = N.prepared_weights(cfg, fr["weights"])
    n_layers = sum(n for _s, _c, n in stages)
    with make_ctx(cfg, fr) as ctx:
        plans = [R.rtcc_conv_plan(ctx, l) for l in range(n_layers)]
        # every layer of these shapes but those of 96 input channels, whose
        # pixels are no 128, 256 or 512 bytes (test_conv_plan.py has the rule)
        ci, l = c_pfn, 0
        for stride, co, n in stages:
            for s in (stride,) + (1,) * (n - 1):
                slices = {128: 2, 256: 4, 512: 4}.get(ci * (2 if precision == "bf16" else 4))
                if slices:
                    assert tuple(plans[l]) == (2 if s == 1 else 4, slices), (l, plans)
                ci, l = co, l + 1
        got = []
        for group in (False, True):
            _run(ctx, fr, group)
            for k in (0, cfg["K"] - 1):
                check_conv_layers(ctx, cfg, pw, k)
            got.append([R.rtcc_get_tensor(ctx, R.RTCC_T_CONV_OUT, (l << 8) | k, np.uint8)
                        for l in range(n_layers) for k in range(cfg["K"])])
            if up:
                got[-1] += [R.rtcc_get_tensor(ctx, R.RTCC_T_SLOT, k, np.uint8) for k in range(cfg["K"])]
        for a, b in zip(*got):
            assert np.array_equal(a, b)
