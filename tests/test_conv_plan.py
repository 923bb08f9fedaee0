"""The conv planner through the C ABI (host computation, no GPU): the c5
plan at 256 CUs for launches over 1, 2, 4 and 8 agents' maps, and on every
layer shape of the configs, for several CU counts and every batch size, the
invariant that lets a group release equal separate releases bit for bit:
all tilings a layer takes accumulate each output element in the same order
(the same channel chunks and taps, so the same chunk width and one wave
group), with the same K split.  Where the K slices of a tile are summed side by
side in one block, and from how many maps on by the halo tilings, is not part of
the C ABI: the planner is compiled into a small program of its own."""

import os
import subprocess

import pytest

import synth
from paper_2608_08330_amd import rtcc as R

IMPLICIT = (0,)         # implicit GEMM, 128 x 128 tiles
IMPLICIT256 = (12,)     # 256 x 128 tiles, every other tile's K steps backwards
HALO_RULE = (1, 2, 9)   # halo tilings whose chunk width follows the channel rule
HALO_C64 = (8, 10)      # halo tilings with 64-byte chunks
HALO_S2 = (3, 4, 11)    # stride-2 halo tilings (64-byte chunks)
TWO_GROUPS = (5, 6)     # split chunk sums (another order): never planned


def _lib():
    return R.load("host")


def _layers(name):
    cfg = synth.config(name)
    h = round((cfg["y_range"][1] - cfg["y_range"][0]) / cfg["pillar"])
    w = round((cfg["x_range"][1] - cfg["x_range"][0]) / cfg["pillar"])
    c = cfg["c_pfn"]
    out = []
    for stride, co, n in cfg["stages"]:
        for l in range(n):
            s = stride if l == 0 else 1
            ho, wo = -(-h // s), -(-w // s)
            out.append((h, w, c, ho, wo, co, s))
            h, w, c = ho, wo, co
    return cfg, out


def _family(variant, ci, elt):
    if variant in IMPLICIT:
        return "implicit"
    if variant in IMPLICIT256:
        return "implicit256"
    if variant in HALO_RULE:
        return ("halo", 128 if (ci * elt) % 128 == 0 and ci * elt >= 512 else 64)
    if variant in HALO_C64 or variant in HALO_S2:
        return ("halo", 64)
    raise AssertionError("tiling %d is not planned" % variant)


def test_c5_plans_at_256_cus():
    _cfg, layers = _layers("c5")
    lib = _lib()
    want = {1: (12, 1, 1, 3, 8, 8, 8, 8, 4, 2, 2, 2, 2),
            2: (12, 1, 1, 11, 10, 10, 10, 10, 4, 2, 2, 2, 2),
            4: (12, 1, 1, 11, 10, 10, 10, 10, 3, 1, 1, 1, 1),
            8: (12, 1, 1, 11, 10, 10, 10, 10, 11, 9, 9, 9, 9)}
    for maps, v in want.items():
        got = [R.rtcc_conv_tiling(*s, 256, maps, lib=lib) for s in layers]
        assert got == [(x, 1) for x in v], maps


@pytest.mark.parametrize("name", ["c1", "c2", "c3", "c5", "t_var", "t_max"])
@pytest.mark.parametrize("n_cu", [80, 104, 228, 256, 304])
def test_every_batch_size_accumulates_alike(name, n_cu):
    cfg, layers = _layers(name)
    bf16 = cfg["precision"] == "bf16"
    elt = 2 if bf16 else 4
    lib = _lib()
    for shape in layers:
        plans = [R.rtcc_conv_tiling(*shape, n_cu, m, bf16=bf16, lib=lib) for m in range(1, 17)]
        fams = {_family(v, shape[2], elt) for v, _sp in plans}
        assert len(fams) == 1, (shape, plans)
        assert len({sp for _v, sp in plans}) == 1, (shape, plans)
        for v, _sp in plans:
            assert v not in TWO_GROUPS
            if shape[6] == 1:
                assert v not in HALO_S2
            elif v not in IMPLICIT + IMPLICIT256:
                assert v in HALO_S2


PROGRAM = r"""
#include <cstdio>
#include "conv_plan.hpp"
using namespace rtcc::kern;
int main() {
    int b, s[8];
    while (std::scanf("%d %d %d %d %d %d %d %d %d", &b, s, s + 1, s + 2, s + 3, s + 4, s + 5, s + 6, s + 7) == 9) {
        const ConvPlan p = conv_plan(b != 0, s[0], s[1], s[2], s[3], s[4], s[5], s[6], s[7]);
        std::printf("%d %d %d %zu\n", int(p.slices), p.splits, p.halo_maps, p.ws_bytes);
    }
}
"""


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    d = tmp_path_factory.mktemp("planner")
    src = os.path.join(os.path.dirname(R.__file__), "csrc", "kernels")
    (d / "main.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I" + src, str(d / "main.cpp"), os.path.join(src, "conv_plan.cpp"),
                    "-o", str(d / "planner")], check=True)

    def plan(bf16, Ci, Ho, Wo, Co, stride, n_cu=256):
        """(slices side by side or 0, maps from which the halo tilings sum them or None)"""
        shape = (int(bf16), Ho * stride, Wo * stride, Ci, Ho, Wo, Co, stride, n_cu)
        r = subprocess.run([str(d / "planner")], input=" ".join(map(str, shape)), text=True, check=True,
                           stdout=subprocess.PIPE).stdout.split()
        if not int(r[0]):
            return 0, None
        assert int(r[3]) == 0  # no partial sums in memory
        return int(r[1]), int(r[2]) if int(r[2]) < 1 << 30 else None
    return plan


@pytest.mark.parametrize("shape,want", [
    # widths: pixels of 128, 256 and 512 bytes
    ((True, 32, 20, 20, 128, 1), (0, None)), ((True, 64, 20, 20, 128, 1), (2, None)),
    ((True, 96, 20, 20, 128, 1), (0, None)), ((True, 128, 20, 20, 128, 1), (4, None)),
    ((True, 256, 20, 20, 128, 1), (4, 26)), ((True, 512, 20, 20, 128, 1), (0, None)),
    ((False, 32, 20, 20, 128, 1), (2, None)), ((False, 64, 20, 20, 128, 1), (4, None)),
    ((False, 128, 20, 20, 128, 1), (4, 26)),
    # 128 k output channels: up to half the CUs in 4 x 16 x 128 tiles
    ((True, 128, 508, 16, 128, 1), (4, None)), ((True, 128, 509, 16, 128, 1), (0, None)),
    ((True, 128, 252, 16, 256, 2), (4, 2)), ((True, 128, 253, 16, 256, 2), (0, None)),
    ((True, 128, 252, 16, 256, 2, 128), (0, None)),
    # ... and the 64-channel entries up to the 256-pixel implicit GEMM's line
    ((True, 64, 255, 256, 128, 2), (2, None)), ((True, 64, 256, 256, 128, 2), (0, None)),
    ((True, 64, 256, 256, 128, 1), (0, None)),
    # other output channels: always with stride 1 or 64 input channels
    ((True, 256, 2000, 2000, 96, 1), (4, None)), ((True, 64, 2000, 2000, 192, 2), (2, None)),
    # stride 2 from 128 channels: where the GEMM's last 64 channels are not all used, or below two tiles per CU
    ((True, 128, 2000, 2000, 96, 2), (4, None)), ((True, 128, 170, 128, 192, 2), (4, None)),
    ((True, 128, 171, 128, 192, 2), (0, None)), ((False, 64, 171, 128, 192, 2), (0, None)),
    # from 256: up to 32 channels, or below 5 tiles per 8 CUs
    ((True, 256, 2000, 2000, 32, 2), (4, None)), ((True, 256, 79, 128, 96, 2), (4, None)),
    ((True, 256, 80, 128, 96, 2), (0, None)), ((True, 256, 80, 128, 64, 2), (4, None)),
    # the maps from which the halo tilings run: more than 256 tiles, 128, 224
    ((True, 256, 64, 64, 128, 1), (4, 5)), ((True, 256, 64, 68, 128, 1), (4, 4)),
    ((True, 256, 64, 64, 128, 2), (4, 3)), ((True, 256, 64, 68, 128, 2), (4, 2)),
    ((True, 128, 56, 64, 128, 2), (4, 5)), ((True, 128, 60, 64, 128, 2), (4, 4)), ((True, 128, 64, 64, 128, 1), (4, None)),
])
def test_where_slices_are_summed_side_by_side(planner, shape, want):
    assert planner(*shape) == want


def test_arguments_are_checked():
    lib = _lib()
    for bad in [dict(maps=0), dict(maps=17), dict(stride=3), dict(n_cu=0), dict(Ci=0)]:
        kw = dict(Hi=64, Wi=64, Ci=64, Ho=64, Wo=64, Co=128, stride=1, n_cu=256, maps=1)
        kw.update(bad)
        with pytest.raises(R.RtccError) as e:
            R.rtcc_conv_tiling(kw["Hi"], kw["Wi"], kw["Ci"], kw["Ho"], kw["Wo"], kw["Co"], kw["stride"],
                               kw["n_cu"], kw["maps"], lib=lib)
        assert e.value.status == R.RTCC_E_ARG
