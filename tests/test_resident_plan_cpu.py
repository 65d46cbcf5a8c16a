"""How 3x3 layers are cut for the kernel that keeps the whole input window in LDS (csrc/psb_resident_plan.h)."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1904_02205_amd", "csrc")

# argv: seed, layers.  Every cut of so many random layers: nothing is read or written beyond what the plan reserves.
BOUNDS = r"""
#include "psb_resident_plan.h"
#include <cstdio>
#include <cstdlib>
#include <random>
using namespace psb;
#define CHECK(x) do { if (!(x)) { std::printf("%s: N %d C %d %dx%d OC %d planes %d segments %d residual %d\n", #x, N, C, H, W, OC, l.planes, l.n_seg, (int)l.residual); return 1; } } while (0)
int main(int argc, char** argv)
{
    std::mt19937 rng(std::atoi(argv[1]));
    auto upto = [&](int n) { return (int)(1 + rng() % n); };
    int taken = 0, groups[14] = {}, reductions[4] = {}, by_channels = 0, residuals = 0;
    for (int it = 0; it < std::atoi(argv[2]) && argc == 3; ++it) {
        const int N = upto(40), C = upto(600), H = upto(60), W = rng() % 3 ? upto(60) : H, OC = upto(600);
        ResidentLayer l{};
        l.npix = (int64_t)N * H * W; l.H = H; l.W = W; l.OC = OC; l.blocks = (C + 31) / 32;
        l.planes = 2 + rng() % 2; l.n_seg = rng() % 3 ? 0 : 2; l.residual = rng() % 2;
        l.half_tiles = (l.npix + 63) / 64 * ((OC + 31) / 32) <= 1024 ? 1 : 2;
        if (l.npix > 300000) continue;
        ResidentPlan r{};
        if (!resident_plan(l, 256, r)) continue;
        ++taken; ++groups[r.ng]; ++reductions[r.log_wk]; by_channels += r.by_channels; residuals += r.lds_res > 0;
        const int64_t tile = (int64_t)r.part << r.log_wp, chunks = (l.blocks + 1) / 2, oc16 = 2 * ((OC + 31) / 32);
        CHECK(r.log_wo + r.log_wp + r.log_wk == 3 && (r.ng == 4 || r.ng == 7 || r.ng == 13));
        CHECK(r.ng < 13 || (r.log_wk == 0 && l.n_seg == 0));              // no such instances
        CHECK(r.part > 0 && r.part % 4 == 0 && r.part <= 16 * r.ng);
        CHECK(r.px_tiles * tile >= l.npix && (r.px_tiles - 1) * tile < l.npix);
        CHECK(((int64_t)r.oc_tiles << r.log_wo) >= oc16 && ((int64_t)(r.oc_tiles - 1) << r.log_wo) < oc16);
        CHECK(!r.by_channels || r.oc_tiles % 8 == 0);
        CHECK(9 * chunks >= 2 << r.log_wk);                               // every part of the reduction has steps
        // LDS: table of the tile's pixels, window, 16 zero bytes; behind the table the sums meet; the residual behind all
        CHECK(r.lds_window >= tile * kResidentEntry && r.lds_window % 16 == 0 && r.slots_pad % 16 == 0);
        CHECK(r.lds_zero >= r.lds_window + r.slots_pad * 64 * chunks && r.lds_zero % 16 == 0 && r.lds_zero + 16 <= r.lds_bytes);
        CHECK((kResidentWaves >> r.log_wk) * r.ng * ((1 << r.log_wk) - 1) * 1024 <= r.lds_bytes - r.lds_window);
        CHECK(r.lds_bytes <= kResidentLds);
        if (r.lds_res) CHECK(l.residual && r.lds_res >= r.lds_zero + 16 && r.lds_res % 16 == 0 && r.lds_res + (tile << r.log_wo) * 16 <= r.lds_bytes);
        auto position = [&](int64_t pix) { const int64_t row = pix / W; return (row + row / H) * (W + 1) + pix % W; };
        for (int64_t t = 0; t < r.px_tiles; ++t) {
            const int64_t first = t * tile, last = std::min(first + tile, l.npix) - 1;
            CHECK(position(last) - position(first) + 2 * (W + 1) + 3 <= r.slots_pad);
        }
    }
    std::printf("%d taken, groups of pixels 4: %d 7: %d 13: %d, reduction parts 1: %d 2: %d 4: %d 8: %d, by channels %d, residual staged %d\n", taken, groups[4],
                groups[7], groups[13], reductions[0], reductions[1], reductions[2], reductions[3], by_channels, residuals);
    return !(taken > 1000 && groups[4] && groups[7] && groups[13] && reductions[1] && reductions[2] && reductions[3] && by_channels && residuals);
}
"""


def build(tmp_path, program):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(program)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return str(exe)


def test_every_cut_stays_inside_what_it_reserves(tmp_path):
    exe = build(tmp_path, BOUNDS)
    for seed in (1, 2):
        r = subprocess.run([exe, str(seed), "20000"], capture_output=True, text=True)
        assert r.returncode == 0, r.stdout


# stdin: layers, one a line; prints whether the kernel takes them on a device with 256 CUs, and its cut
CHOICE = r"""
#include "psb_resident_plan.h"
#include <cstdio>
int main()
{
    int n, c, h, w, oc, planes, n_seg, residual;
    while (std::scanf("%d %d %d %d %d %d %d %d", &n, &c, &h, &w, &oc, &planes, &n_seg, &residual) == 8) {
        const int64_t npix = (int64_t)n * h * w;
        const int half_tiles = (npix + 63) / 64 * ((oc + 31) / 32) <= 1024 ? 1 : 2;
        psb::ResidentLayer l{npix, h, w, oc, (c + 31) / 32, planes, n_seg, half_tiles, residual != 0};
        psb::ResidentPlan r{};
        const bool taken = psb::resident_plan(l, 256, r);
        std::printf("%d %d %d %d\n", taken, r.ng, 1 << r.log_wk, (int)((r.px_tiles * r.oc_tiles + 255) / 256));
    }
}
"""

# images, input channels, height, width, output channels, digit planes, levels, int8 residual: us in this kernel and in the others
# (of a call with its sampling, or as noted), and the form of the cut (pixel groups, reduction parts, rounds)
MEASURED = [
    ((64, 256, 10, 93, 128, 3, 0, 1), 76.95, 62.14, (13, 1, 2)),       # parts of 120 pixels in groups of 208
    ((16, 512, 112, 22, 96, 2, 0, 0), 67.96, 55.01, (7, 1, 2)),
    ((32, 160, 56, 56, 96, 3, 0, 0), 63.98, 52.57, (13, 1, 2)),
    ((1, 768, 56, 56, 128, 2, 0, 0), 35.60, 29.74, (4, 1, 1)),         # parts of 16 pixels, the window of more does not fit
    ((16, 64, 56, 65, 64, 3, 0, 0), 24.91, 22.46, (13, 1, 1)),
    ((4, 768, 28, 45, 512, 2, 0, 1), 78.24, 67.46, (4, 1, 2)),         # four groups of two planes, two rounds
    ((2, 640, 56, 56, 512, 2, 2, 0), 121.90, 108.15, (4, 1, 2)),
    ((64, 256, 14, 106, 16, 2, 0, 1), 29.32, 26.04, (7, 2, 2)),        # the reduction in parts, two rounds
    ((8, 384, 80, 80, 48, 2, 0, 1), 38.31, 36.13, (7, 2, 2)),
    ((32, 64, 56, 56, 64, 3, 0, 1), 15.0, 20.5, (13, 1, 1)),              # a launch, from the time of a network pass; this line and the next
    ((32, 128, 28, 28, 128, 3, 0, 0), 13.8, 17.0, (7, 1, 1)),
    ((8, 64, 56, 88, 128, 3, 0, 1), 19.27, 28.70, (13, 1, 1)),
    ((64, 128, 28, 28, 200, 3, 0, 0), 47.89, 51.18, (13, 1, 2)),
    ((2, 256, 56, 72, 512, 3, 0, 0), 35.14, 39.14, (4, 1, 2)),         # four groups of three planes
]


def test_layers_go_to_the_faster_kernels(tmp_path):
    out = subprocess.run([build(tmp_path, CHOICE)], input="\n".join(" ".join(map(str, m[0])) for m in MEASURED), capture_output=True, text=True,
                         check=True).stdout.split("\n")
    for (layer, here, there, form), line in zip(MEASURED, out):
        taken, *cut = map(int, line.split())
        assert tuple(cut) == form, (layer, line)
        assert taken == (here < there), (layer, line)
