"""The rule that chooses between the per-product kernels (csrc/psb_choice.h) against times measured on an MI355X."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1904_02205_amd", "csrc")

PROGRAM = """
#include "psb_choice.h"
extern "C" int prefer_lanes(int K, int OC, long long live, double pixels, int blocks, int map, int chunks, int taps, int channels, int n_cus)
{
    psb::LayerWork w{K, OC, live, pixels, blocks, map != 0, chunks, taps, channels, 256, 10};
    return psb::prefer_channel_lanes(w, n_cus);
}
"""

# taps, channels, live weights, output pixels, generator blocks, budget map, chunks of the channel-lane kernel and taps of one;
# us of (lanes, list) with a quarter of the activations not zero, and with all of them
MEASURED = [
    (576, 8, 4608, 4704, 1, False, 9, 64, 59, 131, 188, 229),
    (576, 8, 4608, 4704, 2, False, 9, 64, 96, 140, 331, 255),
    (576, 8, 4608, 4704, 8, False, 9, 64, 351, 251, 1317, 605),
    (576, 8, 4608, 784, 8, False, 18, 32, 72, 251, 229, 601),
    (576, 17, 9792, 4704, 4, False, 9, 64, 179, 217, 648, 504),
    (576, 32, 18432, 25088, 2, False, 9, 64, 458, 580, 1698, 1372),
    (576, 40, 23040, 25088, 4, False, 9, 64, 892, 1012, 3372, 2825),
    (576, 64, 36864, 4704, 4, False, 9, 64, 180, 371, 647, 999),
    (576, 70, 40320, 4704, 2, False, 9, 64, 177, 292, 644, 691),
    (128, 27, 3456, 25088, 1, False, 2, 64, 71, 83, 232, 168),
    (128, 32, 4096, 25088, 2, False, 2, 64, 114, 122, 400, 295),
    (24, 27, 648, 25088, 2, False, 1, 24, 27, 25, 78, 53),
    (24, 12, 288, 4704, 8, False, 2, 12, 28, 26, 67, 55),
    (675, 70, 47250, 4704, 2, False, 11, 62, 202, 338, 721, 785),
    (675, 4, 2700, 4704, 1, False, 11, 62, 67, 153, 214, 267),
    (53, 64, 1357, 14157, 4, True, 2, 27, 49, 71, 143, 212),
    (175, 100, 8750, 2352, 6, False, 3, 59, 96, 66, 325, 177),
    (1818, 7, 5091, 12544, 2, False, 29, 63, 756, 220, 2751, 456),
    (2142, 42, 89626, 45, 6, False, 134, 16, 20, 476, 41, 647),
    (45, 51, 2294, 9408, 6, False, 1, 45, 56, 62, 182, 164),
    (234, 312, 72978, 2000, 8, False, 4, 59, 325, 443, 1099, 1326),
    (335, 9, 3009, 3136, 2, False, 6, 56, 44, 77, 138, 143),
    (74, 85, 6287, 490, 8, True, 5, 15, 22, 52, 49, 131),
    (1050, 2, 2092, 588, 4, True, 33, 32, 36, 418, 105, 979),
    (375, 7, 1313, 16335, 2, False, 6, 63, 218, 60, 717, 113),
    (925, 3, 2759, 6534, 3, False, 15, 62, 364, 260, 1358, 526),
    (3725, 3, 5588, 6272, 8, False, 59, 64, 2745, 815, 10588, 1988),
]


@pytest.fixture(scope="module")
def prefer_lanes(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("choice")
    (d / "choice.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-fPIC", "-shared", "-I", CSRC, str(d / "choice.cpp"), "-o",
                    str(d / "choice.so")], check=True)
    fn = C.CDLL(str(d / "choice.so")).prefer_lanes
    fn.argtypes = [C.c_int, C.c_int, C.c_longlong, C.c_double] + [C.c_int] * 6
    return fn


@pytest.mark.parametrize("case", MEASURED)
def test_choice_against_measured_times(prefer_lanes, case):
    """A kernel that measures a quarter faster at both ends is chosen; and where the choice departs from the plain one (lanes for
    dense layers that fill half of the lanes of their last block) it loses at most 30 % at either: the rule's 15 % and the
    13 % (root mean square) that its estimates are off."""
    K, oc, live, pixels, blocks, budget_map, chunks, taps, *us = case
    lanes = bool(prefer_lanes(K, oc, live, pixels, blocks, budget_map, chunks, taps, min(8, max(1, 64 // K)), 256))
    plain = 2 * live >= oc * K and (oc % 64 == 0 or oc % 64 >= 32 or oc >= 256)
    gain = [us[1] / us[0], us[3] / us[2]] if lanes else [us[0] / us[1], us[2] / us[3]]      # over the kernel not chosen
    assert max(gain) > 1 / 1.25
    if lanes != plain:
        assert min(gain) > 1 / 1.3


def test_choice_at_given_layers(prefer_lanes):
    """3x3 on 64 channels: 8 channels on 4704 pixels change from lanes to the list between 4 and 8 samples (all activations live,
    S = 8: 331 us on lanes, 255 on the list), on 784 pixels lanes are faster at any S; 64 channels are lanes; and with more CUs the
    lanes, which have the more work, catch up."""
    conv = lambda oc, pixels, blocks, n_cus=256: prefer_lanes(576, oc, 576 * oc, pixels, blocks, 0, 9, 64, 1, n_cus)
    assert conv(8, 4704, 1) and not conv(8, 4704, 2) and not conv(8, 4704, 8) and conv(8, 784, 8) and conv(64, 4704, 4)
    assert conv(8, 4704, 2, 512) and not conv(8, 4704, 2, 64)
