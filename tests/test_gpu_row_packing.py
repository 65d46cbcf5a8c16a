"""First layers with packed rows, at the edges of the packing's tiles: several rows to a tile and a remainder, an image row of more than
256 packed pixels, a stride that leaves room for a few pixels only, all 32 slots and hardly any, one packed pixel to a row."""
import numpy as np
import pytest

import helpers
from paper_1904_02205_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def psb():
    from paper_1904_02205_amd import psb as mod
    mod.lib()
    return mod


@pytest.mark.parametrize("nhw,cin,kw,stride,pad", [
    ((3, 5, 9), 3, 7, 2, 3),             # 51 rows of 5 pixels to a tile, 15 there are
    ((2, 70, 13), 4, 8, 1, 4),           # 18 of them, and a remainder; all 32 slots
    ((1, 3, 255), 1, 2, 1, 1),           # 256 pixels: a whole tile, and one
    ((1, 3, 256), 1, 2, 1, 1),           # ... one more: cut into two
    ((2, 2, 1021), 10, 3, 1, 1),         # cut by their number
    ((1, 2, 4000), 16, 2, 31, 0),        # cut by the LDS
    ((2, 4, 7), 5, 6, 3, 0),             # one pixel to a row
])
def test_row_packing(psb, orc, nhw, cin, kw, stride, pad):
    n, h, w = nhw
    rng = np.random.default_rng(w * 31 + kw)
    L = synth.Layer("packed_rows", synth.he_normal((5, cin, 2, kw), rng), synth.gaussian_int8((n, cin, h, w), rng), pad=(0, pad),
                    stride=(1, stride), S=4, seed=9, layer_id=2)
    ref, over, _ = helpers.oracle_layer(orc, L, shared=True)
    acc, _ = helpers.gpu_layer(psb, L, shared=True)
    assert over == 0 and np.array_equal(acc, ref)
