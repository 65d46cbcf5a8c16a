"""Max-pooling on the blocked layout, 3 x 3 windows (a kernel of their own) and the general one, where they can go wrong: images smaller
than a window, windows that hang over both edges, rows and columns that no window reaches, more than one workgroup with a remainder, and
equal maxima that differ in the neighbouring channel (bytes are compared in pairs)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def psb():
    import torch
    assert torch.cuda.is_available()
    from paper_1904_02205_amd import psb as m
    m.lib()
    return m


@pytest.mark.parametrize("values", ["any", "lowest", "two"])
@pytest.mark.parametrize("kernel", [(3, 3), (5, 5)])
@pytest.mark.parametrize("stride,pad,n,c,h,w", [((2, 2), (1, 1), 2, 64, 5, 6), ((1, 1), (1, 1), 3, 33, 3, 4), ((3, 1), (1, 0), 1, 32, 7, 5),
                                                ((4, 5), (0, 1), 2, 70, 23, 18), ((2, 2), (1, 1), 2, 40, 31, 33), ((1, 2), (1, 1), 1, 5, 3, 3)])
def test_pooling_on_the_blocked_layout(psb, orc, kernel, stride, pad, n, c, h, w, values):
    import torch
    from test_gpu_blocked import to_blocked, from_blocked
    h, w = max(h, kernel[0] - 2 * pad[0]), max(w, kernel[1] - 2 * pad[1])
    rng = np.random.default_rng(h * w + c)
    x = {"any": lambda: rng.integers(-128, 128, size=(n, c, h, w)), "lowest": lambda: np.full((n, c, h, w), -128),
         "two": lambda: rng.integers(-1, 1, size=(n, c, h, w))}[values]().astype(np.int8)
    got = psb.maxpool2d_i8_blocked(torch.from_numpy(to_blocked(x, 127)).cuda(), x.shape, kernel, stride, pad).cpu().numpy()
    assert np.array_equal(from_blocked(got, c), orc.maxpool_i8(x, kernel, stride, pad))


@pytest.mark.parametrize("pad", [0, 1])
def test_smallest_images(psb, orc, pad):
    import torch
    from test_gpu_blocked import to_blocked, from_blocked
    h, w = 3 - 2 * pad, 4 - 2 * pad
    x = np.random.default_rng(pad).integers(-128, 128, size=(2, 32, h, w)).astype(np.int8)
    got = psb.maxpool2d_i8_blocked(torch.from_numpy(to_blocked(x, 0)).cuda(), x.shape, (3, 3), (2, 2), (pad, pad)).cpu().numpy()
    assert np.array_equal(from_blocked(got, 32), orc.maxpool_i8(x, (3, 3), (2, 2), (pad, pad)))
