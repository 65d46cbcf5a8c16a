"""Shared-filter mode (Eq. numbersystem:simulation) on the GPU vs the CPU oracle: the sampled integer filter
and the layers built on it (int8 matrix cores for groups = 1, direct kernel otherwise).  Bit-exact."""
import numpy as np
import pytest

import helpers
from paper_1904_02205_amd import synth
from test_gpu_parity import _layer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def psb():
    import torch
    assert torch.cuda.is_available()
    from paper_1904_02205_amd import psb as m
    m.lib()
    yield m
    m.set_mapping(m.MAPPING_AUTO)


@pytest.mark.parametrize("prob_bits", [23, 4, 7])
def test_sampled_filter_matches_oracle(psb, orc, prob_bits):
    rng = np.random.default_rng(800 + prob_bits)
    L = _layer(rng, 1, 20, 70, 5, 3, pad=1, S=32, s_max=48, prune=0.3)
    qo = helpers.oracle_quantize(orc, L, prob_bits=prob_bits)
    qg = helpers.gpu_quantize(psb, L, prob_bits=prob_bits)
    for a, b in ((0, 16), (0, 1), (0, 48), (3, 4), (5, 37), (16, 32)):
        ref = orc.sample_filter(qo, seed=L.seed, layer_id=L.layer_id, sample_from=a, sample_to=b)
        got = psb.sample_filter(qg, b, a, seed=L.seed, layer_id=L.layer_id).cpu().numpy()
        assert np.array_equal(got.astype(np.int64), ref), (a, b)
    for a, b in ((-1, 4), (4, 4), (5, 3), (0, 49)):
        with pytest.raises(psb.PsbError) as ei:
            psb.sample_filter(qg, b, a)
        assert ei.value.code == psb.ERR_VALUE


@pytest.mark.parametrize("cin,oc,k,prob_bits", [
    (1, 1, 1, 23), (33, 31, 1, 4), (32, 33, 3, 23), (40, 64, 3, 7), (70, 65, 3, 23), (3, 97, 5, 23), (4, 40, 7, 4),   # a few slots a wave
    (32 * 287 + 1, 66, 1, 23), (32 * 288, 66, 1, 4), (32 * 287, 128, 1, 23), (64 * 32, 65, 3, 23)])                     # launches around the line to more
def test_digit_planes_hold_the_sampled_filter(psb, cin, oc, k, prob_bits):
    """The filter the matrix cores contract against the int32 filter of psb_sample_filter, over ranges that begin and end inside a
    generator block (one output pixel per image, no activation zero; integers, so exact in 64 bits)."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(cin * 1000 + oc)
    w = torch.randn((oc, cin, k, k), generator=gen, device="cuda") * 0.05
    w[torch.rand(w.shape, generator=gen, device="cuda") < 0.2] = 0.0
    q = psb.Weights(w, s_max=40, prob_bits=prob_bits)
    x = torch.randint(1, 128, (5, cin, k, k), generator=gen, device="cuda", dtype=torch.int8)
    x = torch.where(torch.rand(x.shape, generator=gen, device="cuda") < 0.5, x, -x)
    for a, b in ((0, 8), (0, 40), (0, 3), (4, 8), (5, 6), (3, 37), (16, 32), (31, 34)):
        full = lambda v: torch.full((5, 1, 1), v, dtype=torch.uint8, device="cuda")
        acc = torch.zeros((5, oc, 1, 1), dtype=torch.int32, device="cuda")
        if a == 0:
            psb.conv2d(q, x, b, seed=7, layer_id=2, acc=acc, shared=True)
        else:
            psb.conv2d_progressive(q, x, full(b), full(a), seed=7, layer_id=2, acc=acc, shared=True)
        f = psb.sample_filter(q, b, a, seed=7, layer_id=2)
        ref = x.view(5, -1).double().cpu() @ f.view(oc, -1).double().cpu().t()
        assert torch.equal(acc.view(5, oc).cpu().double(), ref), (a, b)


def _cases():
    rng = np.random.default_rng(900)
    c = []
    both = (0, 1)             # 0: matrix cores for groups = 1; 1: direct kernel
    c.append(("linear_small", _layer(rng, 5, 37, 9, 1, 1, S=8, xkind="u4", std=0.05), both))
    c.append(("linear_ragged", _layer(rng, 67, 130, 100, 1, 1, S=5, xkind="signed", std=0.05), both))
    c.append(("conv3x3_c20_oc70", _layer(rng, 2, 20, 70, (9, 11), 3, pad=1, S=8), both))
    c.append(("conv3x3_c64", _layer(rng, 1, 64, 64, 14, 3, pad=1, S=16), both))
    c.append(("conv3x3_c96_signed", _layer(rng, 1, 96, 33, 6, 3, pad=1, S=32, xkind="signed"), both))
    c.append(("conv7x7_s2_p3_c3", _layer(rng, 2, 3, 16, (23, 19), 7, stride=2, pad=3, S=8, xkind="signed"), both))
    c.append(("conv1x1_s2", _layer(rng, 2, 24, 40, 9, 1, stride=2, S=4), both))
    c.append(("conv_rect_kernel", _layer(rng, 1, 6, 12, (6, 8), (2, 3), stride=(1, 2), pad=(0, 2), S=3), both))
    c.append(("conv_s1", _layer(rng, 1, 5, 7, 5, 3, pad=1, S=1), both))
    c.append(("conv_pad3_tiny_image", _layer(rng, 1, 4, 8, 2, 3, pad=3, S=4), both))
    c.append(("conv_wide_row", _layer(rng, 1, 8, 32, (3, 150), 3, pad=1, S=8), both))
    c.append(("pruned_pointwise", _layer(rng, 2, 96, 40, 5, 1, S=16, prune=0.9), both))
    c.append(("s255", _layer(rng, 1, 3, 8, 4, 3, pad=1, S=255, std=0.01), both))
    c.append(("s12_three_generator_blocks", _layer(rng, 2, 40, 48, 10, 3, pad=1, S=12), both))
    c.append(("deep_reduction_few_pixels", _layer(rng, 1, 256, 64, 6, 3, pad=1, S=8), both))      # reduction split 4 ways
    c.append(("deep_linear", _layer(rng, 3, 2048, 40, 1, 1, S=4, xkind="u4", std=0.02), both))     # split 4 ways
    c.append(("row_packed_5x5_c6", _layer(rng, 2, 6, 20, (13, 17), 5, stride=2, pad=2, S=8, xkind="signed"), both))
    c.append(("row_packed_1x3_c10", _layer(rng, 1, 10, 8, (4, 9), (1, 3), pad=(0, 1), S=4), both))
    # more pixel tiles than workgroups fit the chip, short reduction: the persistent variant of the matrix-core kernel
    c.append(("many_tiles_short_reduction", _layer(rng, 1, 16, 40, (370, 372), 3, pad=1, S=4), (0,)))
    c.append(("many_tiles_row_packed", _layer(rng, 1, 3, 33, (530, 540), 5, stride=2, pad=2, S=4, xkind="signed"), (0,)))
    # two half tiles per wave without the persistent variant: many channel blocks, few pixel tiles per block
    c.append(("two_half_tiles_many_blocks", _layer(rng, 1, 32, 250, (100, 120), 3, pad=1, S=4), (0,)))
    # 3 x 3, stride 1, padding 1 with the input window in LDS, 32 channels at a time (one block of channels) or all of them: ragged sizes,
    # channel padding, a wide image, two half tiles per wave with a tile that crosses an image boundary, tiles that span many tiny images
    # (test_window_of_all_channels and test_window_of_32_channels check which kernel and shape runs)
    c.append(("window_two_teams", _layer(rng, 2, 128, 64, 14, 3, pad=1, S=8), (0,)))
    c.append(("window_two_teams_wide", _layer(rng, 1, 128, 32, 40, 3, pad=1, S=4), (0,)))
    c.append(("window_ragged", _layer(rng, 3, 64, 40, (13, 11), 3, pad=1, S=8), (0,)))
    c.append(("window_one_block_wide", _layer(rng, 1, 20, 33, (37, 45), 3, pad=1, S=4), (0,)))
    c.append(("window_two_half_tiles", _layer(rng, 2, 32, 480, 50, 3, pad=1, S=4), (0,)))
    c.append(("window_many_small_images", _layer(rng, 40, 128, 32, 4, 3, pad=1, S=8, xkind="signed"), (0,)))
    # ... and layers with many weights for their pixels
    c.append(("window_many_channel_blocks", _layer(rng, 3, 128, 250, 6, 3, pad=1, S=8, xkind="signed"), (0,)))
    c.append(("window_sixteen_channel_blocks", _layer(rng, 2, 64, 512, 9, 3, pad=1, S=4), (0,)))
    c.append(("window_one_pixel_images", _layer(rng, 70, 64, 32, 1, 3, pad=1, S=8, xkind="signed"), (0,)))
    c.append(("window_one_column_images", _layer(rng, 9, 64, 32, (17, 1), 3, pad=1, S=8, xkind="signed"), (0,)))
    c.append(("grouped", _layer(rng, 2, 8, 12, 7, 3, pad=1, groups=4, S=8), (0,)))
    c.append(("depthwise", _layer(rng, 2, 70, 70, 9, 3, pad=1, groups=70, S=16), (0,)))
    # 3 x 3 depthwise layers have a kernel of their own: odd channel count, stride 2, two outputs per input channel
    c.append(("depthwise_s2_odd_channels", _layer(rng, 3, 13, 13, (11, 9), 3, stride=2, pad=1, groups=13, S=8), (0,)))
    c.append(("depthwise_multiplier_2_unpadded", _layer(rng, 1, 10, 20, 8, 3, groups=10, S=4, xkind="signed"), (0,)))
    c.append(("depthwise_many_pixels", _layer(rng, 2, 5, 5, (40, 70), 3, pad=1, groups=5, S=8), (0,)))
    c.append(("depthwise_5x5", _layer(rng, 1, 6, 6, 9, 5, pad=2, groups=6, S=8), (0,)))
    return c


@pytest.mark.parametrize("case", _cases(), ids=lambda c: c[0])
def test_layer_bit_exact(psb, orc, case):
    _, L, mappings = case
    ref, over, _ = helpers.oracle_layer(orc, L, shared=True)
    assert over == 0
    qg = helpers.gpu_quantize(psb, L)
    for m in mappings:
        psb.set_mapping(m)
        acc, _ = helpers.gpu_layer(psb, L, qg, shared=True)
        assert np.array_equal(acc, ref), f"mapping {m}"
        acc, _ = helpers.gpu_layer(psb, L, qg, shared=True)      # workspace reuse: same bits
        assert np.array_equal(acc, ref), f"mapping {m}, second call"
    psb.set_mapping(psb.MAPPING_AUTO)


@pytest.mark.parametrize("planes_case", [
    # few taps and a tiny activation range let the window reach deep: filter values up to 2^30
    ("deep_window", dict(exp_bits=5, x_absmax=1, s_max=2), 2),
    ("one_exponent", dict(exp_bits=1, x_absmax=127, s_max=1), 1),
    ("default", dict(exp_bits=0, x_absmax=127, s_max=16), 16),
], ids=lambda c: c[0])
def test_every_digit_plane_count(psb, orc, planes_case):
    """Filters that need 1, 3 and 4 base-256 digit planes."""
    import torch
    _, kw, S = planes_case
    rng = np.random.default_rng(950)
    w = (rng.standard_normal((40, 4, 1, 1)) * 10.0 ** rng.uniform(-6, 0, size=(40, 4, 1, 1))).astype(np.float32)
    x = rng.integers(-kw["x_absmax"], kw["x_absmax"] + 1, size=(3, 4, 9, 9)).astype(np.int8)
    qo = orc.QWeights(w.reshape(40, -1), **kw)
    qg = psb.Weights(torch.from_numpy(w).cuda(), **kw)
    ref, over = orc.conv2d_shared(qo, (40, 4, 1, 1, 1), x, S=S, seed=8, layer_id=2)
    assert over == 0
    acc = psb.conv2d(qg, torch.from_numpy(x).cuda(), S, seed=8, layer_id=2, shared=True).cpu().numpy()
    assert np.array_equal(acc, ref)
    if planes_case[0] == "deep_window":
        assert np.abs(orc.sample_filter(qo, S, seed=8, layer_id=2)).max() >= 2 ** 24      # really four planes


def test_four_digit_planes_on_a_3x3_layer(psb, orc):
    """The both-operands-in-LDS kernel with four planes, with one team and with two."""
    import torch
    rng = np.random.default_rng(951)
    kw = dict(exp_bits=5, x_absmax=1, s_max=2)
    for c, hw in ((64, 9), (128, 12)):
        w = (rng.standard_normal((40, c, 3, 3)) * 10.0 ** rng.uniform(-6, 0, size=(40, c, 3, 3))).astype(np.float32)
        x = rng.integers(-1, 2, size=(3, c, hw, hw)).astype(np.int8)
        qo = orc.QWeights(w.reshape(40, -1), **kw)
        qg = psb.Weights(torch.from_numpy(w).cuda(), **kw)
        ref, over = orc.conv2d_shared(qo, (40, c, 3, 3, 1), x, (1, 1), (1, 1), S=2, seed=8, layer_id=2)
        assert over == 0
        assert np.abs(orc.sample_filter(qo, 2, seed=8, layer_id=2)).max() >= 2 ** 24      # really four planes
        acc = psb.conv2d(qg, torch.from_numpy(x).cuda(), 2, pad=(1, 1), seed=8, layer_id=2, shared=True).cpu().numpy()
        assert np.array_equal(acc, ref), c


def test_filter_value_between_the_ranges_of_two_and_three_digits(psb, orc):
    """W = 64 * (255 + 255) = 32640 has 15 bits but lies above 127 * 257, the largest two-digit balanced number."""
    import torch
    w = np.full((3, 500), np.nextafter(np.float32(2.0), np.float32(0)), np.float32)
    x = np.random.default_rng(955).integers(-128, 128, size=(4, 500)).astype(np.int8)
    qo = orc.QWeights(w, x_absmax=128, s_max=255)
    assert qo.e_top - qo.e_min == 6
    W = orc.sample_filter(qo, 255, seed=1)
    assert W.max() == 32640
    ref, over = orc.conv2d_shared(qo, (3, 500, 1, 1, 1), x.reshape(4, 500, 1, 1), S=255, seed=1)
    qg = psb.Weights(torch.from_numpy(w).cuda(), x_absmax=128, s_max=255)
    acc = psb.linear(qg, torch.from_numpy(x).cuda(), 255, seed=1, shared=True).cpu().numpy()
    assert over == 0 and np.array_equal(acc, ref.reshape(4, 3))


def test_prob_bits_and_seed(psb, orc):
    rng = np.random.default_rng(960)
    L = _layer(rng, 2, 32, 64, 8, 3, pad=1, S=16)
    qo = helpers.oracle_quantize(orc, L, prob_bits=4)
    qg = helpers.gpu_quantize(psb, L, prob_bits=4)
    ref, _, _ = helpers.oracle_layer(orc, L, qo, shared=True)
    acc, _ = helpers.gpu_layer(psb, L, qg, shared=True)
    assert np.array_equal(acc, ref)
    L2 = synth.Layer("t", L.w, L.x, pad=L.pad, S=16, s_max=16, seed=L.seed + 1, layer_id=L.layer_id)
    ref2, _, _ = helpers.oracle_layer(orc, L2, qo, shared=True)
    acc2, _ = helpers.gpu_layer(psb, L2, qg, shared=True)
    assert np.array_equal(acc2, ref2) and not np.array_equal(acc2, acc)
    per_product, _ = helpers.gpu_layer(psb, L, qg)
    assert not np.array_equal(per_product, acc)                   # a different estimator


@pytest.mark.parametrize("mapping", [0, 1])
def test_progressive_bit_exact_and_incremental(psb, orc, mapping):
    rng = np.random.default_rng(970)
    L = _layer(rng, 3, 12, 70, (9, 8), 3, pad=1, S=32, s_max=32)
    oh, ow = L.out_hw
    to = rng.choice([0, 1, 2, 3, 4, 7, 8, 16, 31, 32, 40], size=(3, oh, ow)).astype(np.uint8)   # 40 is clamped to 32
    qo = helpers.oracle_quantize(orc, L)
    ref, over, _ = helpers.oracle_layer(orc, L, qo, budget_to=to, shared=True)
    assert over == 0
    psb.set_mapping(mapping)
    qg = helpers.gpu_quantize(psb, L)
    acc, _ = helpers.gpu_layer(psb, L, qg, budget_to=to, shared=True)
    assert np.array_equal(acc, ref)
    for m in (8, 5):
        first = np.minimum(to, m).astype(np.uint8)
        a1, _ = helpers.gpu_layer(psb, L, qg, budget_to=first, shared=True)
        r1, _, _ = helpers.oracle_layer(orc, L, qo, budget_to=first, shared=True)
        assert np.array_equal(a1, r1)
        a2, _ = helpers.gpu_layer(psb, L, qg, budget_to=to, budget_from=first, acc_in=a1, shared=True)
        assert np.array_equal(a2, ref)
    a3, _ = helpers.gpu_layer(psb, L, qg, budget_to=first, budget_from=to, acc_in=a1, shared=True)   # empty ranges
    assert np.array_equal(a3, a1)
    const, _ = helpers.gpu_layer(psb, L, qg, budget_to=np.full((3, oh, ow), 8, np.uint8), shared=True)
    plain, _ = helpers.gpu_layer(psb, L, qg, S=8, shared=True)
    assert np.array_equal(const, plain)
    psb.set_mapping(psb.MAPPING_AUTO)


def test_progressive_with_many_channel_blocks(psb, orc):
    """Budget segments as masked, accumulating launches of the 3 x 3 kernel with two teams."""
    rng = np.random.default_rng(982)
    L = _layer(rng, 2, 128, 40, 12, 3, pad=1, S=8, s_max=8)
    oh, ow = L.out_hw
    to = rng.choice([0, 2, 4, 8], size=(2, oh, ow)).astype(np.uint8)
    qo, qg = helpers.oracle_quantize(orc, L), helpers.gpu_quantize(psb, L)
    ref, over, _ = helpers.oracle_layer(orc, L, qo, budget_to=to, shared=True)
    assert over == 0
    acc, _ = helpers.gpu_layer(psb, L, qg, budget_to=to, shared=True)
    assert np.array_equal(acc, ref)


def test_progressive_on_a_large_image(psb, orc):
    """Budget segments (masked, accumulating launches) with two half tiles per wave."""
    rng = np.random.default_rng(981)
    L = _layer(rng, 2, 16, 40, (200, 190), 3, pad=1, S=8, s_max=8)
    oh, ow = L.out_hw
    to = rng.choice([0, 2, 4, 8], size=(2, oh, ow)).astype(np.uint8)
    qo, qg = helpers.oracle_quantize(orc, L), helpers.gpu_quantize(psb, L)
    ref, over, _ = helpers.oracle_layer(orc, L, qo, budget_to=to, shared=True)
    assert over == 0
    acc, _ = helpers.gpu_layer(psb, L, qg, budget_to=to, shared=True)
    assert np.array_equal(acc, ref)


def test_activation_pointer_alignment(psb, orc):
    """The layout copy moves 32-bit words when the image plane and the pointer allow it: same integers at any
    byte offset of the input tensor, for planes that are and are not multiples of four bytes."""
    import torch
    rng = np.random.default_rng(983)
    for hw in ((20, 18), (9, 7)):
        L = _layer(rng, 2, 40, 48, hw, 3, pad=1, S=8)
        qo, qg = helpers.oracle_quantize(orc, L), helpers.gpu_quantize(psb, L)
        ref, over, _ = helpers.oracle_layer(orc, L, qo, shared=True)
        assert over == 0
        flat = torch.from_numpy(L.x).reshape(-1)
        for offset in (0, 1, 2, 4):
            buf = torch.zeros(flat.numel() + 8, dtype=torch.int8, device="cuda")
            buf[offset:offset + flat.numel()] = flat.cuda()
            x = buf[offset:offset + flat.numel()].view(L.x.shape)
            acc = psb.conv2d(qg, x, L.S, stride=L.stride, pad=L.pad, seed=L.seed, layer_id=L.layer_id, shared=True)
            assert np.array_equal(acc.cpu().numpy(), ref), (hw, offset)


def test_announced_budget_levels(psb, orc):
    """Budget values announced by the caller (for its next call) instead of read back from the map: same integers
    (exact set, a superset, values above s_max), for the matrix-core and the direct kernel, with and without a
    budget_from map; without the read-back the call can be captured into a HIP graph."""
    import torch
    rng = np.random.default_rng(984)
    for groups in (1, 4):
        L = _layer(rng, 2, 16, 40, (12, 9), 3, pad=1, groups=groups, S=16, s_max=16)
        oh, ow = L.out_hw
        to = rng.choice([4, 8, 16], size=(2, oh, ow)).astype(np.uint8)
        qo, qg = helpers.oracle_quantize(orc, L), helpers.gpu_quantize(psb, L)
        ref, over, _ = helpers.oracle_layer(orc, L, qo, budget_to=to, shared=True)
        assert over == 0
        try:
            for levels in ((4, 8, 16), (16, 4, 8, 2, 12), (4, 8, 200)):          # 200 clamps to s_max = 16
                psb.shared_budget_levels(levels)
                acc, _ = helpers.gpu_layer(psb, L, qg, budget_to=to, shared=True)
                assert np.array_equal(acc, ref), (groups, levels)
            first = np.minimum(to, 8).astype(np.uint8)
            psb.shared_budget_levels((4, 8))
            a1, _ = helpers.gpu_layer(psb, L, qg, budget_to=first, shared=True)
            psb.shared_budget_levels((4, 8, 16))
            a2, _ = helpers.gpu_layer(psb, L, qg, budget_to=to, budget_from=first, acc_in=a1, shared=True)
            assert np.array_equal(a2, ref)
            # captured: replays give the same integers
            x = torch.from_numpy(L.x).cuda()
            bt = torch.from_numpy(to).cuda()
            acc_t = torch.zeros((2, 40, oh, ow), dtype=torch.int32, device="cuda")
            psb.conv2d_progressive(qg, x, bt, stride=L.stride, pad=L.pad, seed=L.seed, layer_id=L.layer_id, acc=acc_t,
                                   shared=True)
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                psb.shared_budget_levels((4, 8, 16))          # an announcement is for the next call only
                psb.conv2d_progressive(qg, x, bt, stride=L.stride, pad=L.pad, seed=L.seed, layer_id=L.layer_id,
                                       acc=acc_t, shared=True)
            for _ in range(3):
                acc_t.fill_(-1)
                graph.replay()
                torch.cuda.synchronize()
                assert np.array_equal(acc_t.cpu().numpy(), ref)
        finally:
            psb.shared_budget_levels(None)
    acc, _ = helpers.gpu_layer(psb, L, qg, budget_to=to, shared=True)       # default path again
    assert np.array_equal(acc, ref)


def test_progressive_depthwise(psb, orc):
    """Budget segments through the 3 x 3 depthwise kernel: masked, accumulating launches; refinement in two calls."""
    rng = np.random.default_rng(982)
    L = _layer(rng, 2, 9, 9, (17, 12), 3, pad=1, groups=9, S=16, s_max=16)
    oh, ow = L.out_hw
    to = rng.choice([0, 2, 4, 8, 16], size=(2, oh, ow)).astype(np.uint8)
    qo, qg = helpers.oracle_quantize(orc, L), helpers.gpu_quantize(psb, L)
    ref, over, _ = helpers.oracle_layer(orc, L, qo, budget_to=to, shared=True)
    assert over == 0
    acc, _ = helpers.gpu_layer(psb, L, qg, budget_to=to, shared=True)
    assert np.array_equal(acc, ref)
    first = np.minimum(to, 4).astype(np.uint8)
    a1, _ = helpers.gpu_layer(psb, L, qg, budget_to=first, shared=True)
    a2, _ = helpers.gpu_layer(psb, L, qg, budget_to=to, budget_from=first, acc_in=a1, shared=True)
    assert np.array_equal(a2, ref)


def test_activation_tensor_beyond_the_offset_range_is_refused(psb):
    """The matrix-core kernel addresses the channels-last activations with 32-bit offsets: a tensor that
    reaches 2 GiB in that layout is an error, not a launch."""
    import torch
    w = torch.full((1, 1, 3, 3), 0.25, device="cuda")
    q = psb.Weights(w, x_absmax=127, s_max=8)
    x = torch.zeros((1, 1, 8192, 8192), dtype=torch.int8, device="cuda")    # 8192 * 8192 * 32 bytes once blocked
    acc = torch.empty((1, 1, 8192, 8192), dtype=torch.int32, device="cuda")
    with pytest.raises(psb.PsbError) as ei:
        psb.conv2d(q, x, 8, pad=(1, 1), acc=acc, shared=True)
    assert ei.value.code == psb.ERR_TOO_LARGE
    ok = psb.conv2d(q, x[:, :, :64, :64].contiguous(), 8, pad=(1, 1), shared=True)
    assert int(ok.abs().max()) == 0


@pytest.mark.parametrize("mapping", [0, 1])
def test_rescale_matches_oracle(psb, orc, mapping):
    rng = np.random.default_rng(980)
    L = _layer(rng, 2, 10, 40, 6, 3, pad=1, S=8, s_max=16)
    oc = 40
    mult = (rng.uniform(0.5, 2.0, size=oc) * 2.0 ** -9).astype(np.float32)
    bias = rng.standard_normal(oc).astype(np.float32)
    qo = helpers.oracle_quantize(orc, L)
    qg = helpers.gpu_quantize(psb, L)
    psb.set_mapping(mapping)
    ref, _, _ = helpers.oracle_layer(orc, L, qo, shared=True)
    acc, y = helpers.gpu_layer(psb, L, qg, want_y=True, mult=mult, bias=bias, shared=True)
    assert np.array_equal(acc, ref)
    assert np.array_equal(y, orc.rescale(ref, qo.e_min, S=8, s_max=16, mult=mult, bias=bias))
    oh, ow = L.out_hw
    to = rng.choice([0, 2, 8, 16], size=(2, oh, ow)).astype(np.uint8)
    refp, _, _ = helpers.oracle_layer(orc, L, qo, budget_to=to, shared=True)
    accp, yp = helpers.gpu_layer(psb, L, qg, budget_to=to, want_y=True, shared=True)
    assert np.array_equal(accp, refp)
    assert np.array_equal(yp, orc.rescale(refp, qo.e_min, s_max=16, budget_to=to))
    psb.set_mapping(psb.MAPPING_AUTO)


def _check_3x3(psb, n, cin, oc, hw, S, exp_bits, residual, ran, mult_to, x_absmax=128):
    """Accumulators against a 64-bit convolution with the sampled filter (exact), and every form of the fused outputs against the
    library's separate requantisation of the rescaled values (exact).  ran(launch, levels, residual): checks what the call ran in."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(n * 1000 + cin + oc)
    h, w = hw
    if x_absmax == 1:
        x = torch.randint(-1, 2, (n, cin, h, w), generator=gen, device="cuda", dtype=torch.int8)
    else:
        x = (torch.rand((n, cin, h, w), generator=gen, device="cuda") * 255 - 128).to(torch.int8)
    q = psb.Weights(torch.randn((oc, cin, 3, 3), generator=gen, device="cuda") * 0.05, exp_bits=exp_bits, s_max=2 * S,
                    x_absmax=min(x_absmax, 127))

    def ran_here(levels=False, blocked_residual=False):
        ran(psb.last_shared_launch(), levels, blocked_residual)
    mult = torch.rand(oc, generator=gen, device="cuda") * mult_to + mult_to / 20
    bias = torch.randn(oc, generator=gen, device="cuda") * 0.1
    geo = dict(stride=(1, 1), pad=(1, 1), seed=3, layer_id=4, mult=mult, bias=bias)
    acc = torch.empty((n, oc, h, w), dtype=torch.int32, device="cuda")
    y = torch.empty((n, oc, h, w), dtype=torch.float32, device="cuda")
    psb.conv2d(q, x, S, acc=acc, y=y, shared=True, **geo)
    ran_here()
    f = psb.sample_filter(q, S, seed=3, layer_id=4).view(oc, cin, 3, 3).double().cpu()
    for i in {0, n // 2, n - 1}:
        assert torch.equal(acc[i:i + 1].cpu().double(), torch.nn.functional.conv2d(x[i:i + 1].double().cpu(), f, padding=1)), i
    res = {}
    if residual == "f32":
        res = dict(res_f32=torch.randn((n, oc, h, w), generator=gen, device="cuda"))
        res["res_f32"].view(-1)[:6] = torch.tensor([float("nan"), float("inf"), -float("inf"), -0.0, 1e30, -1e30])
    elif residual == "i8":
        res = dict(res_i8=(torch.rand((n, oc, h, w), generator=gen, device="cuda") * 255 - 128).to(torch.int8), res_step=0.01)
    # (a gate with bounds below zero, where every result is the upper one, and scales that turn infinities or zeros into NaN among them)
    for relu, lo, hi, inv in ((True, 0, 127, 30.0), (False, -128, 127, 30.0), (True, -5, 127, 30.0), (True, -5, -3, 30.0), (True, -1, -1, 30.0),
                              (True, -100, -5, 30.0), (True, -128, -1, 0.0), (True, -9, -4, float("inf")), (False, -9, -4, 30.0)):
        want = psb.requantize(y, inv, relu=relu, lo=lo, hi=hi, **res)
        got = psb.conv2d_requant(q, x, inv, S=S, relu=relu, lo=lo, hi=hi, shared=True, want_acc=False, **geo, **res)
        assert torch.equal(got, want), (relu, lo, hi, inv)
        if inv == 30.0:
            ran_here()

    def blocked(t):
        cb = (t.shape[1] + 31) // 32
        p = torch.zeros((n, cb * 32, h, w), dtype=t.dtype, device="cuda")
        p[:, :t.shape[1]] = t
        return p.view(n, cb, 32, h, w).permute(0, 3, 1, 4, 2).contiguous()
    layout = psb.BLOCKED_IN | psb.BLOCKED_OUT
    if residual == "i8":
        res = dict(res_i8=blocked(res["res_i8"]), res_step=0.01)
        layout |= psb.BLOCKED_RES
    want = blocked(psb.requantize(y, 30.0, **({} if residual is None else dict(res_f32=res["res_f32"]) if residual == "f32" else
                                              dict(res_i8=res["res_i8"].permute(0, 2, 4, 1, 3).reshape(n, -1, h, w)[:, :oc].contiguous(), res_step=0.01))))
    got = psb.conv2d_shared_requant_blocked(q, blocked(x), (n, cin, h, w), 30.0, S, layout=layout, **geo, **res)
    assert torch.equal(got, want)
    ran_here(blocked_residual=residual == "i8")
    # two budget levels in one launch: a pixel's value is that of a call with its own sample count
    budget = torch.where(torch.rand((n, h, w), generator=gen, device="cuda") < 0.4, 2 * S, S).to(torch.uint8)
    budget[:, 0, 0] = S // 2                       # below every level
    both = [psb.conv2d_shared_requant_blocked(q, blocked(x), (n, cin, h, w), 30.0, s, layout=layout, **geo, **res) for s in (S, 2 * S)]
    got = psb.conv2d_shared_budget_requant_blocked(q, blocked(x), (n, cin, h, w), 30.0, budget, (S, 2 * S), layout=layout, **geo, **res)
    ran_here(levels=True, blocked_residual=residual == "i8")
    at = budget.view(n, h, 1, w, 1).expand_as(got)
    assert torch.equal(torch.where(at == S, both[0], torch.where(at == 2 * S, both[1], got)), got)


# planes: digit planes at S samples (four exponent bits, of which a long reduction leaves fewer, or two).  cut: pixel groups of a wave,
# waves of a workgroup (channel groups, pixel parts, reduction parts), whether an XCD takes an eighth of the channels; groups_seg: pixel
# groups with two budget levels, 0 for a layer that another kernel takes then.
@pytest.mark.parametrize("n,cin,oc,hw,S,exp_bits,planes,cut,groups_seg", [
    (1, 64, 16, (5, 6), 8, 4, 3, (4, (2, 1, 4), 0), 4),              # four pixels a wave
    (3, 40, 33, (9, 7), 4, 4, 3, (4, (2, 1, 4), 0), 4),              # channels that fill neither an instruction nor a block, tiles across images
    (2, 160, 70, (14, 13), 8, 4, 3, (4, (1, 1, 8), 0), 4),           # an odd number of channel blocks, planes no multiple of four bytes
    (1, 256, 64, (40, 36), 8, 4, 2, (4, (1, 1, 8), 0), 4),
    (8, 64, 64, (56, 56), 8, 4, 3, (4, (4, 2, 1), 0), 4),
    (40, 64, 200, (4, 4), 8, 4, 3, (4, (2, 1, 4), 0), 4),            # tiles of many small images, many channel groups
    (33, 512, 48, (7, 7), 2, 4, 2, (4, (1, 1, 8), 0), 4),            # two digit planes, long reduction
    (4, 512, 512, (7, 7), 2, 4, 2, (4, (1, 1, 8), 1), 4),            # more weights than activations: XCDs by channels
    (18, 256, 512, (7, 7), 8, 4, 3, (4, (2, 1, 4), 1), 4),
    (17, 64, 64, (56, 52), 8, 4, 3, (7, (4, 2, 1), 0), 7),
    (17, 64, 64, (56, 52), 8, 2, 2, (7, (4, 2, 1), 0), 7),
    (16, 128, 128, (28, 27), 8, 4, 3, (7, (4, 1, 2), 0), 7),         # seven groups, two of whose waves share a reduction
    (32, 512, 512, (7, 7), 2, 4, 2, (7, (2, 1, 4), 1), 7),
    (26, 64, 64, (55, 53), 8, 4, 3, (13, (4, 2, 1), 0), 0),          # thirteen groups, a last tile in part, planes no multiple of four bytes
    (40, 64, 70, (56, 56), 8, 2, 2, (13, (2, 4, 1), 0), 0),          # ... two rounds, padding channels
    (45, 128, 128, (28, 28), 8, 4, 3, (13, (8, 1, 1), 0), 0)])
@pytest.mark.parametrize("residual", [None, "f32", "i8"])
def test_window_of_all_channels(psb, n, cin, oc, hw, S, exp_bits, planes, cut, groups_seg, residual):
    """3 x 3 layers whose input window stays in LDS with all its channels."""
    def ran(at, levels, blocked_residual):
        if levels and not groups_seg:
            assert at.kernel == psb.SHARED_WINDOW
            return
        groups = groups_seg if levels else cut[0]
        assert (at.kernel, at.planes, at.pixel_groups) == (psb.SHARED_RESIDENT, planes, groups)
        assert at.residual_staged == (groups == 13 and blocked_residual)
        assert groups != cut[0] or ((at.channel_waves, at.pixel_waves, at.reduction_waves), at.by_channels) == cut[1:]
    _check_3x3(psb, n, cin, oc, hw, S, exp_bits, residual, ran, 2e-5 if exp_bits == 4 else 2e-3)


# The layers that are left to the kernels with 32 channels at a time: shape = (kernel, digit planes, half tiles, teams).
@pytest.mark.parametrize("n,cin,oc,hw,S,exp_bits,x_absmax,shape", [
    (1, 20, 33, (37, 45), 4, 4, 128, ("WINDOW", 3, 1, 1)),         # one block of channels on a wide image
    (2, 96, 40, (9, 11), 4, 4, 128, ("WINDOW", 3, 1, 1)),          # three blocks, padding channels
    (2, 32, 480, (50, 50), 4, 4, 128, ("WINDOW", 3, 2, 1)),        # two half tiles a wave, a tile that crosses images
    (2, 615, 2, (1, 85), 8, 2, 128, ("WINDOW", 2, 1, 2)),          # two teams: windows of more than 256 slots ...
    (6, 1068, 1, (41, 39), 8, 2, 128, ("WINDOW", 2, 1, 2)),        # ... and of less
    (2, 684, 2, (1, 94), 8, 4, 1, ("WINDOW", 3, 1, 2)),            # three planes (a long reduction of small activations)
    (6, 1068, 1, (41, 39), 8, 4, 1, ("WINDOW", 3, 1, 2)),
    (2, 775, 1, (1, 78), 8, 2, 128, ("MFMA", 2, 1, 0)),            # two planes, a lone team and many blocks: the plain kernel
    (3, 390, 1, (17, 108), 8, 2, 128, ("MFMA", 2, 1, 0))])
@pytest.mark.parametrize("residual", [None, "f32", "i8"])
def test_window_of_32_channels(psb, n, cin, oc, hw, S, exp_bits, x_absmax, shape, residual):
    """3 x 3 layers with 32 channels at a time, or operands from memory."""
    def ran(at, levels, blocked_residual):
        assert (at.kernel, at.planes, at.half_tiles, at.teams) == (getattr(psb, "SHARED_" + shape[0]),) + shape[1:]
    _check_3x3(psb, n, cin, oc, hw, S, exp_bits, residual, ran, 2e-5 if exp_bits == 4 else 2e-3, x_absmax)
