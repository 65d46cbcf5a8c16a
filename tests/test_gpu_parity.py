"""HIP library vs CPU oracle, element by element, through the C-ABI (needs an MI355X).

Bar: int32 accumulators and packed weights bit-exact; fp32 rescale bit-exact in practice, asserted to
1e-6 relative as the contract states.
"""
import numpy as np
import pytest

import helpers
from paper_1904_02205_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def psb():
    import torch
    assert torch.cuda.is_available()
    from paper_1904_02205_amd import psb as m
    m.lib()                      # raises if the HIP library cannot be loaded: no fallback
    yield m
    m.set_mapping(m.MAPPING_AUTO)


def _layer(rng, n, c, oc, hw, k, stride=1, pad=0, groups=1, S=8, s_max=None, std=None, xkind="relu", seed=11,
           layer_id=3, prune=0.0):
    h, w = hw if isinstance(hw, tuple) else (hw, hw)
    kh, kw = k if isinstance(k, tuple) else (k, k)
    wt = synth.he_normal((oc, c // groups, kh, kw), rng) if std is None else synth.normal_weights(
        (oc, c // groups, kh, kw), std, rng)
    if prune:
        wt = synth.prune_by_magnitude(wt, prune)
    if xkind == "relu":
        x = synth.sparse_relu_int8((n, c, h, w), rng)
    elif xkind == "signed":
        x = rng.integers(-128, 128, size=(n, c, h, w)).astype(np.int8)
    else:
        x = synth.uniform_uint4((n, c, h, w), rng)
    st = stride if isinstance(stride, tuple) else (stride, stride)
    pd = pad if isinstance(pad, tuple) else (pad, pad)
    return synth.Layer("t", wt, x, groups=groups, stride=st, pad=pd, S=S, s_max=s_max or S,
                       x_absmax=128 if xkind == "signed" else 127, seed=seed, layer_id=layer_id)


# ------------------------------------------------------------------ weight encoding

def _weight_sets():
    rng = np.random.default_rng(100)
    sets = []
    sets.append(("he", synth.he_normal((70, 20, 3, 3), rng), 127, 16, 0))
    sets.append(("wide", (rng.standard_normal((5, 300)) * 10.0 ** rng.uniform(-8, 1, size=(5, 300))).astype(np.float32),
                 127, 8, 0))
    w = synth.prune_by_magnitude(synth.he_normal((160, 576, 1, 1), rng), 0.9)
    sets.append(("pruned", w, 127, 16, 0))
    w = synth.he_normal((9, 64), rng)
    w[0, :] = 0.0
    w[1, :5] = [1e-40, -1e-42, 2.0 ** -126, -0.0, 2.0 ** -140]
    sets.append(("zeros_subnormals", w, 128, 4, 0))
    sets.append(("exp3", synth.he_normal((33, 17, 3, 3), rng), 15, 32, 3))
    sets.append(("exp5", synth.he_normal((33, 17, 3, 3), rng), 15, 2, 5))
    sets.append(("exp1", synth.he_normal((4, 3, 3, 3), rng), 127, 255, 1))
    sets.append(("tiny_all", (synth.he_normal((4, 8), rng) * 1e-37).astype(np.float32), 127, 8, 0))
    sets.append(("only_subnormal", np.full((2, 3), 1e-41, np.float32), 127, 8, 0))
    sets.append(("all_zero", np.zeros((3, 5), np.float32), 127, 8, 0))
    return sets


@pytest.mark.parametrize("case", _weight_sets(), ids=lambda c: c[0])
def test_quantize_matches_oracle(psb, orc, case):
    import torch
    _, w, xmax, smax, eb = case
    qo = orc.QWeights(w.reshape(w.shape[0], -1), exp_bits=eb, x_absmax=xmax, s_max=smax)
    qg = psb.Weights(torch.from_numpy(w).cuda(), exp_bits=eb, x_absmax=xmax, s_max=smax)
    assert (qg.n_zero, qg.n_flushed, qg.n_live) == (qo.n_zero, qo.n_flushed, qo.n_live)
    if qo.n_live:
        assert (qg.e_top, qg.e_min) == (qo.e_top, qo.e_min)
    assert np.array_equal(qg.export(), helpers.pack_from_oracle(qo))


def test_quantize_error_codes(psb, orc):
    import torch
    for bad in (np.nan, np.inf, -np.inf):
        w = np.ones((2, 40), np.float32)
        w[1, 17] = bad
        with pytest.raises(psb.PsbError) as ei:
            psb.Weights(torch.from_numpy(w).cuda())
        assert ei.value.code == psb.ERR_VALUE
    w = np.ones((1, 2 ** 16), np.float32)
    with pytest.raises(psb.PsbError) as ei:
        psb.Weights(torch.from_numpy(w).cuda(), x_absmax=128, s_max=255)
    assert ei.value.code == psb.ERR_OVERFLOW_UNSAFE
    with pytest.raises(orc.OracleError) as eo:
        orc.QWeights(w, x_absmax=128, s_max=255)
    assert eo.value.code == orc.ERR_OVERFLOW_UNSAFE
    q = psb.Weights(torch.from_numpy(np.ones((4, 8), np.float32)).cuda(), s_max=8)
    x = torch.zeros((2, 8), dtype=torch.int8, device="cuda")
    for S in (0, -1, 9):
        with pytest.raises(psb.PsbError) as ei:
            psb.linear(q, x, S)
        assert ei.value.code == psb.ERR_VALUE
    qc = psb.Weights(torch.ones((4, 2, 3, 3), device="cuda"))      # a conv handle is not a linear layer
    with pytest.raises(ValueError):
        psb.linear(qc, x, 1)
    import ctypes
    acc = torch.zeros((2, 4), dtype=torch.int32, device="cuda")
    rc = psb.lib().psb_linear(qc._h, ctypes.c_void_p(x.data_ptr()), 2, 1, 0, 0, ctypes.c_void_p(acc.data_ptr()), None,
                              None, None, None)
    assert rc == psb.ERR_SHAPE


# ------------------------------------------------------------------ layers, both mappings

def _cases():
    rng = np.random.default_rng(200)
    c = []
    # (id, layer, mappings)
    both = (1, 2, 3)
    c.append(("linear_small", _layer(rng, 5, 37, 9, 1, 1, S=8, xkind="u4", std=0.05), both))
    c.append(("linear_ragged_oc", _layer(rng, 3, 130, 100, 1, 1, S=5, xkind="signed", std=0.05), both))
    c.append(("conv3x3_multi_chunk", _layer(rng, 2, 20, 70, (9, 11), 3, pad=1, S=8), both))
    c.append(("conv3x3_s16", _layer(rng, 1, 16, 64, 7, 3, pad=1, S=16), both))
    c.append(("conv3x3_s32_signed", _layer(rng, 1, 8, 32, 6, 3, pad=1, S=32, xkind="signed"), both))
    c.append(("conv7x7_s2_p3", _layer(rng, 2, 3, 16, (23, 19), 7, stride=2, pad=3, S=8, xkind="signed"), both))
    c.append(("conv1x1_s2", _layer(rng, 2, 24, 40, 9, 1, stride=2, S=4), both))
    c.append(("conv_rect_kernel", _layer(rng, 1, 6, 12, (6, 8), (2, 3), stride=(1, 2), pad=(0, 2), S=3), both))
    c.append(("conv_s1", _layer(rng, 1, 5, 7, 5, 3, pad=1, S=1), both))
    c.append(("conv_s2samples", _layer(rng, 1, 9, 66, 6, 3, pad=1, S=2), both))
    c.append(("conv_s12", _layer(rng, 1, 9, 10, 6, 3, pad=1, S=12), both))
    c.append(("conv_pad3_tiny_image", _layer(rng, 1, 4, 8, 2, 3, pad=3, S=4), both))
    c.append(("pruned_pointwise", _layer(rng, 2, 96, 40, 5, 1, S=16, prune=0.9), both))
    c.append(("grouped", _layer(rng, 2, 8, 12, 7, 3, pad=1, groups=4, S=8), (1, 3)))
    c.append(("depthwise", _layer(rng, 2, 70, 70, 9, 3, pad=1, groups=70, S=16), (1, 3)))
    c.append(("depthwise_s2", _layer(rng, 1, 10, 10, 8, 3, stride=2, pad=1, groups=10, S=4, xkind="signed"), (1, 3)))
    # no padding: every tap of every pixel is inside the image (the product-list kernel drops its bounds checks)
    c.append(("conv3x3_unpadded_s2", _layer(rng, 2, 7, 9, (12, 10), 3, stride=2, S=8), both))
    c.append(("depthwise_unpadded", _layer(rng, 1, 12, 12, (21, 17), (3, 2), groups=12, S=16, xkind="signed"), (1, 3)))
    return c


@pytest.mark.parametrize("case", _cases(), ids=lambda c: c[0])
def test_layer_bit_exact(psb, orc, case):
    _, L, mappings = case
    ref, over, _ = helpers.oracle_layer(orc, L)
    assert over == 0
    for m in mappings:
        psb.set_mapping(m)
        acc, _ = helpers.gpu_layer(psb, L)
        assert np.array_equal(acc, ref), f"mapping {m}"
    psb.set_mapping(psb.MAPPING_AUTO)
    acc, _ = helpers.gpu_layer(psb, L)
    assert np.array_equal(acc, ref)
    acc2, _ = helpers.gpu_layer(psb, L)          # same call again: same bits
    assert np.array_equal(acc2, ref)


def test_query_mapping_names_the_kernel_that_runs(psb):
    rng = np.random.default_rng(250)
    dense = _layer(rng, 1, 16, 64, 7, 3, pad=1, S=8)
    pruned = _layer(rng, 2, 96, 40, 5, 1, S=16, prune=0.9)
    dw = _layer(rng, 2, 70, 70, 9, 3, pad=1, groups=70, S=16)
    geom = lambda L: (L.x.shape[0], L.x.shape[2], L.x.shape[3]) + L.stride + L.pad
    psb.set_mapping(psb.MAPPING_AUTO)
    assert psb.query_mapping(helpers.gpu_quantize(psb, dense), geom(dense)) == psb.MAPPING_CHANNEL_LANE
    assert psb.query_mapping(helpers.gpu_quantize(psb, pruned), geom(pruned)) == psb.MAPPING_PRODUCT_LIST
    assert psb.query_mapping(helpers.gpu_quantize(psb, dw), geom(dw)) == psb.MAPPING_PRODUCT_LIST
    psb.set_mapping(psb.MAPPING_PIXEL_LANE)
    assert psb.query_mapping(helpers.gpu_quantize(psb, dense), geom(dense)) == psb.MAPPING_PIXEL_LANE
    psb.set_mapping(psb.MAPPING_CHANNEL_LANE)
    with pytest.raises(psb.PsbError) as ei:
        psb.query_mapping(helpers.gpu_quantize(psb, dw), geom(dw))
    assert ei.value.code == psb.ERR_SHAPE
    psb.set_mapping(psb.MAPPING_AUTO)


def test_channel_lane_refuses_grouped_layers(psb):
    rng = np.random.default_rng(201)
    L = _layer(rng, 1, 8, 8, 5, 3, pad=1, groups=2, S=4)
    psb.set_mapping(psb.MAPPING_CHANNEL_LANE)
    with pytest.raises(psb.PsbError) as ei:
        helpers.gpu_layer(psb, L)
    assert ei.value.code == psb.ERR_SHAPE
    psb.set_mapping(psb.MAPPING_AUTO)


def test_seed_and_layer_id_select_the_stream(psb, orc):
    rng = np.random.default_rng(202)
    L = _layer(rng, 1, 8, 64, 5, 3, pad=1, S=8)
    outs = []
    for seed, lid in ((0, 0), (2 ** 63 + 12345, 0), (0, 7), (0xFFFFFFFFFFFFFFFF, 0xFFFFFFFF)):
        L.seed, L.layer_id = seed, lid
        ref, _, _ = helpers.oracle_layer(orc, L)
        for m in (1, 2, 3):
            psb.set_mapping(m)
            acc, _ = helpers.gpu_layer(psb, L)
            assert np.array_equal(acc, ref)
        outs.append(ref)
    psb.set_mapping(psb.MAPPING_AUTO)
    assert not np.array_equal(outs[0], outs[1]) and not np.array_equal(outs[0], outs[2])


# ------------------------------------------------------------------ progressive budgets

@pytest.mark.parametrize("mapping", [1, 2, 3])
def test_progressive_bit_exact_and_incremental(psb, orc, mapping):
    rng = np.random.default_rng(300)
    L = _layer(rng, 3, 12, 70, (9, 8), 3, pad=1, S=32, s_max=32)
    oh, ow = L.out_hw
    to = rng.choice([0, 1, 2, 3, 4, 7, 8, 16, 31, 32, 40], size=(3, oh, ow)).astype(np.uint8)   # 40 is clamped to 32
    qo = helpers.oracle_quantize(orc, L)
    ref, over, _ = helpers.oracle_layer(orc, L, qo, budget_to=to)
    assert over == 0
    psb.set_mapping(mapping)
    qg = helpers.gpu_quantize(psb, L)
    acc, _ = helpers.gpu_layer(psb, L, qg, budget_to=to)
    assert np.array_equal(acc, ref)
    # two-call form: first min(to, m) samples, then the rest on top, for aligned and unaligned splits
    for m in (8, 2, 5):
        first = np.minimum(to, m).astype(np.uint8)
        a1, _ = helpers.gpu_layer(psb, L, qg, budget_to=first)
        r1, _, _ = helpers.oracle_layer(orc, L, qo, budget_to=first)
        assert np.array_equal(a1, r1)
        a2, _ = helpers.gpu_layer(psb, L, qg, budget_to=to, budget_from=first, acc_in=a1)
        assert np.array_equal(a2, ref)
    # from > to is clamped to an empty range: accumulators unchanged
    a3, _ = helpers.gpu_layer(psb, L, qg, budget_to=first, budget_from=to, acc_in=a1)
    assert np.array_equal(a3, a1)
    psb.set_mapping(psb.MAPPING_AUTO)


def test_split_reduction_on_a_large_ragged_layer(psb, orc):
    """More than 2^20 outputs, the tap reduction cut in two chunks: the partial sums meet channels-last and a tiled
    pass turns them into [N][OC][OH][OW] accumulators and rescaled values.  100 channels (two blocks, the second
    ragged), 11,550 pixels (not a multiple of the 64-pixel tile, images not a multiple of it either); a uniform call
    with both outputs, then a refinement pair on budget maps."""
    rng = np.random.default_rng(302)
    L = _layer(rng, 2, 8, 100, (75, 77), 3, pad=1, S=4, s_max=8)
    oh, ow = L.out_hw
    assert 2 * 100 * oh * ow > (1 << 20)
    psb.set_mapping(2)
    try:
        qo = helpers.oracle_quantize(orc, L)
        qg = helpers.gpu_quantize(psb, L)
        ref, over, _ = helpers.oracle_layer(orc, L, qo)
        assert over == 0
        mult = (rng.uniform(0.5, 2.0, size=100) * 2.0 ** qo.e_min).astype(np.float32)
        bias = rng.standard_normal(100).astype(np.float32)
        acc, y = helpers.gpu_layer(psb, L, qg, want_y=True, mult=mult, bias=bias)
        assert np.array_equal(acc, ref)
        assert np.array_equal(y, orc.rescale(ref, qo.e_min, S=4, s_max=8, mult=mult, bias=bias))
        to = rng.choice([0, 1, 3, 4, 8], size=(2, oh, ow)).astype(np.uint8)
        first = np.minimum(to, 3).astype(np.uint8)
        r1, _, _ = helpers.oracle_layer(orc, L, qo, budget_to=first)
        r2, _, _ = helpers.oracle_layer(orc, L, qo, budget_to=to)
        a1, _ = helpers.gpu_layer(psb, L, qg, budget_to=first)
        assert np.array_equal(a1, r1)
        a2, y2 = helpers.gpu_layer(psb, L, qg, budget_to=to, budget_from=first, acc_in=a1, want_y=True, mult=mult, bias=bias)
        assert np.array_equal(a2, r2)
        assert np.array_equal(y2, orc.rescale(r2, qo.e_min, budget_to=to, s_max=8, mult=mult, bias=bias))
    finally:
        psb.set_mapping(psb.MAPPING_AUTO)


def test_progressive_constant_map_equals_plain_call(psb):
    rng = np.random.default_rng(301)
    L = _layer(rng, 2, 10, 64, 6, 3, pad=1, S=8, s_max=16)
    oh, ow = L.out_hw
    q = helpers.gpu_quantize(psb, L)
    plain, _ = helpers.gpu_layer(psb, L, q)
    prog, _ = helpers.gpu_layer(psb, L, q, budget_to=np.full((2, oh, ow), 8, np.uint8))
    assert np.array_equal(plain, prog)


def _several_pixels_per_ticket(psb, orc):
    """The kernel variants for a fixed number of generator blocks, 7-bit uniforms, and per-pixel budgets, with pixel counts that
    leave a ragged last group."""
    rng = np.random.default_rng(260)
    cases = [(_layer(rng, 3, 20, 70, (9, 11), 3, pad=1, S=8), 23, False),           # 297 pixels, 3 chunks, 2 channel blocks
             (_layer(rng, 1, 24, 64, (7, 9), 1, S=16), 23, False),                    # single chunk: fused epilogue
             (_layer(rng, 2, 12, 64, (10, 7), 3, pad=1, S=16, s_max=16), 4, False),   # 7-bit uniforms, one block
             (_layer(rng, 2, 16, 64, (9, 9), 3, pad=1, S=32, s_max=32), 23, True)]    # per-pixel ranges
    psb.set_mapping(2)
    try:
        for L, prob_bits, prog in cases:
            oh, ow = L.out_hw
            to = rng.choice([0, 2, 5, 8, 16, 32], size=(L.x.shape[0], oh, ow)).astype(np.uint8) if prog else None
            qo = helpers.oracle_quantize(orc, L, prob_bits=prob_bits)
            qg = helpers.gpu_quantize(psb, L, prob_bits=prob_bits)
            ref, over, _ = helpers.oracle_layer(orc, L, qo, budget_to=to)
            assert over == 0
            acc, _ = helpers.gpu_layer(psb, L, qg, budget_to=to)
            assert np.array_equal(acc, ref), (L.name, prob_bits)
    finally:
        psb.set_mapping(psb.MAPPING_AUTO)


@pytest.mark.parametrize("ppw", [1, 2, 5, 64])
def test_several_pixels_per_wave_and_ticket(psb, orc, ppw):
    """Calls of more than 2^31 tickets hand a wave several pixels per ticket; here the count is forced (benchmark override of the
    channel-lane launcher, which a process reads once: so each count has a process of its own)."""
    import os
    import subprocess
    import sys
    if ppw == 1:
        return _several_pixels_per_ticket(psb, orc)
    tests = os.path.dirname(os.path.abspath(__file__))
    program = ("import sys; sys.path[:0] = [%r, %r]\nimport test_gpu_parity as t\nfrom paper_1904_02205_amd import psb\n"
               "from oracle import binding as orc\nt._several_pixels_per_ticket(psb, orc)\nprint('equal')" % (tests, os.path.dirname(tests)))
    r = subprocess.run([sys.executable, "-c", program], env=dict(os.environ, PSB_OC_PPW=str(ppw)), capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.endswith("equal\n"), r.stderr[-2000:]


# ------------------------------------------------------------------ fp32 rescale

@pytest.mark.parametrize("mapping", [1, 2, 3])
def test_rescale_matches_oracle(psb, orc, mapping):
    rng = np.random.default_rng(400)
    psb.set_mapping(mapping)
    for S, prog in ((8, False), (7, False), (16, True)):
        L = _layer(rng, 2, 20, 70, 6, 3, pad=1, S=S, s_max=32)          # 3 chunks: rescale runs as its own kernel
        oh, ow = L.out_hw
        to = rng.choice([0, 2, 3, 8, 16, 32], size=(2, oh, ow)).astype(np.uint8) if prog else None
        qo = helpers.oracle_quantize(orc, L)
        mult = (np.ldexp(1.0, qo.e_min) * rng.uniform(0.5, 2.0, size=70)).astype(np.float32)
        bias = rng.standard_normal(70).astype(np.float32)
        for mu, bi in ((None, None), (mult, bias)):
            acc, y = helpers.gpu_layer(psb, L, budget_to=to, want_y=True, mult=mu, bias=bi)
            ref_acc, _, _ = helpers.oracle_layer(orc, L, qo, budget_to=to)
            ref_y = orc.rescale(ref_acc, qo.e_min, S=None if prog else S, s_max=32, budget_to=to, mult=mu, bias=bi)
            assert np.array_equal(acc, ref_acc)
            assert np.array_equal(y, ref_y)                       # in practice: 0 ulp
            np.testing.assert_allclose(y, ref_y, rtol=1e-6, atol=0)
    # single chunk: rescale fused into the layer kernel
    L = _layer(rng, 3, 40, 64, 1, 1, S=5, s_max=8, xkind="u4", std=0.05)
    L.linear = True
    qo = helpers.oracle_quantize(orc, L)
    acc, y = helpers.gpu_layer(psb, L, want_y=True)
    ref_acc, _, _ = helpers.oracle_layer(orc, L, qo)
    assert np.array_equal(acc, ref_acc)
    assert np.array_equal(y, orc.rescale(ref_acc, qo.e_min, S=5))
    psb.set_mapping(psb.MAPPING_AUTO)


# ------------------------------------------------------------------ generator cross-check on the box

def test_oracle_philox_against_rocrand_host_generator(orc):
    """An independent implementation of Philox4x32-10 (rocRAND's host generator, if the library is there)."""
    import ctypes as C
    try:
        R = C.CDLL("librocrand.so")
    except OSError:
        pytest.skip("rocRAND not installed")
    gen = C.c_void_p()
    if R.rocrand_create_generator_host(C.byref(gen), 404) != 0:      # ROCRAND_RNG_PSEUDO_PHILOX4_32_10
        pytest.skip("rocRAND host generator unavailable")
    R.rocrand_set_seed.argtypes = [C.c_void_p, C.c_ulonglong]
    R.rocrand_generate.argtypes = [C.c_void_p, C.c_void_p, C.c_size_t]
    seed = 0x0123456789ABCDEF
    assert R.rocrand_set_seed(gen, seed) == 0
    out = np.zeros(64, dtype=np.uint32)
    if R.rocrand_generate(gen, out.ctypes.data_as(C.c_void_p), out.size) != 0:
        pytest.skip("rocRAND host generation failed")
    R.rocrand_destroy_generator(gen)
    # whatever order the library emits its blocks in, the first 64 words must be made of the blocks of
    # counters 0..15 under key (seed lo, seed hi)
    key = [seed & 0xFFFFFFFF, seed >> 32]
    blocks = {tuple(orc.philox([c, 0, 0, 0], key)) for c in range(16)}
    got = {tuple(int(v) for v in out[i:i + 4]) for i in range(0, 64, 4)}
    assert got == blocks


def test_two_handles_on_two_streams(psb, orc):
    """Calls on different handles may overlap in time: two layers enqueued alternately on two streams (default
    priority) give the bits of the calls made one after the other."""
    import torch
    rng = np.random.default_rng(400)
    La = _layer(rng, 2, 32, 64, 12, 3, pad=1, S=16, seed=5, layer_id=1)
    Lb = _layer(rng, 2, 20, 70, (9, 11), 3, pad=1, S=8, seed=6, layer_id=2)
    refs = [helpers.oracle_layer(orc, L)[0] for L in (La, Lb)]
    qs = [helpers.gpu_quantize(psb, L) for L in (La, Lb)]
    xs = [torch.from_numpy(L.x).cuda() for L in (La, Lb)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = [[], []]
    torch.cuda.synchronize()
    for rep in range(6):
        for i, L in enumerate((La, Lb)):
            with torch.cuda.stream(streams[i]):
                outs[i].append(psb.conv2d(qs[i], xs[i], L.S, pad=L.pad, seed=L.seed, layer_id=L.layer_id))
    torch.cuda.synchronize()
    for i in range(2):
        for acc in outs[i]:
            assert np.array_equal(acc.cpu().numpy(), refs[i])
