"""Per-product layer kernels vs the oracle over all sample ranges: whole generator blocks, first and last blocks that are
drawn in part (32-bit uniforms: 4 samples a block, 7-bit: 16), every number of blocks, refinement from any sample to any
other; and the scratch accumulators of a handle over calls of changing size."""
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
    m.lib()
    yield m
    m.set_mapping(m.MAPPING_AUTO)


def _layer(n=1, oc=70, hw=(5, 6), s_max=40, cin=12):
    rng = np.random.default_rng(77)
    return synth.Layer("ranges", synth.he_normal((oc, cin, 3, 3), rng), synth.sparse_relu_int8((n, cin) + hw, rng), pad=(1, 1), S=1,
                       s_max=s_max, seed=9, layer_id=4)


@pytest.mark.parametrize("mapping", [2, 3])
@pytest.mark.parametrize("prob_bits", [23, 4])
def test_every_sample_count(psb, orc, prob_bits, mapping):
    L = _layer()
    qo, qg = helpers.oracle_quantize(orc, L, prob_bits=prob_bits), helpers.gpu_quantize(psb, L, prob_bits=prob_bits)
    psb.set_mapping(mapping)
    for S in list(range(1, 25)) + [26, 28, 31, 32, 33, 36, 37, 40]:
        ref, over, _ = helpers.oracle_layer(orc, L, qo, S=S)
        acc, _ = helpers.gpu_layer(psb, L, qg, S=S)
        assert over == 0 and np.array_equal(acc, ref), S


@pytest.mark.parametrize("mapping", [2, 3])
@pytest.mark.parametrize("prob_bits", [23, 4])
def test_every_refinement_range(psb, orc, prob_bits, mapping):
    """30 pixels with ranges [from, to) that start and end anywhere, empty ones among them, six maps."""
    L = _layer()
    qo, qg = helpers.oracle_quantize(orc, L, prob_bits=prob_bits), helpers.gpu_quantize(psb, L, prob_bits=prob_bits)
    psb.set_mapping(mapping)
    rng = np.random.default_rng(5)
    for _ in range(6):
        first = rng.integers(0, 24, size=(1, 5, 6)).astype(np.uint8)
        to = np.minimum(first + rng.integers(0, 26, size=first.shape), 45).astype(np.uint8)     # s_max clamps the largest
        ref0, _, _ = helpers.oracle_layer(orc, L, qo, budget_to=first)
        ref, over, _ = helpers.oracle_layer(orc, L, qo, budget_to=to, budget_from=first, acc_in=ref0)
        acc0, _ = helpers.gpu_layer(psb, L, qg, budget_to=first)
        acc, _ = helpers.gpu_layer(psb, L, qg, budget_to=to, budget_from=first, acc_in=acc0)
        assert over == 0 and np.array_equal(acc0, ref0) and np.array_equal(acc, ref)


def test_scratch_accumulators_over_calls_of_changing_size(psb, orc):
    """The partial sums of a split reduction meet in memory that a call leaves at zero: small, large, small again, a linear
    layer, with and without accumulators handed out, twice each."""
    psb.set_mapping(2)
    big = _layer(n=3, hw=(13, 11), s_max=8)
    q = helpers.gpu_quantize(psb, big)
    qo = helpers.oracle_quantize(orc, big)
    for n, hw in [(1, (5, 6)), (3, (13, 11)), (1, (5, 6)), (2, (7, 16)), (3, (13, 11))]:
        L = _layer(n=n, hw=hw, s_max=8)
        ref, _, _ = helpers.oracle_layer(orc, L, qo, S=8)
        for _ in range(2):
            acc, y = helpers.gpu_layer(psb, L, q, S=8, want_y=True)
            assert np.array_equal(acc, ref)
            assert np.array_equal(y, orc.rescale(ref, qo.e_min, S=8, s_max=8))
    lin = synth.config1(batch=5, k=300, oc=70)
    ref, _, _ = helpers.oracle_layer(orc, lin)
    ql = helpers.gpu_quantize(psb, lin)
    for _ in range(2):
        acc, _ = helpers.gpu_layer(psb, lin, ql)
        assert np.array_equal(acc, ref)
