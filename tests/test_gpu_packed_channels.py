"""Channel-lane kernel: last channel blocks of at most 32 channels, computed for several pixels at a time, against the oracle."""
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
    m.set_mapping(m.MAPPING_CHANNEL_LANE)
    yield m
    m.set_mapping(m.MAPPING_AUTO)


# channels around the slots of 8, 16 and 32, alone and behind whole blocks; samples in whole and in parts of generator blocks.
# (2, 61, 67) splits the taps, (3, 57, 55) does not behind a whole block; pixel counts are no multiple of a ticket's.
@pytest.mark.parametrize("nhw", [(2, 61, 67), (3, 57, 55)])
@pytest.mark.parametrize("oc,S,prob_bits", [(1, 8, 23), (8, 10, 23), (9, 5, 8), (16, 4, 4), (17, 16, 23), (32, 12, 7), (33, 8, 23), (65, 32, 23),
                                            (72, 6, 6), (80, 7, 23), (96, 16, 4), (129, 3, 23)])
def test_packed_last_block(psb, orc, nhw, oc, S, prob_bits):
    rng = np.random.default_rng(oc * 31 + S)
    n, h, w = nhw
    L = synth.Layer("packed", synth.he_normal((oc, 7, 3, 3), rng), synth.sparse_relu_int8((n, 7, h, w), rng), pad=(1, 1), stride=(1, 1), S=S,
                    s_max=S, seed=9, layer_id=4)
    q = helpers.gpu_quantize(psb, L, prob_bits=prob_bits)
    qo = helpers.oracle_quantize(orc, L, prob_bits=prob_bits)
    ref, over, _ = helpers.oracle_layer(orc, L, qo)
    acc, y = helpers.gpu_layer(psb, L, q, want_y=True)
    assert over == 0 and psb.last_mapping() == psb.MAPPING_CHANNEL_LANE and np.array_equal(acc, ref)
    np.testing.assert_allclose(y, orc.rescale(ref, qo.e_min, S=S, s_max=S, budget_to=None), rtol=1e-6, atol=0)
    again, _ = helpers.gpu_layer(psb, L, q)                  # the scratch accumulators are left at zero
    assert np.array_equal(again, ref)
