"""The two per-product kernels against the oracle around the sizes where the automatic choice changes between them, and the
channel entropy over tile remainders."""
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


@pytest.mark.parametrize("oc,prune,hw,S", [(1, 0.0, (5, 3), 4), (31, 0.0, (9, 29), 10), (33, 0.5, (9, 29), 3), (64, 0.6, (16, 16), 8),
                                           (65, 0.0, (16, 17), 16), (70, 0.7, (7, 7), 5)])
def test_automatic_choice(psb, orc, oc, prune, hw, S):
    rng = np.random.default_rng(oc)
    w = synth.he_normal((oc, 9, 3, 3), rng)
    L = synth.Layer("edge", synth.prune_by_magnitude(w, prune) if prune else w, synth.sparse_relu_int8((1, 9) + hw, rng), pad=(1, 1),
                    S=S, s_max=16, seed=3, layer_id=2)
    q = helpers.gpu_quantize(psb, L)
    ref, over, _ = helpers.oracle_layer(orc, L)
    for mapping in (psb.MAPPING_AUTO, psb.MAPPING_CHANNEL_LANE, psb.MAPPING_PRODUCT_LIST):
        psb.set_mapping(mapping)
        acc, _ = helpers.gpu_layer(psb, L, q)
        assert over == 0 and np.array_equal(acc, ref), mapping
    psb.set_mapping(psb.MAPPING_AUTO)


@pytest.mark.parametrize("n,c,h,w", [(1, 1, 1, 1), (2, 15, 3, 5), (1, 17, 4, 4), (3, 40, 7, 7), (1, 512, 1, 17)])
def test_channel_entropy_remainders(psb, orc, n, c, h, w):
    """Fewer channels than lanes per pixel, pixels that leave a last tile in part; the whole range of activations.  Both sides
    evaluate in binary64 and round once, so at most one binary32 ulp apart; the mask may differ only at its threshold."""
    import torch
    rng = np.random.default_rng(c)
    act = rng.integers(-128, 128, size=(n, c, h, w)).astype(np.int8)
    ent, mean, bud = psb.attention_budget(torch.from_numpy(act).cuda(), 0.03, 4, 9)
    z = act.astype(np.float64) * np.float64(np.float32(0.03))
    z = z - z.max(axis=1, keepdims=True)
    e = np.exp(z)
    Z = e.sum(axis=1)
    ref = np.log(Z) - (e * z).sum(axis=1) / Z
    got = ent.cpu().numpy()
    assert np.all(np.abs(got - ref) <= np.spacing(np.maximum(np.abs(ref), 1e-12).astype(np.float32)) + 1e-13)
    clear = np.abs(ref - ref.mean(axis=(1, 2), keepdims=True)) > 1e-6
    assert np.array_equal(bud.cpu().numpy()[clear], np.where(ref > ref.mean(axis=(1, 2), keepdims=True), 9, 4)[clear])
