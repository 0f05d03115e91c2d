"""Batched prefills whose forwards pack the requests' real tokens (the tiled
GEMM and the prefill attention) against forwards of equal rows per request on
the wide-row GEMM, bit for bit: more requests than one packed forward takes,
requests with nothing to cache at its start, middle and end, lengths around
the attention's 16-row tiles and 64-row groups, capped rows, and a second
prompt on top of the first."""

import numpy as np
import pytest

from synth import ModelWeights, mini_workloads
from tests.helpers import gpu_setup, kv_views

pytestmark = pytest.mark.gpu

MINIS = {w.name: w for w in mini_workloads()}
LENGTHS = {
    "many": [1, 1, 18] + [int(n) for n in np.random.default_rng(5).integers(1, 60, 66)] + [1],
    "edges": [17, 1, 65, 66, 1, 33, 129, 1],
    "long": [700, 5, 1500, 1, 130],
}


@pytest.mark.parametrize("rows", [0, 24])
@pytest.mark.parametrize("lengths", sorted(LENGTHS))
@pytest.mark.parametrize("name", ["mini_bf16_mixed", "mini_gqa_mixed_b5"])
def test_packed_prefill_equals_equal_rows(name, lengths, rows):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_13076_amd import spade
    n = LENGTHS[lengths]
    w = MINIS[name].with_(batch=len(n))
    max_len = 2 * max(n) + 20
    model, kv1 = gpu_setup(w, ModelWeights(w.model, w.seed), max_len=max_len)
    kv2 = spade.KVCache(model, w.batch, max_len)
    rng = np.random.default_rng(len(n))
    prompts = [[rng.integers(0, w.model.vocab, size=k).astype(np.int32) for k in ks] for ks in (n, n[::-1])]
    model.set_prefill_rows(rows)
    for tiled, kv in ((False, kv1), (True, kv2)):
        kv.buf.zero_()
        model.set_mid_gemm(0 if tiled else 1)
        model.set_big_gemm(0 if tiled else 1)
        for part in prompts:
            kv.prefill_batch(part)
    assert np.array_equal(kv1.get_state(w.batch), kv2.get_state(w.batch))
    lens = kv1.get_state(w.batch)[0]
    assert lens.tolist() == [a + b - 2 for a, b in zip(n, n[::-1])]
    from tests.helpers import k_by_position, v_by_position
    k1, v1 = kv_views(kv1, w.model, max_len)
    k2, v2 = kv_views(kv2, w.model, max_len)
    for b, m in enumerate(lens.tolist()):
        assert torch.equal(k_by_position(k1[:, b], w.model, max_len)[..., :m, :],
                           k_by_position(k2[:, b], w.model, max_len)[..., :m, :]), b
        assert torch.equal(v_by_position(v1[:, b], w.model, max_len)[..., :m],
                           v_by_position(v2[:, b], w.model, max_len)[..., :m]), b
    assert model.device_error() == 0
