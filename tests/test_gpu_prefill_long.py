"""Prefill attention on long caches: more than 16 chunks (the merge weights'
general path) and more than 32 (three ring slots instead of four), against
16-row prefill (the verify attention) of the same prompts, bit for bit."""

import numpy as np
import pytest

from synth import ModelWeights, mini_workloads
from tests.helpers import gpu_setup, k_by_position, kv_views, v_by_position

pytestmark = pytest.mark.gpu

MINIS = {w.name: w for w in mini_workloads()}


@pytest.mark.parametrize("name,n", [("mini_bf16_greedy", 4500), ("mini_gqa_greedy", 8700)])
def test_long_prefill_equals_16_rows(name, n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_13076_amd import spade
    w = MINIS[name]
    max_len = n + 20
    model, kv1 = gpu_setup(w, ModelWeights(w.model, w.seed), max_len=max_len)
    kv2 = spade.KVCache(model, w.batch, max_len)
    prompt = np.random.default_rng(n).integers(0, w.model.vocab, n + 1).astype(np.int32)
    model.set_prefill_rows(16)
    kv1.prefill(0, prompt)
    model.set_prefill_rows(0)
    kv2.prefill(0, prompt)
    s = model.shape
    k1, v1 = kv_views(kv1, s, max_len)
    k2, v2 = kv_views(kv2, s, max_len)
    assert torch.equal(k_by_position(k1[:, 0], s, max_len)[..., :n, :], k_by_position(k2[:, 0], s, max_len)[..., :n, :])
    assert torch.equal(v_by_position(v1[:, 0], s, max_len)[..., :n], v_by_position(v2[:, 0], s, max_len)[..., :n])
    assert model.device_error() == 0
