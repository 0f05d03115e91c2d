"""Every built tile of the tiled GEMM, unsplit (weights with and without the
non-temporal policy: up to four row groups and more) and k-split, for every
projection and the LM head, at a full and a ragged last row group, against the
wide-row GEMM, bit for bit.  Four and eleven k-blocks: some of the eight
k-ranges, and some splits, are empty.  The vocabulary ends inside a panel; the
requests' contexts end in different blocks of the cache.
"""

import numpy as np
import pytest

from tests.helpers import kv_views

pytestmark = pytest.mark.gpu

TILES = [(rt, 2) for rt in (2, 3, 4, 5, 6, 8, 9)] + [(rt, 1) for rt in (4, 5, 6, 7, 9)]
B_MAX, CTX = 64, 340


@pytest.fixture(scope="module")
def setup():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_13076_amd import spade
    from synth.configs import ModelShape
    d, ffn, vocab = 1024, 2816, 4090
    s = ModelShape("tiles", n_layers=2, d_model=d, n_heads=8, head_dim=128, d_ffn=ffn, vocab=vocab, n_kv_heads=2)
    m = spade.Model(s, max_batch=B_MAX, max_gamma=15, max_len=CTX + 20)
    g = torch.Generator(device=m.device).manual_seed(7)
    draw = lambda *n: (0.03 * torch.randn(n, device=m.device, generator=g)).to(torch.bfloat16)
    for layer in range(s.n_layers):
        for kind, n in (("wq", (d, d)), ("wk", (256, d)), ("wv", (256, d)), ("wo", (d, d)), ("wg", (ffn, d)),
                        ("wu", (ffn, d)), ("wd", (d, ffn))):
            m.load_tensor(kind, layer, draw(*n))
        for kind in ("g_attn", "g_ffn"):
            m.load_tensor(kind, layer, 1.0 + 0.1 * torch.randn(d, device=m.device, generator=g))
    m.load_tensor("g_final", None, 1.0 + 0.1 * torch.randn(d, device=m.device, generator=g))
    m.load_tensor("embed", None, draw(vocab, d))
    m.load_tensor("lm_head", None, draw(vocab, d))
    kv = spade.KVCache(m, B_MAX, CTX + 20)
    kv.buf.zero_()
    rng = np.random.default_rng(11)
    kv.prefill_batch([rng.integers(0, vocab, n).astype(np.int32) for n in rng.integers(1, CTX, B_MAX)])
    return m, kv, kv.buf.clone(), kv.get_state(B_MAX), {}


def _call(setup, B, R):
    """Logits, n, correction and the whole cache after a verify call of B x R rows."""
    import torch
    from paper_2608_13076_amd import spade
    m, kv, cache, (lens, pending), _ = setup
    kv.buf.copy_(cache)
    kv.set_state(lens, pending)
    drafts = np.random.default_rng(B * R).integers(0, m.shape.vocab, (B, R - 1)).astype(np.int32)
    buf = spade.VerifyBuffers(m, drafts, None, None, np.zeros(B, np.uint8), True)
    spade.verify(m, kv, buf, 1.0)
    torch.cuda.synchronize()
    return buf.logits, buf.n, buf.corr, kv.buf.clone()


def _reference(setup, B, R):
    m, refs = setup[0], setup[4]
    if (B, R) not in refs:
        m.set_mid_gemm(1)
        m.set_big_gemm(1)
        assert all(m.gemm_engine(k, B * R) == 1 for k in ("qkv", "o", "gu", "down", "lm"))
        refs[B, R] = _call(setup, B, R)
        m.set_mid_gemm(0)
        m.set_big_gemm(0)
    return refs[B, R]


def _rows(lo, hi, ragged):
    """(requests, rows each) whose product lies in (lo, hi]: the largest, a multiple of 16 or not."""
    return max(((b, r) for b in range(1, B_MAX + 1) for r in range(1, 17)
                if lo < b * r <= hi and (b * r % 16 != 0) == ragged), key=lambda x: (x[0] * x[1], x[1]))


@pytest.mark.parametrize("rt,p", TILES)
def test_every_tile_bit_identical(setup, rt, p):
    import torch
    m = setup[0]
    # one and two row groups (split too: 144 rows fit the workspace), five row groups
    few = [(16 * rt - 16, 16 * rt), (16 * rt - 16, 16 * rt + 16)]
    sizes = [_rows(max(lo, 32), min(max(hi, 48), 144), ragged) for lo, hi in few for ragged in (False, True)]
    many = [_rows(64 * rt, 80 * rt, ragged) for ragged in (False, True)]
    for B, R in sorted(set(sizes + many)):
        want = _reference(setup, B, R)
        for ks in (1, 2, 3, 8) if B * R <= 144 else (1,):
            print(f"tile ({rt}, {p}) k-splits {ks}: {B} x {R} rows", flush=True)
            m.set_tile_gemm(rt, p, ks)
            assert all(m.gemm_engine(k, B * R) == 2 for k in ("qkv", "o", "gu", "down", "lm"))
            got = _call(setup, B, R)
            for name, a, b in zip(("logits", "n", "correction", "cache"), want, got):
                assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), (name, rt, p, ks, B, R)
    m.set_tile_gemm()
    assert torch.isfinite(want[0]).all() and m.device_error() == 0


def test_setter_rejects_tiles_that_are_not_built(setup):
    from paper_2608_13076_amd import spade
    for bad in ((7, 2, 0), (2, 1, 0), (8, 1, 0), (4, 0, 0), (0, 1, 0), (4, 2, 9), (4, 2, -1)):
        with pytest.raises(spade.SpadeError):
            setup[0].set_tile_gemm(*bad)
