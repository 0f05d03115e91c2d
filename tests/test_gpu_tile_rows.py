"""The tiled GEMM as two shapes' calls pick its tile: 33 to 256 rows of a verify
call (ragged last tiles; a vocabulary that ends inside a panel) and 300 to 2040
prompt rows of a prefill forward, against the wide-row GEMM, bit for bit: every
engine adds the same eight k-ranges in the same order.  The picks depend on the
shape too and leave tiles out; test_gpu_tile_variants.py fixes each in turn.
"""

import numpy as np
import pytest

from tests.helpers import kv_views

pytestmark = pytest.mark.gpu

ROWS = [(11, 3), (8, 5), (7, 7), (13, 5), (9, 9), (14, 7), (16, 7), (10, 13), (16, 9), (16, 10), (16, 16)]
SHAPES = {"wide": (1024, 8192, 65500), "deep": (1792, 4096, 32000)}


@pytest.fixture(scope="module", params=sorted(SHAPES))
def setup(request):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_13076_amd import spade
    from synth.configs import ModelShape
    d, ffn, vocab = SHAPES[request.param]
    s = ModelShape("tiles", n_layers=2, d_model=d, n_heads=d // 128, head_dim=128, d_ffn=ffn, vocab=vocab)
    m = spade.Model(s, max_batch=16, max_gamma=15, max_len=2100)
    g = torch.Generator(device=m.device).manual_seed(d)
    draw = lambda *n: (0.03 * torch.randn(n, device=m.device, generator=g)).to(torch.bfloat16)
    for kind, n in (("wq", (d, d)), ("wk", (d, d)), ("wv", (d, d)), ("wo", (d, d)), ("wg", (ffn, d)), ("wu", (ffn, d)),
                    ("wd", (d, ffn))):
        for layer in range(s.n_layers):
            m.load_tensor(kind, layer, draw(*n))
    gain = lambda: 1.0 + 0.1 * torch.randn(d, device=m.device, generator=g)
    for layer in range(s.n_layers):
        m.load_tensor("g_attn", layer, gain())
        m.load_tensor("g_ffn", layer, gain())
    m.load_tensor("g_final", None, gain())
    m.load_tensor("embed", None, draw(vocab, d))
    m.load_tensor("lm_head", None, draw(vocab, d))
    return m, [spade.KVCache(m, 16, 2100) for _ in range(2)]


def _same_cache(m, kvs, what):
    import torch
    for a, b in zip(kv_views(kvs[0], m.shape, 2100), kv_views(kvs[1], m.shape, 2100)):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16)), what


def _engine(m, tiled):
    m.set_mid_gemm(0 if tiled else 1)
    m.set_big_gemm(0 if tiled else 1)


@pytest.mark.parametrize("B,R", ROWS)
def test_verify_rows_bit_identical(setup, B, R):
    import torch
    from paper_2608_13076_amd import spade
    m, kvs = setup
    rng = np.random.default_rng(B * R)
    drafts = rng.integers(0, m.shape.vocab, (B, R - 1)).astype(np.int32)
    lens, pending = np.arange(B, dtype=np.int32), rng.integers(0, m.shape.vocab, B).astype(np.int32)
    out = []
    for tiled, kv in ((False, kvs[0]), (True, kvs[1])):
        kv.buf.zero_()
        kv.set_state(lens, pending)
        _engine(m, tiled)
        buf = spade.VerifyBuffers(m, drafts, None, None, np.zeros(B, np.uint8), True)
        spade.verify(m, kv, buf, 1.0)
        torch.cuda.synchronize()
        out.append((buf.logits.clone(), buf.n.clone(), buf.corr.clone()))
    _engine(m, True)
    a, b = out
    assert torch.isfinite(a[0]).all()
    assert torch.equal(a[0].view(torch.int32), b[0].view(torch.int32)), (B, R)
    assert torch.equal(a[1], b[1]) and torch.equal(a[2], b[2])
    _same_cache(m, kvs, (B, R))
    assert m.device_error() == 0


@pytest.mark.parametrize("n", [300, 515, 1027, 1500, 2040])
def test_prefill_rows_bit_identical(setup, n):
    m, kvs = setup
    prompt = np.random.default_rng(n).integers(0, m.shape.vocab, n + 1).astype(np.int32)
    for tiled, kv in ((False, kvs[0]), (True, kvs[1])):
        kv.buf.zero_()
        kv.set_state(np.zeros(16, np.int32), np.zeros(16, np.int32))
        _engine(m, tiled)
        kv.prefill(0, prompt)
    _engine(m, True)
    _same_cache(m, kvs, n)
    assert m.device_error() == 0
