"""Row statistics and softmax over slices of the vocabulary, at the sizes where
the cut changes (4096 tokens a slice): accept_from_logits with and without
sampling against float64 decisions, softmax_into against float64, for rows that
start off a 16-byte boundary and rows with masked (-inf), +inf and NaN logits.
"""

import numpy as np
import pytest

from oracle import SAMPLE, speculative_rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def model():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_13076_amd import spade
    from synth.configs import ModelShape
    shape = ModelShape("slices", n_layers=1, d_model=256, n_heads=2, head_dim=128, d_ffn=256,
                       vocab=40000, weight_dtype="f32", kv_dtype="f32")
    return spade.Model(shape, max_batch=4, max_gamma=15, max_len=64)


@pytest.mark.parametrize("V,G", [(33, 15), (1024, 15), (1025, 1), (3071, 4), (4095, 2), (4096, 15),
                                  (4097, 3), (8193, 0), (16385, 15), (39999, 5)])
@pytest.mark.parametrize("sampling", [False, True])
def test_accept_over_slices(model, V, G, sampling):
    import torch
    rng = np.random.default_rng(V)
    B, dev = 3, model.device
    logits = (3.0 * rng.standard_normal((B, G + 1, V))).astype(np.float32)
    logits[:, :, rng.permutation(V)[: V // 3]] = -np.inf  # masked tokens
    drafts = logits[:, :G].argmax(-1).astype(np.int32)
    q = rng.dirichlet(np.full(V, 0.5), (B, max(G, 1))).astype(np.float32)[:, :G]
    u = rng.random((B, G + 1)).astype(np.float32)
    modes = np.array([0, 1, 1] if sampling else [0, 0, 0], np.uint8)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    n, c = model.accept_from_logits(up(logits), up(drafts), up(q) if sampling and G else None,
                                    up(u) if sampling else None, up(modes))
    n, c = n.cpu().numpy(), c.cpu().numpy()
    for b in range(B):
        r = speculative_rows(logits[b].astype(np.float64), drafts[b],
                             q[b].astype(np.float64) if modes[b] == SAMPLE else None, u[b], int(modes[b]), 1.0)
        if modes[b] == 0:
            assert n[b] == G and c[b] == int(logits[b, G].argmax())
        else:
            assert not r.pinned_n or n[b] == r.n_accepted
            assert not r.pinned_correction or c[b] == r.correction


@pytest.mark.parametrize("sampling", [False, True])
def test_accept_extreme_rows(model, sampling):
    """All -inf: the lowest id; ties: the lowest id; NaN skipped; +inf wins."""
    import torch
    V, dev = 9001, model.device
    logits = np.full((4, 1, V), -np.inf, np.float32)
    logits[1, 0, [5000, 8999]] = 2.0
    logits[2] = np.random.default_rng(1).standard_normal(V)
    logits[2, 0, 100] = np.nan
    logits[2, 0, 4096] = 50.0
    logits[3, 0, :] = 1.0
    logits[3, 0, 7777] = np.inf
    modes = np.array([0, 0, 0, 0], np.uint8)
    u = torch.full((4, 1), 0.5, device=dev) if sampling else None
    n, c = model.accept_from_logits(torch.from_numpy(logits).to(dev), torch.zeros((4, 0), dtype=torch.int32, device=dev),
                                    None, u, torch.from_numpy(modes).to(dev))
    assert c.cpu().tolist() == [0, 5000, 4096, 7777]


@pytest.mark.parametrize("V", [4096, 4097, 8192, 8193, 128256, 128257])
@pytest.mark.parametrize("offset", [0, 1])
def test_softmax_over_slices(model, V, offset):
    """Against float64: the largest |z - max| here is under 40, so expf's
    argument is off by at most 40 * 2^-24 = 2.4e-6 and the sum adds less."""
    import torch
    from paper_2608_13076_amd import spade
    rows, dev = 5, model.device
    g = torch.Generator(dev).manual_seed(V + offset)
    buf = torch.empty(rows * V + 4, device=dev)
    z = buf[offset:offset + rows * V].view(rows, V)
    z.copy_(3.0 * torch.randn((rows, V), device=dev, generator=g))
    z[1, torch.randperm(V, device=dev, generator=g)[: V // 2]] = -np.inf
    z[2, :] = -np.inf
    z[2, V - 1] = 1.0
    z[3, 7] = np.nan
    z[4, :] = -np.inf
    out = torch.empty(rows * V + 4, device=dev)[offset:offset + rows * V].view(rows, V)
    spade.softmax_into(z, out, 0.8)
    ref = torch.softmax(z[:3].double() / 0.8, -1)
    assert torch.allclose(out[:3].double(), ref, rtol=5e-6, atol=0)
    assert bool(out[3].isnan().all()) and bool(out[4].isnan().all())


@pytest.mark.parametrize("V", [4096, 4097, 33001])
def test_softmax_in_place(model, V):
    """d_probs == d_logits gives what two buffers give (float64, the bound of
    test_softmax_over_slices), whatever the vocabulary."""
    import torch
    from paper_2608_13076_amd import spade
    g = torch.Generator(model.device).manual_seed(V)
    z = 3.0 * torch.randn((3, V), device=model.device, generator=g)
    ref = torch.softmax(z.double() / 0.8, -1)
    spade.softmax_into(z, z, 0.8)
    assert torch.allclose(z.double(), ref, rtol=5e-6, atol=0)


@pytest.mark.parametrize("rows,V", [(600, 5119), (600, 5121), (5, 7167), (5, 7169), (513, 12289)])
@pytest.mark.parametrize("offset", [0, 3])
def test_softmax_where_its_cut_changes(model, rows, V, offset):
    """Against float64; nothing outside the output is written.  Scaled logits
    lie within 20 of 0 and 40 of their maximum: 1 / 0.8 is off by 2^-25 of
    itself (1.2e-6), the two products by 20 * 2^-24 each (2.4e-6), their
    difference by 2^-19 (1.9e-6); the exponential and the sum add under 1e-6."""
    import torch
    from paper_2608_13076_amd import spade
    g = torch.Generator(model.device).manual_seed(rows + V)
    z = 3.0 * torch.randn(rows * V + 4, device=model.device, generator=g)[offset:offset + rows * V].view(rows, V)
    buf = torch.full((rows * V + 8,), 7.0, device=model.device)
    out = buf[offset:offset + rows * V].view(rows, V)
    spade.softmax_into(z, out, 0.8)
    assert torch.allclose(out.double(), torch.softmax(z.double() / 0.8, -1), rtol=7e-6, atol=0)
    assert bool((buf[:offset] == 7.0).all()) and bool((buf[offset + rows * V:] == 7.0).all())
