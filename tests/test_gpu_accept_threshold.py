"""The probability that the accept step gives a draft, to the last bit: for one
row it must not depend on the correction's schedule, on gamma or on whose
scratch the call uses.  With q = 1 at the draft the test is u < p, so a
bisection over u's float32 bits finds p itself.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

B = 24


@pytest.fixture(scope="module")
def model():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_13076_amd import spade
    from synth.configs import ModelShape
    shape = ModelShape("thresholds", n_layers=1, d_model=256, n_heads=2, head_dim=128, d_ffn=256,
                       vocab=66000, weight_dtype="f32", kv_dtype="f32")
    return spade.Model(shape, max_batch=B, max_gamma=15, max_len=64)


def _accepted_p(call, logits, drafts, q, G):
    """Bits of the least u at which request b's first draft is rejected."""
    import torch
    dev = logits.device
    lo = torch.zeros(B, dtype=torch.int32, device=dev)
    hi = torch.full((B,), 0x3F800000, dtype=torch.int32, device=dev)  # 1.0
    u = torch.full((B, G + 1), 0.5, device=dev)
    modes = torch.ones(B, dtype=torch.uint8, device=dev)
    for _ in range(31):
        mid = lo + (hi - lo) // 2
        u[:, 0] = mid.view(torch.float32)
        n, _ = call(logits, drafts, q, u, modes)
        lo, hi = torch.where(n > 0, mid, lo), torch.where(n > 0, hi, mid)
    return hi.cpu().numpy()


@pytest.mark.parametrize("V", [1001, 1025, 3072, 4096, 4097, 20000, 65999])
def test_accept_probability_bit_identical(model, V):
    import torch
    from paper_2608_13076_amd import spade
    dev = model.device
    g = torch.Generator(dev).manual_seed(V)
    logits = 2.5 * torch.randn((B, 16, V), device=dev, generator=g)
    drafts = torch.randint(0, V, (B, 15), device=dev, dtype=torch.int32, generator=g)
    n = torch.empty(B, dtype=torch.int32, device=dev)
    c, err = torch.empty_like(n), torch.zeros(1, dtype=torch.int32, device=dev)

    def noalloc(lg, d, q, u, modes):
        spade.accept_from_logits_noalloc(lg, d, q, u, modes, 1.0, n, c, err)
        return n, c

    got = {}
    for G in (1, 6, 15):
        lg, d = logits[:, :G + 1].contiguous(), drafts[:, :G].contiguous()
        q = torch.zeros((B, G, V), device=dev).scatter_(2, d.long()[..., None], 1.0)
        for mode in (0, 1, 2):
            model.set_correction_slices(mode)
            got[f"gamma {G}, correction mode {mode}"] = _accepted_p(model.accept_from_logits, lg, d, q, G)
        model.set_correction_slices(0)
        got[f"gamma {G}, static scratch"] = _accepted_p(noalloc, lg, d, q, G)
    ref = got["gamma 1, correction mode 0"]
    for what, p in got.items():
        assert np.array_equal(p, ref), (what, int((p != ref).sum()))
    # z - lse: a rounding of about 2^-24 * 16 each; the sum and the two
    # exponentials a few 2^-24 more
    p64 = torch.softmax(logits[:, 0].double(), -1).gather(1, drafts[:, :1].long())[:, 0].cpu().numpy()
    assert np.all(np.abs(ref.view(np.float32) / p64 - 1.0) < 6e-6)
