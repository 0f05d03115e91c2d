"""The calls a user of this library makes, as measurable cases.

A case is one pass of a serving or drafting loop through the public binding
(``paper_2608_13076_amd.spade``):

``verify``  restore the committed state, one ``verify`` of gamma drafts for B
            requests over their cached contexts, ``commit`` (the cloud step of
            Algorithm 1); gamma 0 is plain decoding of one token per request.
``draft``   the edge's step: a ``verify`` without drafts on the draft model and
            ``softmax_into`` for the distribution its token came from.
``prefill`` one prompt into an empty cache; the whole cache is the result.
``ttft``    the prompts of B requests into an empty cache and the logits and
            token that follow each (time to first token).
``accept``  ``accept_from_logits``: the decision step alone, for logits that
            another program computed.

Shapes are the ones of ``synth.configs`` (7B, 13B, 33B and grouped-query 8B
shaped bf16 verifiers, the tiny float32 one).  Two cases run the whole 7B
model; the others run its blocks -- a few layers and the LM head -- so that a
result stays close to what one layer's arithmetic gives.  Weights are N(0,
0.02) as in the rest of the repository, prompts and greedy requests' drafts
uniform ids; sampling requests draft from q = softmax(N(0, 1)).
"""

import math
import random
from types import SimpleNamespace

import numpy as np
import torch

from paper_2608_13076_amd import spade

DEV = "cuda:0"

# name: layers of the whole model, d_model, query heads, K/V heads, d_ffn, vocab, RoPE base, data type
_DIMS = {
    "tiny": (2, 256, 4, 4, 1024, 4096, 10000.0, "f32"),
    "7b": (32, 4096, 32, 32, 11008, 32000, 10000.0, "bf16"),
    "13b": (40, 5120, 40, 40, 13824, 32000, 10000.0, "bf16"),
    "33b": (60, 6656, 52, 52, 17920, 32000, 10000.0, "bf16"),
    "8b": (32, 4096, 32, 8, 14336, 128256, 500000.0, "bf16"),
}


def _case(kind, model, layers, batch, gamma, lo, hi, mode, lens_seed=0, name=None):
    """lo..hi: the range of the cached tokens (prompt tokens) of a request;
    each request's own count is drawn from it by lens_seed."""
    c = {"kind": kind, "model": model, "layers": layers, "batch": batch, "gamma": gamma, "lo": lo, "hi": hi,
         "mode": mode, "lens_seed": lens_seed}
    if name:
        c = {"name": name, **c}
    return c


def listed():
    return [
        # the smallest call: a tiny float32 verifier, where launches and latency count
        _case("verify", "tiny", 2, 1, 4, 128, 128, "sample", name="verify_tiny_f32"),
        # the edge's draft step: an early exit of the 8B shape drafts one token
        _case("draft", "8b", 4, 1, 0, 777, 777, "sample", name="draft_8b_exit4"),
        # the benchmark's own call: the whole 7B verifier, one request
        _case("verify", "7b", 32, 1, 5, 1024, 1024, "greedy", name="verify_7b_b1"),
        # one sampling request on the 13B shape (operand too long for one LDS copy)
        _case("verify", "13b", 4, 1, 8, 2048, 2048, "sample", name="verify_13b_b1_sample"),
        # a small batch on the 33B shape
        _case("verify", "33b", 2, 4, 6, 1536, 1536, "greedy", name="verify_33b_b4"),
        # an ordinary half-full batch, odd row count and ragged contexts
        _case("verify", "8b", 4, 7, 6, 100, 2500, "mixed", 3, name="verify_8b_b7"),
        # full batches with ragged contexts: multi-head and grouped-query
        _case("verify", "7b", 4, 16, 8, 256, 4096, "mixed", 1, name="verify_7b_b16"),
        _case("verify", "8b", 4, 16, 8, 256, 4096, "mixed", 2, name="verify_8b_b16"),
        # a chat-sized prompt into the whole 7B verifier
        _case("prefill", "7b", 32, 1, 0, 1019, 1019, "greedy", name="prefill_7b_1k"),
        # short ragged prompts of a few requests, up to the first token
        _case("ttft", "8b", 4, 5, 0, 33, 210, "greedy", 4, name="ttft_8b_short_b5"),
        # long ragged prompts of a full batch, up to the first token: the largest pass
        _case("ttft", "7b", 8, 16, 0, 256, 4096, "mixed", 1, name="ttft_7b_b16"),
        # decisions alone over the 128K vocabulary
        _case("accept", "8b", 1, 16, 8, 0, 0, "mixed", name="accept_8b_b16"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["verify"] * 6 + ["prefill", "ttft", "draft", "accept"])
    model = rng.choice(["7b", "8b", "13b", "33b", "7b", "8b", "tiny"])
    if kind == "accept" and model == "tiny":
        model = "7b"
    if kind == "prefill" and model == "tiny":
        model = "7b"
    layers = {"tiny": 2, "7b": rng.randint(2, 6), "8b": rng.randint(2, 6), "13b": rng.randint(2, 4),
              "33b": rng.randint(1, 2)}[model]
    mode = rng.choice(["greedy", "sample", "mixed"])
    seed = rng.randrange(1 << 20)
    if kind == "accept":
        return _case(kind, model, 1, _log_int(rng, 1, 32), rng.randint(1, 15), 0, 0, mode, seed)
    if kind == "draft":
        n = _log_int(rng, 1, 4096)
        return _case(kind, model, layers, 1, 0, n, n, mode, seed)
    if kind == "prefill":
        n = _log_int(rng, 17, 3000)
        return _case(kind, model, min(layers, 4), 1, 0, n, n, "greedy", seed)
    batch = 1 if rng.random() < 0.25 else _log_int(rng, 1, 32 if kind == "verify" else 16)
    lo = _log_int(rng, 2, 2048)
    hi = min(4096, lo * rng.randint(1, 8))
    if model == "tiny":
        lo, hi = min(lo, 500), min(hi, 500)
    gamma = rng.choice([0, 1, 2, 3, 4, 4, 5, 5, 6, 6, 7, 8, 8, 11, 15]) if kind == "verify" else 0
    return _case(kind, model, min(layers, 4), batch, gamma, lo, hi, mode, seed)


# --------------------------------------------------------------------------- inputs

def _shape(case):
    _, d, h, kvh, f, v, theta, dt = _DIMS[case["model"]]
    return SimpleNamespace(name=case["model"], n_layers=case["layers"], d_model=d, n_heads=h, head_dim=d // h,
                           d_ffn=f, vocab=v, weight_dtype=dt, kv_dtype=dt, rms_eps=1e-5, rope_theta=theta,
                           n_kv_heads=kvh, kv_heads=kvh)


def _lens(case):
    """Cached tokens of each request (a prompt has one more: the pending token)."""
    r = random.Random(case["lens_seed"])
    return [r.randint(case["lo"], case["hi"]) for _ in range(case["batch"])]


def _modes(case):
    return [{"greedy": 0, "sample": 1, "mixed": b % 2}[case["mode"]] for b in range(case["batch"])]


def _weights(s, seed):
    """(kind, layer, tensor) of every weight, on the GPU, from the seed alone."""
    g = torch.Generator(DEV).manual_seed(seed)
    dt = torch.bfloat16 if s.weight_dtype == "bf16" else torch.float32
    d, f, v, dkv = s.d_model, s.d_ffn, s.vocab, s.kv_heads * s.head_dim

    def mat(n, k):
        return torch.empty((n, k), dtype=dt, device=DEV).normal_(0.0, 0.02, generator=g)

    def gain():
        return 1.0 + 0.1 * torch.randn(d, device=DEV, generator=g)

    yield "embed", None, mat(v, d)
    for l in range(s.n_layers):
        yield "g_attn", l, gain()
        yield "wq", l, mat(d, d)
        yield "wk", l, mat(dkv, d)
        yield "wv", l, mat(dkv, d)
        yield "wo", l, mat(d, d)
        yield "g_ffn", l, gain()
        yield "wg", l, mat(f, d)
        yield "wu", l, mat(f, d)
        yield "wd", l, mat(d, f)
    yield "g_final", None, gain()
    yield "lm_head", None, mat(v, d)


def _prompts(case, vocab, seed):
    r = np.random.default_rng([seed, 1])
    return [r.integers(0, vocab, n + 1, dtype=np.int32) for n in _lens(case)]


def _calls(case, vocab, seed):
    """Drafts [B, gamma], q (on the GPU, or None), uniforms and modes of one call."""
    B, G = case["batch"], case["gamma"]
    r = np.random.default_rng([seed, 2])
    modes = np.array(_modes(case), dtype=np.uint8)
    drafts = r.integers(0, vocab, (B, G), dtype=np.int32)
    u = r.random((B, G + 1), dtype=np.float32)
    q = None
    if G and modes.any():
        g = torch.Generator(DEV).manual_seed(seed + 2)
        q = torch.softmax(torch.randn((B, G, vocab), device=DEV, generator=g), -1)
        picks = torch.multinomial(q.view(B * G, vocab), 1, generator=g).view(B, G).cpu().numpy()
        drafts = np.where(modes[:, None] == 1, picks, drafts).astype(np.int32)
    return drafts, q, u, modes


def _logit_calls(case, vocab, seed):
    """An accept call's logits (peaked as a language model's are), drafts that
    the draft distribution proposes, q, uniforms and modes."""
    B, G = case["batch"], case["gamma"]
    g = torch.Generator(DEV).manual_seed(seed + 3)
    logits = 2.5 * torch.randn((B, G + 1, vocab), device=DEV, generator=g)
    q = torch.softmax(logits[:, :G] + 0.5 * torch.randn((B, G, vocab), device=DEV, generator=g), -1)
    modes = torch.tensor(_modes(case), dtype=torch.uint8, device=DEV)
    picks = torch.multinomial(q.view(B * G, vocab), 1, generator=g).view(B, G)
    best = logits[:, :G].argmax(-1)
    other = torch.randint(0, vocab, (B, G), device=DEV, generator=g)
    keep = torch.rand((B, G), device=DEV, generator=g) < 0.8
    drafts = torch.where(modes[:, None] == 1, picks, torch.where(keep, best, other)).to(torch.int32)
    u = torch.rand((B, G + 1), device=DEV, generator=g)
    return logits, drafts.contiguous(), q, u, modes


def prepare(case, seed):
    s = _shape(case)
    st = SimpleNamespace(case=case)
    if case["kind"] == "accept":
        st.model = spade.Model(s, case["batch"], case["gamma"], 256, DEV)
        st.args = _logit_calls(case, s.vocab, seed)
        return st
    lens = _lens(case)
    max_len = max(lens) + case["gamma"] + 2
    st.model = spade.Model(s, case["batch"], case["gamma"], max_len, DEV)
    for kind, layer, t in _weights(s, seed):
        st.model.load_tensor(kind, layer, t)
    st.kv = spade.KVCache(st.model, case["batch"], max_len)
    st.prompts = _prompts(case, s.vocab, seed)
    if case["kind"] in ("prefill", "ttft"):
        st.kv.buf.zero_()
    else:
        st.kv.prefill_batch(st.prompts)
    st.state = st.kv.snapshot(case["batch"])
    if case["kind"] != "prefill":
        drafts, q, u, modes = _calls(case, s.vocab, seed)
        st.buf = spade.VerifyBuffers(st.model, drafts, None, u, modes)
        st.buf.q = q
    if case["kind"] == "draft":
        st.probs = torch.empty_like(st.buf.logits)
    return st


def run(st):
    kind = st.case["kind"]
    if kind == "accept":
        logits, drafts, q, u, modes = st.args
        return st.model.accept_from_logits(logits, drafts, q, u, modes)
    st.kv.restore(*st.state)
    if kind == "prefill":
        st.kv.prefill(0, st.prompts[0])
        dt = torch.bfloat16 if st.model.shape.kv_dtype == "bf16" else torch.float32
        return {"cache": st.kv.buf.view(dt), "lens": st.kv.lens, "pending": st.kv.pending}
    if kind == "ttft":
        st.kv.prefill_batch(st.prompts)
    spade.verify(st.model, st.kv, st.buf)
    out = {"logits": st.buf.logits, "n": st.buf.n, "correction": st.buf.corr}
    if kind == "draft":
        spade.softmax_into(st.buf.logits, st.probs)
        out["probs"] = st.probs
    st.kv.commit(st.buf.n, st.buf.corr)
    return {**out, "lens": st.kv.lens, "pending": st.kv.pending}


# --------------------------------------------------------------------------- work and tolerance

def work(case):
    s = _shape(case)
    B, G, V, d, f = case["batch"], case["gamma"], s.vocab, s.d_model, s.d_ffn
    elt = 2 if s.weight_dtype == "bf16" else 4
    dkv = s.kv_heads * s.head_dim
    sampled = sum(_modes(case))
    if case["kind"] == "accept":
        rows = B * (G + 1)
        return {"bytes": rows * V * 4 + sampled * V * 4, "flops": 5 * rows * V}
    kv_row = 2 * dkv * elt  # one position of one layer
    layer_w = 2 * d * d + 2 * d * dkv + 3 * d * f
    lens = _lens(case)
    nbytes = flops = 0
    if case["kind"] in ("prefill", "ttft"):
        T = sum(lens)
        pairs = sum(n * (n + 1) // 2 for n in lens)
        # the last layer is needed only up to its K and V
        nbytes += ((s.n_layers - 1) * layer_w + 2 * d * dkv) * elt + T * d * elt + s.n_layers * T * kv_row
        flops += 2 * T * ((s.n_layers - 1) * layer_w + 2 * d * dkv) + (s.n_layers - 1) * 4 * d * pairs
    if case["kind"] != "prefill":
        M = B * (G + 1)
        nbytes += (s.n_layers * layer_w + V * d) * elt + M * d * elt + M * V * 4
        nbytes += s.n_layers * (sum(lens) + M) * kv_row
        nbytes += sampled * V * 4 if G else 0
        flops += 2 * M * (s.n_layers * layer_w + V * d)
        flops += s.n_layers * 4 * d * sum((n + G + 1) * (G + 1) for n in lens)
    if case["kind"] == "draft":
        nbytes += 2 * V * 4
        flops += 4 * V
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times the distance from ``exact`` measured on an MI355X:
    5e-7 in float32; 5e-4 to 1e-3 for blocks of a bf16 model and 1.5e-3 to
    2.3e-3 over 32 layers, where the K and V that round to the other bf16
    neighbour (a few in a thousand under another order of the sums) make the
    difference."""
    if case["kind"] == "accept":
        return {"rel": 1e-5, "differ": 0.01}
    if case["model"] == "tiny":
        return {"rel": 2e-6, "max": 2e-5, "differ": 0.01}
    if case["layers"] > 8 or case["kind"] == "prefill":
        return {"rel": 0.01, "max": 0.1, "differ": 0.01}
    return {"rel": 0.004, "max": 0.04, "differ": 0.01}


# --------------------------------------------------------------------------- the same in 64 bits

def _rope(x, pos, theta):
    """Rotate-half RoPE of x [heads, T, hd] at positions pos."""
    hd = x.shape[-1]
    inv = theta ** (-torch.arange(0, hd, 2, dtype=torch.float64, device=x.device) / hd)
    a = pos.double()[:, None] * inv
    c, s = a.cos(), a.sin()
    x1, x2 = x[..., :hd // 2], x[..., hd // 2:]
    return torch.cat((x1 * c - x2 * s, x2 * c + x1 * s), -1)


def _forward64(s, seed, seqs, keep_rows):
    """float64 decoder over whole sequences.  Returns the logits of the last
    keep_rows rows of each ([B, keep_rows, V], None for 0) and each layer's
    stored (K, V) [KVH, T, hd] of each sequence.  K and V are rounded to the
    cache's type, which every attention read sees."""
    kvt = torch.bfloat16 if s.kv_dtype == "bf16" else torch.float32
    H, KVH, hd = s.n_heads, s.kv_heads, s.head_dim
    it = _weights(s, seed)
    E = next(it)[2]
    xs = [E[torch.as_tensor(t, device=DEV).long()].double() for t in seqs]
    del E

    def norm(x, g):
        return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + s.rms_eps) * g.double()

    stored = []
    for _ in range(s.n_layers):
        w = {}
        for _ in range(9):
            k, _, t = next(it)
            w[k] = t if k.startswith("g_") else t.double().t()
        layer = []
        for i, x in enumerate(xs):
            T = x.shape[0]
            pos = torch.arange(T, device=DEV)
            h = norm(x, w["g_attn"])
            q = _rope((h @ w["wq"]).view(T, H, hd).transpose(0, 1), pos, s.rope_theta)
            k = _rope((h @ w["wk"]).view(T, KVH, hd).transpose(0, 1), pos, s.rope_theta).to(kvt)
            v = (h @ w["wv"]).view(T, KVH, hd).transpose(0, 1).to(kvt)
            layer.append((k, v))
            mask = pos[None, :] > pos[:, None]
            o = torch.empty((T, H * hd), dtype=torch.float64, device=DEV)
            for kh in range(KVH):
                kd, vd = k[kh].double(), v[kh].double()
                for hh in range(kh * H // KVH, (kh + 1) * H // KVH):
                    a = (q[hh] @ kd.t()) / math.sqrt(hd)
                    a.masked_fill_(mask, -math.inf)
                    o[:, hh * hd:(hh + 1) * hd] = torch.softmax(a, -1) @ vd
            x = x + o @ w["wo"]
            h = norm(x, w["g_ffn"])
            xs[i] = x + (torch.nn.functional.silu(h @ w["wg"]) * (h @ w["wu"])) @ w["wd"]
        stored.append(layer)
    g_final, lm = next(it)[2], next(it)[2].double().t()
    logits = None
    if keep_rows:
        logits = torch.stack([norm(x[-keep_rows:], g_final) @ lm for x in xs])
    return logits, stored


def _gumbel(u, vocab):
    """-log(-log U_v), U_v from SplitMix64 seeded with the bits of float32 u."""
    with np.errstate(over="ignore"):
        z = np.uint64(np.float32(u).view(np.uint32)) + np.arange(1, vocab + 1, dtype=np.uint64) * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z = z ^ (z >> np.uint64(31))
    U = ((z >> np.uint64(41)).astype(np.float64) + 0.5) * 2.0 ** -23
    return torch.from_numpy(-np.log(-np.log(U))).to(DEV)


def _decide64(logits, drafts, q, u, modes):
    """n accepted and the correction of each request, from float64 logits."""
    B, R, V = logits.shape
    ns, cs = [], []
    for b in range(B):
        n = 0
        while n < R - 1:
            x = int(drafts[b][n])
            if modes[b] == 0:
                ok = int(logits[b, n].argmax()) == x
            else:
                ok = float(u[b][n]) * float(q[b, n, x]) < float(torch.softmax(logits[b, n], -1)[x])
            if not ok:
                break
            n += 1
        if modes[b] == 0:
            c = int(logits[b, n].argmax())
        else:
            w = torch.softmax(logits[b, n], -1)
            if n < R - 1:
                w = (w - q[b, n].double()).clamp_min(0.0)
            c = int((w.log() + _gumbel(float(u[b][R - 1]), V)).argmax())
        ns.append(n)
        cs.append(c)
    i32 = dict(dtype=torch.int32, device=DEV)
    return torch.tensor(ns, **i32), torch.tensor(cs, **i32)


def exact(case, seed):
    s = _shape(case)
    if case["kind"] == "accept":
        logits, drafts, q, u, modes = _logit_calls(case, s.vocab, seed)
        return _decide64(logits.double(), drafts.tolist(), q, u.tolist(), modes.tolist())
    lens = _lens(case)
    prompts = _prompts(case, s.vocab, seed)
    last = torch.tensor([int(p[-1]) for p in prompts], dtype=torch.int32, device=DEV)
    n0 = torch.tensor(lens, dtype=torch.int32, device=DEV)
    if case["kind"] == "prefill":
        _, stored = _forward64(s, seed, [prompts[0][:-1]], 0)
        S = (max(lens) + case["gamma"] + 2 + 255) // 256 * 256
        hd, KVH, T = s.head_dim, s.kv_heads, lens[0]
        kvt = stored[0][0][0].dtype
        parts = [[], []]
        for (kv,) in stored:
            for which in (0, 1):
                full = torch.zeros((KVH, S, hd), dtype=kvt, device=DEV)
                full[:, :T] = kv[which]
                if which == 0:  # fragments (16 positions, 32 features), pieces of 8 features
                    t = full.view(KVH, S // 256, 16, 16, hd // 32, 4, 8).permute(0, 1, 2, 4, 5, 3, 6)
                else:  # fragments (16 features, 32 positions), pieces of 8 positions
                    t = full.view(KVH, S // 256, 8, 4, 8, hd // 16, 16).permute(0, 1, 5, 2, 3, 6, 4)
                parts[which].append(t.reshape(-1))
        return {"cache": torch.cat(parts[0] + parts[1]), "lens": n0, "pending": last}
    drafts, q, u, modes = _calls(case, s.vocab, seed)
    seqs = [np.concatenate([p, drafts[b]]) for b, p in enumerate(prompts)]
    logits, _ = _forward64(s, seed, seqs, case["gamma"] + 1)
    n, c = _decide64(logits, drafts, q, u, modes)
    out = {"logits": logits, "n": n, "correction": c}
    if case["kind"] == "draft":
        out["probs"] = torch.softmax(logits, -1)
    return {**out, "lens": n0 + n + 1, "pending": c}
