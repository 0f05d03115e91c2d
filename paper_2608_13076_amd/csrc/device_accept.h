// Accept / reject and the correction draw for one request (Sec. III-C;
// Algorithm 1, the verify / accept / sample / correct steps), run by one
// workgroup of NT threads (COH: logits and LM-head statistics are read with
// sc1 loads, for a caller whose other workgroups wrote them in the same
// launch).
#pragma once

#include "device_util.h"

namespace spade {

struct AcceptParams {
  const float* logits;
  const float* stats;  // (max, sum exp, argmax) entries: NU per row, rows stat_stride floats apart; NULL: scan the logits
  int NU;
  int stat_stride;
  int given;           // the entries are row_stats_kernel's, of logits the caller computed
  int B, V, gamma, R;
  const int32_t* drafts;
  const float* q;
  const float* u;
  const uint8_t* mode;
  float inv_T;
  int32_t* n_out;
  int32_t* corr_out;
  uint32_t* err;
  // > 0: the correction draws of sampling requests are left to
  // correct_slices over this many vocabulary slices (accept_request stores
  // the log-sum-exp of the draw's row in corr_lse[b]); corr_part /
  // corr_cnt: per-slice winners and per-request arrival counters
  int corr_slices;
  float* corr_lse;
  float* corr_part;
  uint32_t* corr_cnt;
};

// SplitMix64 output v (0-based) of the stream seeded with `seed`.
__device__ __forceinline__ uint64_t splitmix64_at(uint64_t seed, uint64_t v) {
  uint64_t z = seed + (v + 1ull) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

__device__ __forceinline__ float gumbel_at(uint64_t seed, int v) {
  const uint64_t x = splitmix64_at(seed, (uint64_t)v);
  const float U = ((float)(uint32_t)(x >> 41) + 0.5f) * 0x1p-23f;
  return -logf(-logf(U));
}

struct Best {
  float s;
  int a;
};

__device__ __forceinline__ Best better(Best x, Best y) {
  if (y.s > x.s || (y.s == x.s && y.a < x.a)) return y;
  return x;
}

template <bool COH>
__device__ __forceinline__ float ld_any(const float* p) {
  if constexpr (COH) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else return *p;
}

// Gumbel-max scores of token v for the correction draw: the residual
// max(0, p - q) (log w + g, -inf where w <= 0) and p itself (z + g), with z
// the logit over the temperature and g the token's Gumbel noise.  No
// contraction, so every caller gets the same roundings.
__device__ __forceinline__ float corr_score_p(float logit, float invT, float g) {
#pragma clang fp contract(off)
  const float z = logit * invT;
  return z + g;
}

__device__ __forceinline__ float corr_score_res(float logit, float invT, float lse, float qv, float g) {
#pragma clang fp contract(off)
  const float z = logit * invT;
  const float w = expf(z - lse) - qv;
  return w > 0.f ? logf(w) + g : -INFINITY;
}

// Whether request b draws by sampling (else greedily); the accept step and
// the sliced correction decide it the same way.
__device__ __forceinline__ bool accept_samples(const AcceptParams& p, int b) {
  return p.mode[b] == SPADE_SAMPLE && p.u != nullptr && (p.gamma == 0 || p.q != nullptr);
}

// (max, sum exp, argmax) of z = logit / T over tokens [v0, v1) of a row, by
// NT threads (tid: the thread's number among them), 16 tokens per thread and
// step (16-byte loads where the row allows them): the step's maximum first,
// then one exponential per token.  NaN is skipped; ties keep the lower id.
// The thread's own part; wave_stat combines a wave's.
template <int NT, bool COH>
__device__ __forceinline__ RowStat scan_lane(const float* row, int v0, int v1, float invT, int tid) {
  const bool vec = !COH && ((size_t)(row + v0) & 15u) == 0u;
  RowStat st{-INFINITY, 0.f, 0x7fffffff};
  for (int base = v0; base < v1; base += NT * 16) {
    float z[16];
    int id0[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int v = base + (j * NT + tid) * 4;
      id0[j] = v;
      if (vec && v + 3 < v1) {
        const float4 x = *(const float4*)(row + v);
        z[4 * j] = x.x;
        z[4 * j + 1] = x.y;
        z[4 * j + 2] = x.z;
        z[4 * j + 3] = x.w;
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) z[4 * j + i] = v + i < v1 ? ld_any<COH>(row + v + i) : __uint_as_float(0x7fc00000u);
      }
    }
    float m = -INFINITY;
    int a = 0x7fffffff;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      z[k] *= invT;
      const int id = id0[k >> 2] + (k & 3);
      // (ids ascend, so an equal later one is never lower)
      if (z[k] > m || (z[k] == m && a == 0x7fffffff)) {
        m = z[k];
        a = id;
      }
    }
    float e = 0.f;
#pragma unroll
    for (int k = 0; k < 16; ++k) e += z[k] == m ? 1.f : (z[k] < m ? expf(z[k] - m) : 0.f);
    if (a != 0x7fffffff) st = merge_stat(st, RowStat{m, m == -INFINITY ? 1.f : e, a});
  }
  return st;
}

__device__ __forceinline__ RowStat wave_stat(RowStat st) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    RowStat o;
    o.m = __shfl_xor(st.m, off);
    o.s = __shfl_xor(st.s, off);
    o.a = __shfl_xor(st.a, off);
    st = (threadIdx.x & off) ? merge_stat(o, st) : merge_stat(st, o);
  }
  return st;
}

// Rows of at most this many tokens: a wave scans a row in steps of 1024, or,
// where the steps of all rows fit the workgroup's waves, a wave takes one step
// and the steps' lanes are merged in the same order, so a sampling call's
// log-sum-exp does not depend on gamma.
constexpr int kScanShort = 4096;

// A longer row is scanned in the accept workgroup only by greedy calls, whose
// results no order changes: pieces of at most 8192 tokens, at least one for
// every wave.  The rows one after the other, each by the whole workgroup (a
// round trip and a reduction per row), took 75 us for 16 requests of 16 rows
// of 1000 tokens and 79 for 5000 (greedy; now 11 and 23).
__device__ __forceinline__ int scan_pieces(int V, int R) {
  const int s = (V + 8191) / 8192, w = 16 / R;
  return min(16, s > w ? s : w);
}

// The skinny LM head's row statistics from the per-panel statistics of the
// other engines, by the 256 threads of a workgroup per row, in place (the
// row's first entry): its NU workgroup entries are rebuilt (workgroup q folds
// panels q, q + NU, ... in order; requested sixteen at a time and then folded,
// so the loads do not wait for one another) and merged as accept_request
// merges entries, so decisions do not depend on the engine.  Folded in the
// accept kernel, one workgroup per request, this took most of its 36 us for
// 16 requests of 9 rows and 8016 panels.
__device__ __forceinline__ void fold_panels(float* row, int panels, int NU, RowStat* ent) {
  constexpr int kBatch = 16;
  for (int q = threadIdx.x; q < NU; q += 256) {
    RowStat one{-INFINITY, 0.f, 0x7fffffff};
    for (int u0 = q; u0 < panels; u0 += kBatch * NU) {
      RowStat ps[kBatch];
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        const int u = u0 + j * NU;
        ps[j] = RowStat{-INFINITY, 0.f, 0x7fffffff};
        if (u < panels) ps[j] = RowStat{row[u * 3], row[u * 3 + 1], __float_as_int(row[u * 3 + 2])};
      }
#pragma unroll
      for (int j = 0; j < kBatch; ++j)
        if (ps[j].m != -INFINITY) one = merge_stat(one, ps[j]);
    }
    ent[q] = one;
  }
  __syncthreads();
  if (threadIdx.x >= 64) return;
  const int lane = threadIdx.x;
  RowStat st{-INFINITY, 0.f, 0x7fffffff};
  for (int q = lane; q < NU; q += 64)
    if (ent[q].m != -INFINITY) st = merge_stat(st, ent[q]);
  st = wave_stat(st);
  if (lane == 0) {
    row[0] = st.m;
    row[1] = st.s;
    row[2] = __int_as_float(st.a);
  }
}

struct AcceptSmem {
  RowStat scan[16][64];  // given logits only: per wave and lane, or per row and piece
  float rlse[kMaxR];
  int rarg[kMaxR];
  int x[kMaxR];                     // draft tokens (clamped)
  float lx[kMaxR], qx[kMaxR], ux[kMaxR];  // sampling: logit and q at the draft, its uniform
  Best bpart[16];
  int n_s;
};

template <int NT, bool COH>
__device__ __forceinline__ void accept_request(const AcceptParams& p, int b, AcceptSmem& sm) {
  constexpr int NWV = NT / 64;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int R = p.R, V = p.V, G = p.gamma;

  const bool sample = accept_samples(p, b);
  if (!sample && p.mode[b] == SPADE_SAMPLE && tid == 0) flag_error(p.err, SPADE_DERR_NOQ);
  const float invT = sample ? p.inv_T : 1.0f;
  const float* lg = p.logits + (size_t)b * R * V;

  // the drafts and what the accept chain reads for them, one thread per draft
  if (tid < G) {
    int x = p.drafts[(size_t)b * G + tid];
    if (x < 0 || x >= V) {
      flag_error(p.err, SPADE_DERR_TOKEN);
      x = x < 0 ? 0 : V - 1;
    }
    sm.x[tid] = x;
    if (sample) {
      sm.lx[tid] = ld_any<COH>(lg + (size_t)tid * V + x);
      sm.qx[tid] = p.q[((size_t)b * G + tid) * V + x];
      sm.ux[tid] = p.u[(size_t)b * (G + 1) + tid];
    }
  }

  // given logits of a short vocabulary or of a greedy-only call (which uses no
  // scratch; the others come with row_stats_kernel's slices)
  const int steps = (V + 1023) / 1024;
  const bool lanes = V <= kScanShort && R * steps <= NWV;
  const int pieces = V <= kScanShort ? 1 : scan_pieces(V, R);
  if (p.stats == nullptr && lanes) {
    if (wave < R * steps) {
      const int r = wave / steps, v0 = (wave - r * steps) * 1024;
      sm.scan[wave][lane] = scan_lane<64, COH>(lg + (size_t)r * V, v0, min(V, v0 + 1024), invT, lane);
    }
    __syncthreads();
  } else if (p.stats == nullptr) {
    const int per = ((V + pieces - 1) / pieces + 3) / 4 * 4;
    for (int i = wave; i < R * pieces; i += NWV) {
      const int r = i / pieces, v0 = (i - r * pieces) * per;
      const RowStat st = wave_stat(scan_lane<64, COH>(lg + (size_t)r * V, v0, min(V, v0 + per), invT, lane));
      if (lane == 0) sm.scan[r][i - r * pieces] = st;
    }
    __syncthreads();
  }

  // row statistics over the vocabulary: wave r merges row r from the LM
  // head's per-workgroup partials, from the slices of row_stats_kernel or
  // from the scan above, in a fixed order
  for (int r = wave; r < R; r += NWV) {
    RowStat st{-INFINITY, 0.f, 0x7fffffff};
    if (p.stats != nullptr) {
      const float* sp = p.stats + (size_t)(b * R + r) * p.stat_stride;
#pragma unroll 8
      for (int q = lane; q < p.NU; q += 64) {
        const RowStat one{ld_any<COH>(sp + q * 3), ld_any<COH>(sp + q * 3 + 1),
                          __float_as_int(ld_any<COH>(sp + q * 3 + 2))};
        // (given logits may be -inf throughout: the lowest id then)
        if (one.m != -INFINITY || p.given) st = merge_stat(st, one);
      }
    } else if (lanes) {
      for (int s = 0; s < steps; ++s) st = merge_stat(st, sm.scan[r * steps + s][lane]);
    } else if (lane < pieces) {
      st = sm.scan[r][lane];
    }
    if (p.stats != nullptr || lanes || pieces > 1) st = wave_stat(st);
    if (lane == 0) {
      sm.rlse[r] = st.m + logf(st.s);
      sm.rarg[r] = st.a;
    }
  }
  __syncthreads();

  if (tid == 0) {
    int n = G;
    for (int i = 0; i < G; ++i) {
      bool ok;
      if (!sample) {
        ok = (sm.x[i] == sm.rarg[i]);
      } else {
        const float px = expf(sm.lx[i] * invT - sm.rlse[i]);
        ok = sm.ux[i] * sm.qx[i] < px;
      }
      if (!ok) {
        n = i;
        break;
      }
    }
    sm.n_s = n;
  }
  __syncthreads();
  const int n = sm.n_s;
  int corr = 0;
  if (!sample) {
    corr = sm.rarg[n];
  } else if (p.corr_slices > 0) {
    // correct_slices draws it after this launch; its arrival counter starts
    // that launch at zero
    if (tid == 0) {
      p.corr_lse[b] = sm.rlse[n];
      p.n_out[b] = n;
      p.corr_cnt[b] = 0u;
    }
    return;
  } else {
    const uint64_t seed = (uint64_t)__float_as_uint(p.u[(size_t)b * (G + 1) + G]);
    const float* row = lg + (size_t)n * V;
    const bool residual = n < G;
    const float* qrow = residual ? p.q + ((size_t)b * G + n) * V : nullptr;
    const float lse = sm.rlse[n];
    for (int pass = 0; pass < 2; ++pass) {
      const bool use_res = residual && pass == 0;
      Best bst{-INFINITY, 0x7fffffff};
#pragma unroll 4
      for (int v = tid; v < V; v += NT) {
        const float lv = ld_any<COH>(row + v), g = gumbel_at(seed, v);
        const float sc = use_res ? corr_score_res(lv, invT, lse, qrow[v], g) : corr_score_p(lv, invT, g);
        if (sc != sc) continue;
        bst = better(bst, Best{sc, v});
      }
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) {
        const Best o{__shfl_xor(bst.s, off), __shfl_xor(bst.a, off)};
        bst = better(bst, o);
      }
      if (lane == 0) sm.bpart[wave] = bst;
      __syncthreads();
      Best t = sm.bpart[0];
      for (int w = 1; w < NWV; ++w) t = better(t, sm.bpart[w]);
      __syncthreads();
      if (t.s != -INFINITY || !use_res) {
        corr = t.a;
        break;
      }
      if (tid == 0) flag_error(p.err, SPADE_DERR_RESIDUAL);
    }
  }
  if (tid == 0) {
    p.n_out[b] = n;
    p.corr_out[b] = corr;
  }
}

__device__ __forceinline__ Best wave_best(Best x) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) x = better(x, Best{__shfl_xor(x.s, off), __shfl_xor(x.a, off)});
  return x;
}

// Slice s of corr_slices of the correction draw of a sampling request b,
// after accept_request (previous launch) stored n and the row's log-sum-exp:
// the best residual score and the best score under p over the slice's tokens
// (NaN scores skipped, as in the one-workgroup draw), published write-through;
// the last slice to arrive takes the best of all slices (the order of this
// maximum does not matter: ties go to the lower token id) and stores the
// correction, the residual's winner unless the residual had no mass.
// NT threads, one workgroup per (slice, request).
template <int NT>
__device__ __forceinline__ void correct_slice(const AcceptParams& p, int b, int s) {
  constexpr int NWV = NT / 64;
  __shared__ Best sres[NWV], sp[NWV];
  __shared__ int last;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  if (!accept_samples(p, b)) return;  // uniform
  const int V = p.V, G = p.gamma, S = p.corr_slices;
  const int n = p.n_out[b];
  const bool residual = n < G;
  const float invT = p.inv_T, lse = p.corr_lse[b];
  const uint64_t seed = (uint64_t)__float_as_uint(p.u[(size_t)b * (G + 1) + G]);
  const float* row = p.logits + ((size_t)b * (G + 1) + n) * V;
  const float* qrow = residual ? p.q + ((size_t)b * G + n) * V : nullptr;
  const int per = (V + S - 1) / S;
  const int v0 = s * per, v1 = min(V, v0 + per);
  Best br{-INFINITY, 0x7fffffff}, bp{-INFINITY, 0x7fffffff};
  // four tokens per thread and step: their logits and q requested first, the
  // noise (which needs neither) computed while they travel.  No load
  // is under a branch.
  // (16 rows of a 128K vocabulary: a loop of single loads took 23.0 us, this 19.8)
  const uint32_t bytes = (uint32_t)(v1 - v0) * 4u;
  const Rsrc rl = make_rsrc(row + v0, bytes), rq = make_rsrc(residual ? qrow + v0 : row, residual ? bytes : 0u);
  for (int base = v0; base < v1; base += 4 * NT) {
    float lv[4], qv[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t off = (uint32_t)(base - v0 + j * NT + tid) * 4u;  // past the slice: past the resource
      lv[j] = ld_f32<false>(rl, off);
      qv[j] = ld_f32<false>(rq, off);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int v = base + j * NT + tid;
      const float g = gumbel_at(seed, v);
      const float sc = corr_score_p(lv[j], invT, g);
      if (v < v1 && sc == sc) bp = better(bp, Best{sc, v});
      if (residual) {
        const float sr = corr_score_res(lv[j], invT, lse, qv[j], g);
        if (v < v1 && sr == sr) br = better(br, Best{sr, v});
      }
    }
  }
  br = wave_best(br);
  bp = wave_best(bp);
  if (lane == 0) {
    sres[wave] = br;
    sp[wave] = bp;
  }
  __syncthreads();
  const Rsrc rp = make_rsrc(p.corr_part, (uint32_t)(p.B * kCorrMaxSlices * 4 * 4));
  const uint32_t base = (uint32_t)((b * kCorrMaxSlices + s) * 4) * 4u;
  if (tid == 0) {
    for (int w = 1; w < NWV; ++w) {
      br = better(br, sres[w]);
      bp = better(bp, sp[w]);
    }
    st_f32<true>(rp, base, br.s);
    st_f32<true>(rp, base + 4u, __int_as_float(br.a));
    st_f32<true>(rp, base + 8u, bp.s);
    st_f32<true>(rp, base + 12u, __int_as_float(bp.a));
    __builtin_amdgcn_s_waitcnt(0);  // the winners have landed: arrive
    const uint32_t old = __hip_atomic_fetch_add(p.corr_cnt + b, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last = old == (uint32_t)S - 1u;
    if (last) __hip_atomic_store(p.corr_cnt + b, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (!last || wave != 0) return;
  Best r{-INFINITY, 0x7fffffff}, q{-INFINITY, 0x7fffffff};
  for (int i = lane; i < S; i += 64) {
    const uint32_t off = (uint32_t)((b * kCorrMaxSlices + i) * 4) * 4u;
    r = better(r, Best{ld_f32<true>(rp, off), __float_as_int(ld_f32<true>(rp, off + 4u))});
    q = better(q, Best{ld_f32<true>(rp, off + 8u), __float_as_int(ld_f32<true>(rp, off + 12u))});
  }
  r = wave_best(r);
  q = wave_best(q);
  if (lane == 0) {
    int corr = q.a;
    if (residual) {
      if (r.s != -INFINITY) corr = r.a;
      else flag_error(p.err, SPADE_DERR_RESIDUAL);
    }
    p.corr_out[b] = corr;
  }
}

}  // namespace spade
