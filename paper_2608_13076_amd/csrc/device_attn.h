// Verify attention for a bf16 cache with head_dim 128 (Sec. III-A: the
// gamma+1 appended rows of a request attend causally to its cached keys and
// to each other).
//
// Work item: (request, head, chunk of CK keys), one 8-wave workgroup.  Row i
// of the request sits at position L + i and sees keys <= L + i.  Scores
// S = Q K^T run with keys split over the waves (wave w: keys
// [k_lo + w CK/8, k_lo + (w+1) CK/8)); the chunk softmax runs one wave per
// row; O = P V runs with features split over the waves (wave w: features
// [16 w, 16 w + 16) over every key of the chunk), so each wave ends with
// final chunk outputs and no cross-wave sum is needed.  Both products use
// MFMA 16x16x32 bf16 with Q and P split into two bf16 terms (hi + lo).  K and
// V are stored in blocks of 256 positions in the order of the B operands of
// S = Q K^T and O = P V (k_cache_index, v_cache_index), so every B-operand
// fragment a wave loads is 1 KB contiguous.  A chunk writes its unnormalised output, row
// max and row sum; the chunks of a (request, head) are merged in chunk order
// with weights exp(m_c - max) / sum_c(l_c exp(m_c - max)).
#pragma once

#include "device_util.h"

namespace spade {

constexpr int kAttnRows = 16;  // rows per request (gamma + 1 <= 16)
constexpr int kAttnThreads = 512;

template <int CK>
struct AttnRegs {
  uint4 vf[CK / 32];      // [32-key step]: V^T row 16 w + kl, keys k_lo + 32 ks + 8 g .. + 8
};

struct AttnItem {
  bool active;
  int bl, h, c;
  int L;           // cached keys of the request (row i sits at L + i)
  int nc;          // chunks of the request
  int k_lo, k_hi;  // keys of this chunk: [k_lo, k_hi)
  const uint16_t* kc;  // K blocks of (request, head) (k_cache_index)
  const uint16_t* vc;  // V^T rows of (request, head)
};

// Item (request bl, head h, chunk c) of a request with L cached keys and R
// rows; chunks at or past the request's last key are inactive.
template <int CK>
__device__ __forceinline__ AttnItem attn_item(bool valid, int bl, int h, int c, int L, int R, const void* kc,
                                              const void* vc, size_t head_off) {
  AttnItem it;
  it.bl = bl;
  it.h = h;
  it.c = c;
  it.L = L;
  it.nc = (L + R + CK - 1) / CK;
  it.active = valid && c < it.nc;
  it.k_lo = c * CK;
  it.k_hi = it.active ? min(it.k_lo + CK, L + R) : it.k_lo;
  it.kc = (const uint16_t*)kc + head_off;
  it.vc = (const uint16_t*)vc + head_off;
  return it;
}

// Zero the V^T entries of keys at or past k_hi (their P is zero, but the
// cache may hold anything there).
template <int CK>
__device__ __forceinline__ void attn_mask_tail(const AttnItem& it, int lane, AttnRegs<CK>& r) {
  const int g = lane >> 4;
#pragma unroll
  for (int ks = 0; ks < CK / 32; ++ks) {
    const int kv0 = it.k_lo + 32 * ks + 8 * g;
    if (kv0 + 8 > it.k_hi) {
      uint32_t w[4] = {r.vf[ks].x, r.vf[ks].y, r.vf[ks].z, r.vf[ks].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int p0 = kv0 + 2 * e;
        if (p0 >= it.k_hi) w[e] = 0u;
        else if (p0 + 1 >= it.k_hi) w[e] &= 0xffffu;
      }
      r.vf[ks] = make_uint4(w[0], w[1], w[2], w[3]);
    }
  }
}

// f2bf without the NaN canonicalisation (the probabilities of a chunk are
// NaN only when its scores are, and then the outputs are NaN either way).
__device__ __forceinline__ uint16_t f2bf_num(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

__device__ __forceinline__ void attn_split2(const float* xs, uint4& hi, uint4& lo) {
  uint32_t hw[4], lw[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint16_t h0 = f2bf(xs[2 * e]), h1 = f2bf(xs[2 * e + 1]);
    const uint16_t l0 = f2bf(xs[2 * e] - bf2f(h0)), l1 = f2bf(xs[2 * e + 1] - bf2f(h1));
    hw[e] = (uint32_t)h0 | ((uint32_t)h1 << 16);
    lw[e] = (uint32_t)l0 | ((uint32_t)l1 << 16);
  }
  hi = make_uint4(hw[0], hw[1], hw[2], hw[3]);
  lo = make_uint4(lw[0], lw[1], lw[2], lw[3]);
}

// Queries staged in LDS as their two bf16 terms (rows of kAttnQPitch
// elements: 16-byte aligned, consecutive rows four banks apart).  Four
// consecutive features x of row `row` go in as attn_split2 splits them.
constexpr int kAttnQPitch = kAttnHd + 8;

__device__ __forceinline__ void attn_stage_q(uint16_t (*sqh)[kAttnQPitch], uint16_t (*sql)[kAttnQPitch], int row,
                                             int f, float4 x) {
  const float xs[4] = {x.x, x.y, x.z, x.w};
  uint32_t hw[2], lw[2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const uint16_t h0 = f2bf(xs[2 * e]), h1 = f2bf(xs[2 * e + 1]);
    const uint16_t l0 = f2bf(xs[2 * e] - bf2f(h0)), l1 = f2bf(xs[2 * e + 1] - bf2f(h1));
    hw[e] = (uint32_t)h0 | ((uint32_t)h1 << 16);
    lw[e] = (uint32_t)l0 | ((uint32_t)l1 << 16);
  }
  *(uint2*)&sqh[row][f] = make_uint2(hw[0], hw[1]);
  *(uint2*)&sql[row][f] = make_uint2(lw[0], lw[1]);
}

// lanes l, l ^ 16 (then ^ 32) combined in every lane
__device__ __forceinline__ float attn_add16(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float attn_add32(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float attn_max4(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(t[0]), __uint_as_float(t[1]));
}

// Quads q (this lane's four keys 4 g ..) of two 16-key groups, one register
// each, to octet order: lane group g gets keys 8 g .. + 3 in a, + 4 .. + 7 in
// b of the 32 keys.
__device__ __forceinline__ void attn_octet(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  const auto t = __builtin_amdgcn_permlane16_swap(r[0], r[1], false, false);
  a = t[0];
  b = t[1];
}

// One chunk of the verify attention for the NR rows of a workgroup, packed
// into T 16-row tiles: one query head's R rows (T = 1), or, for a
// grouped-query model, the G R rows of all query heads of a K/V head, so the
// chunk's keys and values pass through the compute unit once (packed row pr =
// gg R + i: query head gg of the group, request row i; rows past NR are
// masked).  Every packed row goes through the same instructions in the same
// order, so a row's partial does not depend on the packing.
//
// The K fragments come from attn_load_k, the queries from LDS (sqh / sql,
// their bf16 terms staged by the caller with attn_stage_q, rows past NR zero);
// the V^T fragments are requested only after the score products, into the
// registers the K fragments held, so a wave holds one of the two at a time.
//
// The products are transposed (S^T = K Q^T, each wave its 32 keys; O^T = V^T
// P^T, each wave its 16 features): a lane holds one query's scores, so the row
// maximum and sum reduce in-lane first (the adds of a butterfly over 16 keys),
// then over two lane swaps and the eight waves (LDS, in wave order), and the
// probabilities (exp2 of the log2(e)-scaled difference, as two bf16 terms)
// reach the second product's layout by lane swaps and one 16-byte LDS write
// per term.  With rows across registers, reduced over 16 lanes, and the
// probabilities written two bytes at a time, the grouped chunks took 55 us per
// layer (8B, 16 requests x 9 rows; now 51), one request at batch 1 11.1 (7B,
// 1030 keys; now 10.9); the multi-head batch is bound by HBM (7B, 16 requests:
// 105 us either way).
//
// o[t]: packed row 16 t + kl, features 16 wave + 4 g + i (i = 0..3).
template <int CK, int T>
struct AttnSmem {
  // probabilities as two bf16 terms (the operand of O^T = V^T P^T); rows padded
  // by 16 bytes so the 16 rows of a fragment read start in different banks
  alignas(16) uint16_t ph[16 * T][CK + 8];
  alignas(16) uint16_t pl[16 * T][CK + 8];
  float pm[16 * T][8], ps[16 * T][8];  // per-wave row max / row sum
  float m[16 * T], l[16 * T];
};

template <int CK>
__device__ __forceinline__ void attn_load_k(const AttnItem& it, int wave, int lane, uint4 (&kf)[CK / 128][4]) {
  const int g = lane >> 4, kl = lane & 15;
#pragma unroll
  for (int grp = 0; grp < CK / 128; ++grp) {
    const int key = it.k_lo + (CK / 8) * wave + 16 * grp + kl;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) kf[grp][ks] = make_uint4(0, 0, 0, 0);
    if (key < it.k_hi) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) kf[grp][ks] = ld_stream_g128(it.kc + k_cache_index(32 * ks + 8 * g, key, kAttnHd));
    }
  }
}

// Query head within the group (gg) and request row (rw) of packed rows
// p0 + 16 t + i (t < T, i < NI), p0 + 16 t + i = gg R + rw: two divisions,
// then steps (a division per row costs some twenty VALU instructions).
template <int T, int NI>
__device__ __forceinline__ void attn_grp_rows(int p0, int R, int (&gg)[T][NI], int (&rw)[T][NI]) {
  const int sq = 16 / R, sr = 16 - sq * R;
  int q = p0 / R, r = p0 - q * R;
#pragma unroll
  for (int t = 0; t < T; ++t) {
    int qi = q, ri = r;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      gg[t][i] = qi;
      rw[t][i] = ri;
      if (++ri == R) {
        ri = 0;
        ++qi;
      }
    }
    r += sr;
    q += sq;
    if (r >= R) {
      r -= R;
      ++q;
    }
  }
}

template <int CK, int T>
__device__ __forceinline__ void attn_chunk(const AttnItem& it, const uint4 (&kf)[CK / 128][4],
                                           const uint16_t (*sqh)[kAttnQPitch], const uint16_t (*sql)[kAttnQPitch],
                                           int R, int NR, float scale, AttnSmem<CK, T>& sm, floatx4 (&o)[T]) {
  static_assert(CK == 256, "32 keys per wave");
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int g = lane >> 4, kl = lane & 15;
  const int ke = (it.k_hi + 7) & ~7;
  int gg[T][1], rw[T][1];  // request row of packed row 16 t + kl
  if constexpr (T > 1) attn_grp_rows<T, 1>(kl, R, gg, rw);
  else rw[0][0] = R == NR ? kl : kl % R;
  float sv[T][2][4];  // key k_lo + 32 wave + 16 grp + 4 g + i
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const bool ok = 16 * t + kl < NR;
    const int last = min(it.k_hi - 1, it.L + rw[t][0]);  // the row's last key of the chunk
#pragma unroll
    for (int grp = 0; grp < 2; ++grp) {
      floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const uint4 qh = *(const uint4*)&sqh[16 * t + kl][32 * ks + 8 * g];
        const uint4 ql = *(const uint4*)&sql[16 * t + kl][32 * ks + 8 * g];
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[grp][ks]),
                                                      __builtin_bit_cast(bf16x8, ql), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[grp][ks]),
                                                      __builtin_bit_cast(bf16x8, qh), acc, 0, 0, 0);
      }
      const int key = it.k_lo + 32 * wave + 16 * grp + 4 * g;
#pragma unroll
      for (int i = 0; i < 4; ++i) sv[t][grp][i] = (ok && key + i <= last) ? acc[i] * scale : -INFINITY;
    }
  }
  // the V^T fragments, after the score products (the K registers are free);
  // fragment (wave, 32-key step ks) of the chunk's V block is 512 elements
  // after step ks - 1's
  __builtin_amdgcn_sched_barrier(0);
  AttnRegs<CK> r;
  const uint16_t* vfr = it.vc + v_cache_index(16 * wave + kl, it.k_lo + 8 * g, kAttnHd);
#pragma unroll
  for (int ks = 0; ks < CK / 32; ++ks) {
    const int kv0 = it.k_lo + 32 * ks + 8 * g;
    r.vf[ks] = make_uint4(0, 0, 0, 0);
    if (kv0 + 8 <= ke) r.vf[ks] = ld_stream_g128(vfr + ks * 512);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int t = 0; t < T; ++t) {
    float mx = sv[t][0][0];
#pragma unroll
    for (int grp = 0; grp < 2; ++grp)
#pragma unroll
      for (int i = 0; i < 4; ++i) mx = fmaxf(mx, sv[t][grp][i]);
    mx = attn_max4(mx);
    if (g == 0) sm.pm[16 * t + kl][wave] = mx;
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int row = 16 * t + kl;
    const float4 a = *(const float4*)&sm.pm[row][0];
    const float4 b = *(const float4*)&sm.pm[row][4];
    const float M = fmaxf(fmaxf(fmaxf(a.x, a.y), fmaxf(a.z, a.w)), fmaxf(fmaxf(b.x, b.y), fmaxf(b.z, b.w)));
    float e[2][4];
    uint32_t hw[2][2], lw[2][2];
#pragma unroll
    for (int grp = 0; grp < 2; ++grp) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        e[grp][i] = (M == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f((sv[t][grp][i] - M) * 1.44269504088896341f);
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const float p0 = e[grp][2 * x], p1 = e[grp][2 * x + 1];
        const uint16_t h0 = f2bf_num(p0), h1 = f2bf_num(p1);
        hw[grp][x] = (uint32_t)h0 | ((uint32_t)h1 << 16);
        lw[grp][x] = (uint32_t)f2bf_num(p0 - bf2f(h0)) | ((uint32_t)f2bf_num(p1 - bf2f(h1)) << 16);
      }
    }
    float sum = (e[0][0] + e[1][0]) + (e[0][1] + e[1][1]);
    sum += (e[0][2] + e[1][2]) + (e[0][3] + e[1][3]);
    sum = attn_add32(attn_add16(sum));
    if (g == 0) sm.ps[row][wave] = sum;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      attn_octet(hw[0][x], hw[1][x]);
      attn_octet(lw[0][x], lw[1][x]);
    }
    *(uint4*)&sm.ph[row][32 * wave + 8 * g] = make_uint4(hw[0][0], hw[0][1], hw[1][0], hw[1][1]);
    *(uint4*)&sm.pl[row][32 * wave + 8 * g] = make_uint4(lw[0][0], lw[0][1], lw[1][0], lw[1][1]);
  }
  __syncthreads();
  if (tid < NR) {
    float l = 0.f, M = -INFINITY;
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      l += sm.ps[tid][w];
      M = fmaxf(M, sm.pm[tid][w]);
    }
    sm.m[tid] = M;
    sm.l[tid] = l;
  }
  attn_mask_tail(it, lane, r);
#pragma unroll
  for (int t = 0; t < T; ++t) {
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < CK / 32; ++ks) {
      const uint4 ph = *(const uint4*)&sm.ph[16 * t + kl][32 * ks + 8 * g];
      const uint4 pl = *(const uint4*)&sm.pl[16 * t + kl][32 * ks + 8 * g];
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, r.vf[ks]),
                                                    __builtin_bit_cast(bf16x8, pl), acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, r.vf[ks]),
                                                    __builtin_bit_cast(bf16x8, ph), acc, 0, 0, 0);
    }
    o[t] = acc;
  }
}

// Last-arrival merge of the chunks of one (request, head).
struct AttnMergeSmem {
  float sc[kAttnMaxChunks][kAttnRows];  // merge weights
  int last;
};

// partials of output o (= row * kAttnHd + dd) for chunks c0 .. c0 + 15
// (COH: sc1 loads; chunks past nc and ok == false read 0)
template <bool COH>
__device__ __forceinline__ void attn_load16(Rsrc rpo, int c0, int nc, int Rmax, int o, bool ok, float (&v)[16]) {
  const int row = o / kAttnHd, dd = o - row * kAttnHd;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const int c = c0 + j;
    v[j] = ld_f32<COH>(rpo, (ok && c < nc) ? (uint32_t)((c * Rmax + row) * kAttnHd + dd) * 4u : kOob);
  }
}

// One chunk's term of a merged output: O + w v (a zero weight adds zero
// whatever v holds), rounded after the product and after the sum, never
// fused, so every merge gives the same bits.
__device__ __forceinline__ float attn_acc1(float O, float v, float w) {
#pragma clang fp contract(off)
  return O + (w != 0.f ? v * w : 0.f);
}

// add chunks c0 .. c0 + 15 of output o to O, in chunk order
__device__ __forceinline__ void attn_acc16(const AttnMergeSmem& ms, int c0, int nc, int o, const float (&v)[16],
                                           float& O) {
  const int row = o / kAttnHd;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const int c = c0 + j;
    if (c < nc) O = attn_acc1(O, v[j], ms.sc[c][row]);
  }
}

// merged outputs oa and oa + 512 (each where < nout); va / vb hold their
// chunks 0..15 on entry
template <bool COH, class Out>
__device__ __forceinline__ void attn_merge_pair(Rsrc rpo, const AttnMergeSmem& ms, int nc, int Rmax, int nout,
                                                int oa, float (&va)[16], float (&vb)[16], Out&& out) {
  const int ob = oa + 512;
  float Oa = 0.f, Ob = 0.f;
  attn_acc16(ms, 0, nc, oa, va, Oa);
  attn_acc16(ms, 0, nc, ob, vb, Ob);
  for (int c0 = 16; c0 < nc; c0 += 16) {
    attn_load16<COH>(rpo, c0, nc, Rmax, oa, oa < nout, va);
    attn_load16<COH>(rpo, c0, nc, Rmax, ob, ob < nout, vb);
    attn_acc16(ms, c0, nc, oa, va, Oa);
    attn_acc16(ms, c0, nc, ob, vb, Ob);
  }
  if (oa < nout) out(oa, Oa);
  if (ob < nout) out(ob, Ob);
}

// Store the chunk's partials (o: attn_chunk's result; m / l from sa) with
// write-through stores, without waiting for them: packed row pr of the rows of
// query heads h0 .. (R rows each) goes to head h0 + pr / R, row pr % R.
// part_o / part_ml: [bh][NC][Rmax][kAttnHd] / [bh][NC][Rmax][2].  All 512
// threads call it.
template <int CK, int T>
__device__ __forceinline__ void attn_publish(const AttnItem& it, int h0, const floatx4 (&o)[T], const AttnSmem<CK, T>& sa,
                                             float* part_o, float* part_ml, int H, int NC, int Rmax, int R, int NR) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int g = lane >> 4, kl = lane & 15;
  const size_t bh0 = (size_t)it.bl * H + h0;
  const Rsrc rpo = wave_rsrc(part_o + bh0 * NC * Rmax * kAttnHd);
  int gq[T][1], rw[T][1];
  if constexpr (T > 1) attn_grp_rows<T, 1>(kl, R, gq, rw);
  else {
    gq[0][0] = R == NR ? 0 : kl / R;
    rw[0][0] = kl - gq[0][0] * R;
  }
  typedef uint32_t u32x4a __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const uint32_t off = (uint32_t)(((gq[t][0] * NC + it.c) * Rmax + rw[t][0]) * kAttnHd + 16 * wave + 4 * g) * 4u;
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4a, o[t]), rpo, (int)(16 * t + kl < NR ? off : kOob), 0,
                                           kAuxCoh);
  }
  if (tid < NR) {
    const int gg = tid / R, row = tid - gg * R;
    float* pml = part_ml + (((bh0 + gg) * NC + it.c) * Rmax + row) * 2;
    __hip_atomic_store(pml, sa.m[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(pml + 1, sa.l[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Merge weights of one row's nc chunks, by one wave (chunk c on lane c % 64,
// slot c / 64): w_c = exp(m_c - max) / sum_c(l_c exp(m_c - max)), the sum
// taken per lane in slot order and then across the lanes by butterfly.
// ml(c, ok, m, l) fetches chunk c's row max and row sum (ok false: no such
// chunk, values unused); put(c, w) receives each weight after every fetch.
template <class ML, class PUT>
__device__ __forceinline__ void attn_row_weights(int nc, ML&& ml, PUT&& put) {
  const int lane = threadIdx.x & 63;
  constexpr int NJ = kAttnMaxChunks / 64;
  float mc[NJ], lc[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int c = lane + 64 * j;
    const bool ok = c < nc;
    float m, l;
    ml(c, ok, m, l);
    mc[j] = ok ? m : -INFINITY;
    lc[j] = l;
  }
  float Mx = -INFINITY;
#pragma unroll
  for (int j = 0; j < NJ; ++j) Mx = fmaxf(Mx, mc[j]);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) Mx = fmaxf(Mx, __shfl_xor(Mx, off));
  float Ls = 0.f;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    mc[j] = (mc[j] == -INFINITY) ? 0.f : expf(mc[j] - Mx);
    Ls += lc[j] * mc[j];
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) Ls += __shfl_xor(Ls, off);
  const float inv = 1.0f / Ls;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int c = lane + 64 * j;
    if (c < nc) put(c, mc[j] * inv);
  }
}

// Merge weights of the nc chunks of R rows into ms.sc (attn_row_weights, one
// wave per row: rows wave and wave + 8); ml(c, row, ok, m, l) as there.  All
// 512 threads call it; the caller synchronises before reading ms.sc.
template <class ML>
__device__ __forceinline__ void attn_merge_weights(AttnMergeSmem& ms, int nc, int R, ML&& ml) {
  const int wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int row = wave + 8 * k;
    if (row < R)  // uniform across the wave
      attn_row_weights(
          nc, [&](int c, bool ok, float& m, float& l) { ml(c, row, ok, m, l); },
          [&](int c, float w) { ms.sc[c][row] = w; });
  }
}

// Merge the nc chunk partials of (request, head) bh in chunk order and pass
// each merged output o = row * kAttnHd + dd to out(o, value).  Merge weights
// of a row: one wave, chunks over its lanes; the weight of chunk c is
// exp(m_c - max) / sum_c(l_c exp(m_c - max)).  All 512 threads call it.
template <bool COH, class Out>
__device__ __forceinline__ void attn_merge(size_t bh, int nc, AttnMergeSmem& ms, float* part_o, float* part_ml,
                                           int NC, int Rmax, int R, Out&& out) {
  const int tid = threadIdx.x;
  // this thread's first partials, and the (m, l) pairs of the wave's rows
  // (wave and wave + 8: R <= 16), in one round trip
  const Rsrc rpo = wave_rsrc(part_o + (bh * NC * Rmax) * kAttnHd);
  const Rsrc rpm = wave_rsrc(part_ml + (bh * NC * Rmax) * 2);
  const int nout = R * kAttnHd;
  float va[16], vb[16];
  attn_load16<COH>(rpo, 0, nc, Rmax, tid, tid < nout, va);
  attn_load16<COH>(rpo, 0, nc, Rmax, tid + 512, tid + 512 < nout, vb);
  attn_merge_weights(ms, nc, R, [&](int c, int row, bool ok, float& m, float& l) {
    const uint32_t off = ok ? (uint32_t)((c * Rmax + row) * 2) * 4u : kOob;
    m = ld_f32<COH>(rpm, off);
    l = ld_f32<COH>(rpm, off == kOob ? kOob : off + 4u);
  });
  __syncthreads();
  attn_merge_pair<COH>(rpo, ms, nc, Rmax, nout, tid, va, vb, out);
  for (int oa = tid + 1024; oa < nout; oa += 1024) {
    attn_load16<COH>(rpo, 0, nc, Rmax, oa, true, va);
    attn_load16<COH>(rpo, 0, nc, Rmax, oa + 512, oa + 512 < nout, vb);
    attn_merge_pair<COH>(rpo, ms, nc, Rmax, nout, oa, va, vb, out);
  }
}

// Once this workgroup's published partials (n_mine chunks of the (request,
// head) of it) have landed, arrive on the counter of that (request, head)
// with n_mine, and, in the workgroup whose arrival completes the request's
// chunks, merge them and pass each merged output o = row * kAttnHd + dd to
// out(o, value).  The completing arrival resets the counter.  All 512 threads
// call it.  COH: read the partials with sc1 loads; without it they are read
// with plain loads, which is enough within one launch (no workgroup of the
// launch reads a partial before its write-through store has landed, and the
// launch starts with the L2 invalidated).
template <bool COH = true, class Out>
__device__ __forceinline__ void attn_arrive_merge(const AttnItem& it, int n_mine, AttnMergeSmem& ms, float* part_o,
                                                  float* part_ml, uint32_t* attn_cnt, int H, int NC, int Rmax, int R,
                                                  Out&& out) {
  const int tid = threadIdx.x;
  const size_t bh = (size_t)it.bl * H + it.h;
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (tid == 0) {
    int last = 0;
    if (n_mine > 0) {
      uint32_t* cnt = attn_cnt + bh;
      const uint32_t old = __hip_atomic_fetch_add(cnt, (uint32_t)n_mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (old + (uint32_t)n_mine == (uint32_t)it.nc) {
        __hip_atomic_store(cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = 1;
      }
    }
    ms.last = last;
  }
  __syncthreads();
  if (!ms.last) return;  // uniform across the workgroup
  attn_merge<COH>(bh, it.nc, ms, part_o, part_ml, NC, Rmax, R, out);
}

// attn_publish and attn_arrive_merge for a workgroup that computed the one
// chunk it.
template <int CK, bool COH = true, class Out>
__device__ __forceinline__ void attn_publish_merge(const AttnItem& it, const floatx4 (&o)[1], const AttnSmem<CK, 1>& sa,
                                                   AttnMergeSmem& ms, float* part_o, float* part_ml,
                                                   uint32_t* attn_cnt, int H, int NC, int Rmax, int R, Out&& out) {
  attn_publish<CK, 1>(it, it.h, o, sa, part_o, part_ml, H, NC, Rmax, R, R);
  attn_arrive_merge<COH>(it, it.active ? 1 : 0, ms, part_o, part_ml, attn_cnt, H, NC, Rmax, R, out);
}

// ---------------------------------------------------------------------------
// Prefill attention: R prompt rows of a request (R > 16), appended at
// positions L .. L + R - 1, each attending causally to the cache and the
// rows before it.  The rows form 16-row tiles; tile t is computed as a verify
// call of its own (L + 16 t cached keys, up to 16 rows), operation for
// operation, so each row gets the verify path's result bit for bit: the same
// 256-key chunks, the same scores (the query's two bf16 terms against 16 keys
// per MFMA output tile, four 32-feature steps each), the same chunk softmax
// (row max and row sum over each 32-key slice, then over the eight slices in
// order), the same probabilities' two bf16 terms against V^T in 32-key steps,
// the same merge weights (attn_row_weights) and the same chunk-order sum
// (attn_acc1).  A row's result does not depend on which other rows share its
// tile: every product and reduction of a chunk is per row, and chunks past a
// row's position get weight zero.
//
// Where the verify kernel spreads one chunk over eight waves, here one wave
// runs a whole tile: the eight 32-key slices of a chunk one after another,
// with no barrier between them.  The W waves of a workgroup take W
// consecutive tiles of one (request, head) and share every K and V block: 64
// keys (16 KB) at a time through an LDS ring of NS slots, filled by direct
// buffer->LDS loads NS - 1 blocks ahead.  The cache holds K and V in MFMA
// fragment order, so a block is 16 contiguous 1 KB fragments and a fragment
// read is one conflict-free ds_read_b128; the ring is read with inline asm and
// explicit waits (the compiler would wait for every fill in flight).
//
// The products are computed transposed (S^T = K Q^T, O^T = V^T P^T: the same
// products summed over the same k order, so the same bits): a lane then holds
// one query's column, the row maximum and sum are mostly in-lane (the adds of
// the verify kernel's butterfly, two of the four steps across lanes), and the
// probabilities reach the second product's operand layout by two lane swaps
// per register instead of through LDS.
//
// Each chunk is walked twice: the first walk keeps every chunk's row max and
// row sum in LDS, the merge weights follow from them, and the second walk
// recomputes the probabilities (the chunk's maximum known) block by block,
// multiplies them with V and adds each chunk's result, times its weight, to
// the tile's running sums in registers.
//
// What bounds it: the longest tile's chain of blocks for one prompt, VALU
// (masks, exponentials, bf16 terms) and MFMA about evenly for many.  Staging
// through registers with two slots, a barrier and a load's latency per block
// and the probabilities through LDS took 99 us per layer for 1018 rows of 32
// heads (253 for 2048 rows after up to 2048 more); this takes 52 (170).
// ---------------------------------------------------------------------------
constexpr int kPfBlock = 16384;  // bytes of a 64-key block of K or V

// Dynamic LDS: the ring, then per wave, chunk and row a pair: the chunk's row
// max and row sum, later max and merge weight.
__host__ __device__ inline unsigned attn_prefill_dyn_bytes(int W, int NS, int NC) {
  return (unsigned)NS * kPfBlock + (unsigned)W * NC * 16 * 8;
}

typedef uint32_t u32x4p __attribute__((ext_vector_type(4)));

template <int F>
__device__ __forceinline__ u32x4p pf_read(uint32_t addr) {
  u32x4p v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(F * 1024));
  return v;
}

// wait until at most N of the wave's LDS reads are outstanding; the eight
// fragments depend on the wait
template <int N>
__device__ __forceinline__ void pf_wait(u32x4p (&x)[8]) {
  asm volatile("s_waitcnt lgkmcnt(%8)"
               : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(x[4]), "+v"(x[5]), "+v"(x[6]), "+v"(x[7])
               : "n"(N));
}

// Wave-local ordering of LDS traffic between the lanes of one wave.
__device__ __forceinline__ void pf_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// q: this request's query rows ([R][d], head h's features at h * kAttnHd);
// rk / rv: the K and V blocks of (request, K/V head), kv_stride positions; L:
// the request's cached keys; t0: the group's first tile (tile t0 + wave for
// this wave).  out4(row, dd, v) receives outputs dd .. dd + 3 of a row (counted
// from the request's first prompt row).  lds: the ring, then W * NCP * 16
// pairs; NCP bounds the chunks of any tile.  All 64 W threads call it.
template <int W, int NS, class Out>
__device__ __forceinline__ void attn_prefill_tiles(uint8_t* lds, int NCP, const float* q, int d, int h, Rsrc rk,
                                                   Rsrc rv, int L, int R, int t0, float scale, Out&& out4) {
  static_assert(W == 4, "a wave moves four of a block's 16 fragments");
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int g = lane >> 4, kl = lane & 15;
  const int ntile = (R + 15) / 16;
  const int tl = t0 + wave;                            // this wave's tile
  const int Rt = tl < ntile ? min(16, R - 16 * tl) : 0;  // its rows (0: idle)
  const int Lt = L + 16 * tl;
  const int end = Rt > 0 ? Lt + Rt : 0;                // its keys
  // the group's furthest key: the end of its last tile
  const int tlast = min(t0 + W, ntile) - 1;
  const int kend = L + 16 * tlast + min(16, R - 16 * tlast);
  const int nk = (kend + 63) / 64;                     // 64-key blocks
  float2* ml = (float2*)(lds + NS * kPfBlock) + (size_t)wave * NCP * 16;
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) void*)lds;
  const uint32_t frag = lds0 + (uint32_t)lane * 16u;
  const uint32_t mla = lds0 + (uint32_t)(NS * kPfBlock) + (uint32_t)(wave * NCP * 16 + kl) * 8u;  // this lane's query

  // this lane's query fragments (row kl of the tile, features 32 ks + 8 g ..),
  // as two bf16 terms; rows past the tile: zeros
  uint4 qh[4], ql[4];
  {
    const bool ok = kl < Rt;
    const float* qr = q + (size_t)(16 * tl + kl) * d + h * kAttnHd;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = 0.f;
      if (ok) {
        const float4 a = *(const float4*)(qr + 32 * ks + 8 * g), b = *(const float4*)(qr + 32 * ks + 8 * g + 4);
        x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w; x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
      }
      attn_split2(x, qh[ks], ql[ks]);
    }
  }

  // The block stream: nk K blocks (first walk), then K and V of each block in
  // turn (second walk).  Block t goes to slot t % NS; wave w moves fragments
  // 4 w .. + 3 (of V: feature tiles 2 w, 2 w + 1 at the block's two 32-key
  // steps).  Blocks past the stream read zeros.
  const int nt = 3 * nk;
  auto fill = [&](int t) {
    const bool first = t < nk;
    const int r = t - nk, kb = first ? t : r >> 1;
    const bool is_v = !first && (r & 1);
    uint32_t off[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int f = 4 * wave + i;
      const uint32_t at = is_v ? (uint32_t)((kb >> 2) * 65536 + (f >> 1) * 8192 + ((kb & 3) * 2 + (f & 1)) * 1024)
                               : (uint32_t)(kb * kPfBlock + f * 1024);
      off[i] = t < nt ? at + (uint32_t)lane * 16u : kOob;
    }
    __attribute__((address_space(3))) uint8_t* dst =
        (__attribute__((address_space(3))) uint8_t*)(lds + (t % NS) * kPfBlock + 4 * wave * 1024);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (is_v) __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, (__attribute__((address_space(3))) void*)(dst + i * 1024), 16, off[i], 0, 0, 0);
      else __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, (__attribute__((address_space(3))) void*)(dst + i * 1024), 16, off[i], 0, 0, 0);
    }
  };
  // Block t: this wave's share has landed (the NS - 2 blocks after it have
  // four loads each), every wave's after the barrier, which also ends every
  // wave's reads of block t - 1; block t + NS - 1 goes into its slot.
  auto step = [&](int t) {
    wait_vmcnt<(NS - 2) * 4>();
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    fill(t + NS - 1);
    __builtin_amdgcn_sched_barrier(0);
  };

  // scaled, masked scores of the K block kb in slot t % NS: sv[u][i] of this
  // lane's query with key 64 kb + 16 u + 4 g + i
  auto scores = [&](int t, int kb, float (&sv)[4][4]) {
    const uint32_t base = frag + (uint32_t)(t % NS) * (uint32_t)kPfBlock;
    u32x4p xa[8], xb[8];  // features 32 ks ..: ks = 0, 1 of the four groups, then 2, 3
    xa[0] = pf_read<0>(base);
    xa[1] = pf_read<4>(base);
    xa[2] = pf_read<8>(base);
    xa[3] = pf_read<12>(base);
    xa[4] = pf_read<1>(base);
    xa[5] = pf_read<5>(base);
    xa[6] = pf_read<9>(base);
    xa[7] = pf_read<13>(base);
    xb[0] = pf_read<2>(base);
    xb[1] = pf_read<6>(base);
    xb[2] = pf_read<10>(base);
    xb[3] = pf_read<14>(base);
    xb[4] = pf_read<3>(base);
    xb[5] = pf_read<7>(base);
    xb[6] = pf_read<11>(base);
    xb[7] = pf_read<15>(base);
    floatx4 acc[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[u] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto mul = [&](const u32x4p (&x)[8], int ks0) {
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int term = 0; term < 2; ++term)
#pragma unroll
          for (int u = 0; u < 4; ++u)
            acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, x[4 * k + u]),
                __builtin_bit_cast(bf16x8, term ? qh[ks0 + k] : ql[ks0 + k]), acc[u], 0, 0, 0);
    };
    pf_wait<8>(xa);
    mul(xa, 0);
    __builtin_amdgcn_sched_barrier(0);
    pf_wait<0>(xb);
    mul(xb, 2);
    const int k0 = 64 * kb + 4 * g;
    if (64 * kb + 64 > Lt) {  // keys some row of the tile does not see
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int key = k0 + 16 * u + i;
          sv[u][i] = (key < end && key <= Lt + kl) ? acc[u][i] * scale : -INFINITY;
        }
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma clang fp contract(off)
          sv[u][i] = acc[u][i] * scale;
        }
    }
  };
  auto prob = [](float sv, float M) {
#pragma clang fp contract(off)
    return __builtin_amdgcn_exp2f((sv - M) * 1.44269504088896341f);
  };

#pragma unroll
  for (int t = 0; t < NS - 1; ++t) fill(t);
  // first walk: every chunk's row max and row sum
  for (int c = 0; 4 * c < nk; ++c) {
    float sv[4][4][4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int kb = 4 * c + b;
      if (kb >= nk) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i) sv[b][u][i] = -INFINITY;
        continue;
      }
      step(kb);
      if (64 * kb < end) {
        scores(kb, kb, sv[b]);
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i) sv[b][u][i] = -INFINITY;
      }
    }
    if (256 * c < end) {
      float M = sv[0][0][0];  // (NaN only if every score is)
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i) M = fmaxf(M, sv[b][u][i]);
      M = attn_max4(M);
      const float Mz = M == -INFINITY ? 0.f : M;  // an empty chunk: every probability exp2(-inf) = 0
      float lsum = 0.f;
#pragma unroll
      for (int vw = 0; vw < 8; ++vw) {  // 32-key slices, each in the verify kernel's order
        float e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          e[i] = prob(sv[vw >> 1][2 * (vw & 1)][i], Mz) + prob(sv[vw >> 1][2 * (vw & 1) + 1][i], Mz);
        lsum += attn_add32(attn_add16((e[0] + e[1]) + (e[2] + e[3])));
      }
      if (M == -INFINITY) lsum = 0.f;
      if (g == 0) {
        const uint64_t v = (uint64_t)__float_as_uint(fmaxf(-INFINITY, M)) | ((uint64_t)__float_as_uint(lsum) << 32);
        asm volatile("ds_write_b64 %0, %1" ::"v"(mla + (uint32_t)c * 128u), "v"(v) : "memory");
      }
    }
  }
  // merge weights of this wave's rows, in place of the row sums
  const int nct = (end + 255) / 256;
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  pf_wave_sync();
  if (nct <= 16) {
    // attn_row_weights for this lane's row: the same terms, the adds of its
    // butterfly over lanes (chunk c in lane c)
#pragma clang fp contract(off)
    float m[16], t[16], Mx = -INFINITY;
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      const float2 v = c < nct ? ml[c * 16 + kl] : make_float2(-INFINITY, 0.f);
      m[c] = v.x;
      t[c] = v.y;
      Mx = fmaxf(Mx, m[c]);
    }
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      m[c] = m[c] == -INFINITY ? 0.f : expf(m[c] - Mx);
      t[c] = t[c] * m[c];
    }
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1)
#pragma unroll
      for (int c = 0; c < off; ++c) t[c] = t[c] + t[c + off];
    const float inv = 1.0f / t[0];
    pf_wave_sync();
#pragma unroll
    for (int c = 0; c < 16; ++c)
      if (c < nct && g == 0) ml[c * 16 + kl].y = m[c] * inv;
  } else {
    for (int row = 0; row < Rt; ++row)
      attn_row_weights(
          nct,
          [&](int c, bool ok, float& m, float& l) {
            const float2 v = ok ? ml[c * 16 + row] : make_float2(0.f, 0.f);
            m = v.x;
            l = v.y;
          },
          [&](int c, float w) { ml[c * 16 + row].y = w; });
  }
  pf_wave_sync();

  // second walk: per block the probabilities, then P V
  float O[8][4];
  floatx4 o[8];
#pragma unroll
  for (int fb = 0; fb < 8; ++fb) {
    o[fb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i) O[fb][i] = 0.f;
  }
  float M = 0.f, wgt = 0.f;
  for (int kb = 0; kb < nk; ++kb) {
    const int t = nk + 2 * kb;
    const bool live = 64 * kb < end;  // uniform
    u32x4p ph[2], pl[2];
    step(t);
    if (live) {
      if ((kb & 3) == 0) {  // the chunk's row max and weight
        uint64_t v;
        asm volatile("ds_read_b64 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(mla + (uint32_t)(kb >> 2) * 128u));
        M = __uint_as_float((uint32_t)v);
        if (M == -INFINITY) M = 0.f;
        wgt = kl < Rt ? __uint_as_float((uint32_t)(v >> 32)) : 0.f;
      }
      float sv[4][4];
      scores(t, kb, sv);
      // the probabilities' two bf16 terms, in the operand layout
#pragma unroll
      for (int ss = 0; ss < 2; ++ss) {
        uint32_t hw[2][2], lw[2][2];
#pragma unroll
        for (int grp = 0; grp < 2; ++grp)
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const float p0 = prob(sv[2 * ss + grp][2 * e], M), p1 = prob(sv[2 * ss + grp][2 * e + 1], M);
            const uint16_t h0 = f2bf_num(p0), h1 = f2bf_num(p1);
            hw[grp][e] = (uint32_t)h0 | ((uint32_t)h1 << 16);
            lw[grp][e] = (uint32_t)f2bf_num(p0 - bf2f(h0)) | ((uint32_t)f2bf_num(p1 - bf2f(h1)) << 16);
          }
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          attn_octet(hw[0][e], hw[1][e]);
          attn_octet(lw[0][e], lw[1][e]);
        }
        ph[ss] = u32x4p{hw[0][0], hw[0][1], hw[1][0], hw[1][1]};
        pl[ss] = u32x4p{lw[0][0], lw[0][1], lw[1][0], lw[1][1]};
      }
    }
    step(t + 1);
    if (live) {
      const uint32_t base = frag + (uint32_t)((t + 1) % NS) * (uint32_t)kPfBlock;
      u32x4p xa[8], xb[8];  // feature tiles 0-3, then 4-7: their two 32-key steps
      xa[0] = pf_read<0>(base);
      xa[1] = pf_read<1>(base);
      xa[2] = pf_read<2>(base);
      xa[3] = pf_read<3>(base);
      xa[4] = pf_read<4>(base);
      xa[5] = pf_read<5>(base);
      xa[6] = pf_read<6>(base);
      xa[7] = pf_read<7>(base);
      xb[0] = pf_read<8>(base);
      xb[1] = pf_read<9>(base);
      xb[2] = pf_read<10>(base);
      xb[3] = pf_read<11>(base);
      xb[4] = pf_read<12>(base);
      xb[5] = pf_read<13>(base);
      xb[6] = pf_read<14>(base);
      xb[7] = pf_read<15>(base);
      pf_wait<0>(xa);
      pf_wait<0>(xb);
      if (64 * kb + 64 > end) {  // this tile's keys only (the verify kernel's tail mask)
#pragma unroll
        for (int x = 0; x < 8; ++x)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int p0 = 64 * kb + 32 * (x & 1) + 8 * g + 2 * e;
            const uint32_t mask = p0 >= end ? 0u : (p0 + 1 >= end ? 0xffffu : 0xffffffffu);
            xa[x][e] &= mask;
            xb[x][e] &= mask;
          }
      }
      auto mul = [&](const u32x4p (&x)[8], int fb0) {
#pragma unroll
        for (int ss = 0; ss < 2; ++ss)
#pragma unroll
          for (int term = 0; term < 2; ++term)
#pragma unroll
            for (int f = 0; f < 4; ++f)
              o[fb0 + f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                  __builtin_bit_cast(bf16x8, x[2 * f + ss]), __builtin_bit_cast(bf16x8, term ? ph[ss] : pl[ss]),
                  o[fb0 + f], 0, 0, 0);
      };
      mul(xa, 0);
      mul(xb, 4);
      if ((kb & 3) == 3 || 64 * kb + 64 >= end) {  // the chunk's (or the tile's) last block
#pragma unroll
        for (int fb = 0; fb < 8; ++fb) {
#pragma unroll
          for (int i = 0; i < 4; ++i) O[fb][i] = attn_acc1(O[fb][i], o[fb][i], wgt);
          o[fb] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
      }
    }
  }
  // the fills past the stream have landed before the LDS is given up
  __builtin_amdgcn_s_waitcnt(0);
  if (kl < Rt)
#pragma unroll
    for (int fb = 0; fb < 8; ++fb) out4(16 * tl + kl, 16 * fb + 4 * g, O[fb]);
}

}  // namespace spade
