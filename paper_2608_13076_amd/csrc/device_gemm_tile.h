// Tiled GEMM for launches of more than 16 rows: batched verification (any
// projection and the LM head) and prefill forwards, with the skinny engine's
// arithmetic and fused epilogues.
//
// A workgroup of eight waves, two per SIMD, owns RT row tiles (16 rows each)
// and 8 P panels (16 columns each); wave w takes panels P w .. with every row
// tile: RT P MFMA output tiles, each with a running k-range accumulator and a
// total.  Weights go straight to the one wave that multiplies them, so a
// 32-k slice costs a compute unit 2 RT KB of activations and 8 P KB of weights
// from L2 and 16 RT KB of LDS reads for 16 RT P MFMAs.  What bounds it is what
// enters the compute unit: all twelve tiles take 17 to 24 ns per KB of
// 2 RT + 8 P (42 to 58 KB/us, a compute unit's read rate), while pairs of tiles
// with a third to three times one another's LDS reads take the same time
// ((6, 1) 96 KB 0.378 us a slice, (2, 2) 32 KB 0.362; (9, 1) 144 KB 0.545,
// (5, 2) 80 KB 0.560).  Counters of the 7B gate/up launch of 144 rows at (9, 1):
// on the compute units in use the matrix cores are busy 0.41 of the time and
// the LDS data path 0.42, without bank conflicts; 69% L2 hits.  Few rows and
// long weights: RT = 9, P = 1 covers 144 rows with one row group; prefill:
// RT = 6 to 9, P = 2 (at (8, 2) the MFMAs need 0.61 of a slice's time).  Four waves of twice
// the panels (one per SIMD, 512 registers) halve the LDS reads and measured
// 5-10% slower: a lone wave's MFMAs wait behind its own loads.
//
// The k-loop runs in 32-k slices (one MFMA k-step, 8 per 256-k block).  The
// activations (two bf16 terms) go by direct buffer->LDS loads, a pair of
// slices (64 k: whole 128-byte lines of the row-major operand; 32-k fills of
// half lines cost 24 us of 90) per ring slot, three pairs ahead; the weight
// fragments of a slice (1 KB per panel, contiguous in the arena's tiles) load
// straight into a register ring, three slices ahead (seven measured the same:
// 82 against 76 us).  Loads are spread over the row tiles instead of issued
// at a slice's ends (7B O projection at 1019 rows 84 -> 78 us); the LDS
// fragments of a row tile are requested three row tiles ahead, across the
// slice boundary; a k-range's partial joins the total one row tile behind the
// MFMAs that finish it.
//
// Measured against the engines this one replaced (us per launch, cold
// weights): 7B gate/up, O, down and QKV at 144 rows 97 -> 72, 31 -> 23,
// 61 -> 40, 57 -> 51; LM head 130 -> 85 (8B: 482 -> 346); 7B O and down at
// 1019 rows 101 -> 68, 252 -> 195.
//
// Arithmetic is the skinny engine's, operation for operation: per output,
// the k-blocks of each of the eight k-ranges (range r: k-blocks
// [NKB r / 8, NKB (r + 1) / 8)) accumulate in a fresh MFMA accumulator, slice
// by slice, the low bf16 term of the activation before the high one; the
// range partials are added to the total in range order (an empty range adds
// nothing).  A row's result does not depend on the engine, the k-splits or
// the other rows.
//
// K-splits (SPLIT): where the panel groups and row groups leave compute units
// idle, split s of KS streams k-ranges [8s / KS, 8(s + 1) / KS); split 0
// stores its running total, every other split each range partial as the range
// ends (write-through).  A second launch (gemm_tile_finish_kernel), one
// workgroup per panel group and row tile, adds them in range order and runs
// the epilogue.
//
// The epilogue moves the totals through a wave-private LDS block so that a
// lane holds the 16 columns of one (row, panel): RoPE and SwiGLU partners and
// the panel's sums are then in one lane, and results leave as 16-byte stores.
#pragma once

#include "device_gemm.h"

#include <utility>

namespace spade {

constexpr int kTileWaves = 8;
constexpr int kTileThreads = kTileWaves * 64;
constexpr int kTileRowPad = 20;                   // floats per staged (row, panel): 16 and padding
constexpr int tile_units(int p) { return kTileWaves * p; }           // panels per workgroup, p per wave
constexpr int tile_stage(int p) { return p * 16 * kTileRowPad; }     // floats of one staged row tile of a wave

// slices of weights in the register ring (divides the 8 of a k-block)
constexpr int kTileDepth = 4;
// row tiles staged at once by the epilogue
constexpr int tile_chunk(int rt, int p) { return rt * p > 12 ? (rt + 1) / 2 : rt; }

template <int RT, int P>
struct GemmTileSmem {
  union {
    // slot (64 k), split, row tile: 16 rows x 128 bytes, the eight 16-byte
    // pieces of row r at piece p ^ (r / 2): the 16 rows of a fragment read
    // land on distinct banks
    uint8_t ring[kTileDepth / 2 + 2][kActSplits][RT][2048];
    float stage[kTileWaves][tile_chunk(RT, P)][tile_stage(P)];
  };
  uint8_t pad[1024];  // target of the fill loads past a slot's blocks (never read)
  float rinv[RT * 16];
};

template <int P>
struct GemmTileFinishSmem {
  float stage[kTileWaves][tile_stage(P)];
  float rinv[16];
};

typedef uint32_t u32x4t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x3t __attribute__((ext_vector_type(3)));

// Published floats of one panel group of a k-split launch of `tiles` row
// tiles: slot r (0: split 0's total, else range r's partial), then per row
// tile, panel and lane one floatx4.
inline __host__ __device__ constexpr size_t tile_item_floats(int tiles, int p) {
  return (size_t)8 * tiles * tile_units(p) * 64 * 4;
}

__device__ __forceinline__ void tile_st16(Rsrc r, uint32_t off, const float* v) {
  const u32x4t d = {__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])};
  __builtin_amdgcn_raw_buffer_store_b128(d, r, (int)off, 0, 0);
}

// The two bf16 terms of eight values, one 16-byte store each (ok == false
// drops them).
__device__ __forceinline__ void tile_st_act8(Rsrc r, uint32_t split_bytes, uint32_t elem, bool ok, const float* v) {
  float rem[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) rem[j] = v[j];
#pragma unroll
  for (int s = 0; s < kActSplits; ++s) {
    u32x4t d;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint16_t h0 = f2bf(rem[2 * j]), h1 = f2bf(rem[2 * j + 1]);
      d[j] = (uint32_t)h0 | ((uint32_t)h1 << 16);
      rem[2 * j] -= bf2f(h0);
      rem[2 * j + 1] -= bf2f(h1);
    }
    __builtin_amdgcn_raw_buffer_store_b128(d, r, (int)(ok ? s * split_bytes + elem * 2u : kOob), 0, 0);
  }
}

// Sum of 16 values in the order of a butterfly over lanes 8, 4, 2, 1 apart
// (no contraction: the terms are rounded products).
__device__ __forceinline__ float tile_sum16(const float* v) {
#pragma clang fp contract(off)
  float s[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) s[j] = v[j] + v[j + 8];
#pragma unroll
  for (int j = 0; j < 4; ++j) s[j] = s[j] + s[j + 4];
  s[0] = s[0] + s[2];
  s[1] = s[1] + s[3];
  return s[0] + s[1];
}

// Epilogue of the 16 columns of (row ml of the launch, panel u): the values
// of gemm_epilogue / gemm_lm_panel, a row's panel per lane.  v: the dot
// products; ok == false stores nothing.
template <int KIND>
__device__ __forceinline__ void tile_epilogue(const GemmParams& a, int u, int ml, bool ok, float rinv, float (&v)[16],
                                              bool& nan_seen) {
  if constexpr (KIND == GEMM_QKV) {
    const int m = a.m0 + ml;
    int bl = m / a.R, ir = m - bl * a.R;
    if (a.row_map != nullptr) {
      const int rm = ok ? a.row_map[m] : 0;
      bl = rm >> 16;
      ir = rm & 0xffff;
    }
    const int bg = a.b0 + bl;
    const int pos = ok ? a.lens[bg] + ir : 0;
    const int pph = a.hd >> 4;
    int pw;
    const int sec = qkv_section(a.unit0 + u, a.d, a.Hkv * a.hd, &pw);
    const int h = pw / pph, wg = pw - h * pph;  // query head (sec 0) or K/V head
    float o[16];
    if (sec < 2) {
      const Rsrc rr = make_rsrc(a.rope, 0x7ffffff0u);
      const uint32_t ro = ok ? (uint32_t)((pos * (a.hd >> 1) + wg * 8) * 2) * 4u : kOob;
      float cs[16];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint4 t = ld_b128<false>(rr, ok ? ro + 16u * j : kOob);
        cs[4 * j] = __uint_as_float(t.x);
        cs[4 * j + 1] = __uint_as_float(t.y);
        cs[4 * j + 2] = __uint_as_float(t.z);
        cs[4 * j + 3] = __uint_as_float(t.w);
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float x = v[j] * rinv, y = v[j + 8] * rinv;
        const float c = cs[2 * j], sn = cs[2 * j + 1];
        // (the fused forms that gemm_epilogue's expressions compile to)
        o[j] = __builtin_fmaf(x, c, -(y * sn));
        o[j + 8] = __builtin_fmaf(y, c, x * sn);
      }
    } else {
#pragma unroll
      for (int j = 0; j < 16; ++j) o[j] = v[j] * rinv;
    }
    const int f0 = wg * 8, f1 = f0 + (a.hd >> 1);
    if (sec == 0) {
      const Rsrc rq = make_rsrc(a.q_out + (size_t)a.m0 * a.d, (uint32_t)((size_t)a.M * a.d * 4));
      const uint32_t e = (uint32_t)(ml * a.d + h * a.hd) * 4u;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        tile_st16(rq, ok ? e + (uint32_t)f0 * 4u + 16u * j : kOob, o + 4 * j);
        tile_st16(rq, ok ? e + (uint32_t)f1 * 4u + 16u * j : kOob, o + 8 + 4 * j);
      }
    } else {
      const Rsrc rkv = make_rsrc(sec == 1 ? a.kc : a.vc, a.kv_bytes);
      const uint32_t head = (uint32_t)(bg * a.Hkv + h) * (uint32_t)a.kv_stride * (uint32_t)a.hd;
      if (a.kv_bf16 && sec == 1) {
        // eight features of a position are one 16-byte piece of its fragment
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          u32x4t d;
#pragma unroll
          for (int j = 0; j < 4; ++j)
            d[j] = (uint32_t)f2bf(o[8 * q + 2 * j]) | ((uint32_t)f2bf(o[8 * q + 2 * j + 1]) << 16);
          const uint32_t el = head + (uint32_t)k_cache_index(q ? f1 : f0, pos, a.hd);
          __builtin_amdgcn_raw_buffer_store_b128(d, rkv, (int)(ok ? el * 2u : kOob), 0, 0);
        }
      } else {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const int f = j < 8 ? f0 + j : f1 + j - 8;
          if (a.kv_bf16) {
            const uint32_t el = head + (uint32_t)v_cache_index(f, pos, a.hd);
            st_b16<false>(rkv, ok ? el * 2u : kOob, f2bf(o[j]));
          } else {
            const uint32_t el = head + (sec == 1 ? (uint32_t)(pos * a.hd + f) : (uint32_t)v_cache_index_f32(f, pos, a.hd));
            st_f32<false>(rkv, ok ? el * 4u : kOob, o[j]);
          }
        }
      }
    }
  } else if constexpr (KIND == GEMM_O || KIND == GEMM_DOWN) {
    const int col = u * 16;
    const Rsrc rx = make_rsrc(a.x + (size_t)a.m0 * a.d, (uint32_t)((size_t)a.M * a.d * 4));
    const Rsrc rg = make_rsrc(a.g_next, (uint32_t)(a.d * 4));
    const uint32_t xo = (uint32_t)(ml * a.d + col) * 4u;
    float x[16], gn[16], sq[16], y[16];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint4 t = ld_b128<false>(rx, ok ? xo + 16u * j : kOob);
      const uint4 s = ld_b128<false>(rg, ok ? (uint32_t)col * 4u + 16u * j : kOob);
      x[4 * j] = __uint_as_float(t.x);
      x[4 * j + 1] = __uint_as_float(t.y);
      x[4 * j + 2] = __uint_as_float(t.z);
      x[4 * j + 3] = __uint_as_float(t.w);
      gn[4 * j] = __uint_as_float(s.x);
      gn[4 * j + 1] = __uint_as_float(s.y);
      gn[4 * j + 2] = __uint_as_float(s.z);
      gn[4 * j + 3] = __uint_as_float(s.w);
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      x[j] = x[j] + v[j];
      y[j] = x[j] * gn[j];
      sq[j] = x[j] * x[j];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) tile_st16(rx, ok ? xo + 16u * j : kOob, x + 4 * j);
    const uint32_t split_b = (uint32_t)(a.act_out_split * 2);
    const Rsrc ro = make_rsrc((const uint8_t*)a.act_out + (size_t)a.m0 * a.act_out_stride * 2,
                              (uint32_t)((kActSplits - 1) * (size_t)split_b + (size_t)a.M * a.act_out_stride * 2));
#pragma unroll
    for (int q = 0; q < 2; ++q)
      tile_st_act8(ro, split_b, (uint32_t)(ml * a.act_out_stride + col + 8 * q), ok, y + 8 * q);
    const Rsrc rs = make_rsrc(a.ssq_out + (size_t)a.m0 * a.n_ssq_out, (uint32_t)((size_t)a.M * a.n_ssq_out * 4));
    st_f32<false>(rs, ok ? (uint32_t)(ml * a.n_ssq_out + u) * 4u : kOob, tile_sum16(sq));
  } else if constexpr (KIND == GEMM_GU) {
    float act[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float g = v[j] * rinv, up = v[j + 8] * rinv;
      act[j] = g / (1.0f + expf(-g)) * up;
    }
    const uint32_t split_b = (uint32_t)(a.act_out_split * 2);
    const Rsrc ro = make_rsrc((const uint8_t*)a.act_out + (size_t)a.m0 * a.act_out_stride * 2,
                              (uint32_t)((kActSplits - 1) * (size_t)split_b + (size_t)a.M * a.act_out_stride * 2));
    tile_st_act8(ro, split_b, (uint32_t)(ml * a.act_out_stride + u * 8), ok, act);
  } else {
#pragma clang fp contract(off)  // (the exponents' differences take rounded products)
    // LM head: the panel's (max, sum exp, argmax) of z (tile_logits stores the
    // logits).  A wave whose lanes all hold sixteen finite-or-infinite logits
    // with a maximum above -inf takes the short form, the same values: the
    // maximum first, its lowest column after, no test per exponential (about
    // 300 instead of 600 instructions per step).
    const float sc = gemm_lm_samp(a, ml, ok) ? a.inv_T : 1.0f;
    const int col = u * 16;
    float z[16], ex[16];
    bool nan = false;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      z[j] = v[j] * rinv;
      z[j] = z[j] * sc;
    }
#pragma unroll
    for (int j = 0; j < 16; j += 2) nan = nan || __builtin_isunordered(z[j], z[j + 1]);
    RowStat ps{z[0], 0.f, 0};
#pragma unroll
    for (int j = 1; j < 16; ++j) ps.m = fmaxf(ps.m, z[j]);
    if (__all(!ok || (col + 16 <= a.V && !nan && ps.m > -INFINITY))) {
#pragma unroll
      for (int j = 15; j >= 0; --j) ps.a = z[j] == ps.m ? col + j : ps.a;
#pragma unroll
      for (int j = 0; j < 16; ++j) ex[j] = expf(z[j] - ps.m);
    } else {
      ps = RowStat{-INFINITY, 0.f, 0x7fffffff};
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const bool valid = ok && col + j < a.V;
        const float lg = v[j] * rinv;
        const bool isnan = lg != lg;
        nan_seen = nan_seen || (valid && isnan);
        const bool use = valid && !isnan;
        z[j] = use ? z[j] : -INFINITY;
        const int id = use ? col + j : 0x7fffffff;
        if (z[j] > ps.m || (z[j] == ps.m && id < ps.a)) {
          ps.m = z[j];
          ps.a = id;
        }
      }
#pragma unroll
      for (int j = 0; j < 16; ++j) ex[j] = (z[j] == -INFINITY) ? 0.f : expf(z[j] - ps.m);
    }
    ps.s = tile_sum16(ex);
    const Rsrc rs = make_rsrc(a.pstats + (size_t)a.m0 * a.n_units * 3, (uint32_t)((size_t)a.M * a.n_units * 12));
    const u32x3t d = {__float_as_uint(ps.m), __float_as_uint(ps.s), (uint32_t)ps.a};
    __builtin_amdgcn_raw_buffer_store_b96(d, rs, (int)(ok ? (uint32_t)(ml * a.n_units + u) * 12u : kOob), 0, 0);
  }
}

// The logits of NT row tiles from the wave's staging block: consecutive lanes
// store consecutive columns of a row, whole lines where the rows allow it (a
// row's panel per lane took eight requests of 16 bytes per 128-byte line).
// With the short statistics above: 8B at 144 rows, 128K vocabulary, the verify
// call of four layers 1275 -> 1265 us; 7B, 32K vocabulary, 1372 -> 1369.
template <int NT, int P>
__device__ __forceinline__ void tile_logits(const GemmParams& a, const float* stage, int first, int u0,
                                            const float* rinv, int lane) {
  const Rsrc rl = make_rsrc(a.logits + (size_t)a.m0 * a.V, (uint32_t)((size_t)a.M * a.V * 4));
  // whole 16-byte pieces when every row of the logits starts on one
  if ((((uint32_t)(size_t)a.logits | (uint32_t)(a.V * 4)) & 15u) == 0u) {
    constexpr int W = 4 * P;  // lanes per row
    const int c = (lane % W) * 4;
    const int col = u0 * 16 + c;
#pragma unroll 2
    for (int r = lane / W; r < NT * 16; r += 64 / W) {
      const floatx4 x = *(const floatx4*)(stage + (r >> 4) * tile_stage(P) + ((c >> 4) * 16 + (r & 15)) * kTileRowPad + (c & 15));
      const float ri = rinv[r];
      const float lg[4] = {x[0] * ri, x[1] * ri, x[2] * ri, x[3] * ri};
      tile_st16(rl, (first + r < a.M && col < a.V) ? (uint32_t)((first + r) * a.V + col) * 4u : kOob, lg);
    }
  } else {
    constexpr int W = 16 * P;
    const int c = lane % W;
    const int col = u0 * 16 + c;
#pragma unroll 4
    for (int r = lane / W; r < NT * 16; r += 64 / W) {
      const float x = stage[(r >> 4) * tile_stage(P) + ((c >> 4) * 16 + (r & 15)) * kTileRowPad + (c & 15)];
      st_f32<false>(rl, (first + r < a.M && col < a.V) ? (uint32_t)((first + r) * a.V + col) * 4u : kOob, x * rinv[r]);
    }
  }
}

// Totals of NT row tiles (MFMA layout: lane 16 g + c holds rows 4 g .. + 3 of
// column c) through the wave's staging block, then the epilogue of each
// (row, panel).  first: the launch row of the first tile.
template <int KIND, int NT, int P>
__device__ __forceinline__ void tile_store(const GemmParams& a, float* stage, const floatx4 (&t)[NT][P], int first,
                                           int u0, const float* rinv, int lane, bool& nan_seen) {
  static_assert(P == 1 || P == 2 || P == 4, "whole row tiles per step");
  constexpr int U = 4 / P;  // row tiles per step of 64 (row, panel) lanes
  const int g = lane >> 4, kl = lane & 15;
#pragma unroll
  for (int mt = 0; mt < NT; ++mt)
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        stage[mt * tile_stage(P) + (p * 16 + 4 * g + i) * kTileRowPad + kl] = t[mt][p][i];
  // the block is this wave's own: its LDS operations complete in order
  __builtin_amdgcn_wave_barrier();
  if constexpr (KIND == GEMM_LM) tile_logits<NT, P>(a, stage, first, u0, rinv, lane);
  const int u = u0 + g % P;
  const bool uok = u < a.n_units;
#pragma unroll 1
  for (int m0 = 0; m0 < NT; m0 += U) {
    const int mt = m0 + g / P;
    const bool in = mt < NT;
    const int mr = in ? mt : 0;
    const int ml = first + mr * 16 + kl;
    float v[16];
    const float* src = stage + mr * tile_stage(P) + ((g % P) * 16 + kl) * kTileRowPad;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const floatx4 x = *(const floatx4*)(src + 4 * j);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[4 * j + i] = x[i];
    }
    tile_epilogue<KIND>(a, uok ? u : 0, ml, in && uok && ml < a.M, rinv[mr * 16 + kl], v, nan_seen);
  }
  __builtin_amdgcn_wave_barrier();
}

// NTW: weights with the non-temporal policy.
template <int KIND, int RT, int P, bool SPLIT, bool NTW>
struct GemmTile {
  static_assert(!SPLIT || KIND != GEMM_LM, "the LM head is not k-split");
  static constexpr int S = kActSplits;
  static constexpr int D = kTileDepth;
  static constexpr int DP = D / 2 + 1;             // slots (pairs of slices) requested ahead
  static constexpr int SLOTS = DP + 1;
  static constexpr int SLOT = S * RT * 2048;       // bytes of a slot
  static constexpr int NFB = (4 * RT + kTileWaves - 1) / kTileWaves;  // 1 KB fill blocks per wave and slot
  static constexpr int NL = NFB + 2 * P;           // loads per wave and slot, with 2 P weight fragments
  static constexpr int PF = RT < 3 ? RT : 3;       // row tiles whose fragments are read ahead
  // whether a range's partials join the totals after its last slice instead of
  // among its MFMAs: two copies of that slice cost RT P > 12 tiles their
  // registers (RT = 8, P = 2: 226 instead of 256 and 204 bytes of scratch)
  static constexpr bool LATE = RT * P > 12;
  static constexpr int NX = 4;                     // fragment registers: row tiles in flight and in use
  static_assert(8 % D == 0 && (8 * RT) % NX == 0 && PF < NX, "rings indexed by the slice within its k-block");
  static_assert((DP - 1) * NFB + (D - 1) * P < 64, "vmcnt range");
  const GemmParams& a;
  GemmTileSmem<RT, P>& sm;
  int tid, lane, wave, g, kl;
  int row0, u0;        // first row of the workgroup, first panel of this wave
  int NKB, ks, KS;
  int kb0, kb1, T;     // k-blocks [kb0, kb1) of the split, T = 8 (kb1 - kb0) slices
  uint32_t lds_ring;   // LDS byte address of the ring
  uint32_t frag_off;   // this lane's fragment offset within a row tile's block (first k-step; the second: ^ 64)
  uint32_t foff[NFB];  // this lane's byte offsets of its fill blocks at the split's start
  Rsrc ract;           // activations of the launch's rows, both splits
  Rsrc rw[P];          // this wave's weight panels (empty past n_units)
  Rsrc rp;             // published values (SPLIT)
  int ptiles;          // row tiles of the launch (published layout)
  floatx4 acc[RT][P], tot[RT][P];
  uint4 wq[D][P];      // weight fragments of the slices in flight
  u32x4t x[NX][S];      // activation fragments of the row tiles in flight
  int rnext, bnd;      // next k-range, the k-block its range starts at

  __device__ __forceinline__ GemmTile(const GemmParams& a_, GemmTileSmem<RT, P>& sm_, int rg, int ug, int ks_, int KS_,
                                      float* part)
      : a(a_), sm(sm_), ks(ks_), KS(KS_) {
    tid = threadIdx.x;
    lane = tid & 63;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    g = lane >> 4;
    kl = lane & 15;
    row0 = rg * RT * 16;
    u0 = ug * tile_units(P) + wave * P;
    NKB = a.NKB;
    lds_ring = (uint32_t)(size_t)(__attribute__((address_space(3))) void*)&sm.ring[0][0][0][0];
    frag_off = (uint32_t)(kl * 128 + 16 * (g ^ (kl >> 1)));
    ract = make_rsrc((const uint8_t*)a.act + (size_t)a.m0 * a.act_stride * 2,
                     (uint32_t)(((size_t)(S - 1) * a.act_split + (size_t)a.M * a.act_stride) * 2));
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const int u = u0 + p;
      const bool ok = u < a.n_units;
      rw[p] = make_rsrc(a.w + (size_t)(ok ? u : 0) * NKB * kTileBytes, ok ? (uint32_t)(NKB * kTileBytes) : 0u);
    }
    if constexpr (SPLIT) {
      ptiles = (a.M + 15) / 16;
      rp = make_rsrc(part + (size_t)ug * tile_item_floats(ptiles, P), (uint32_t)(tile_item_floats(ptiles, P) * 4));
    }
#pragma unroll
    for (int mt = 0; mt < RT; ++mt)
#pragma unroll
      for (int p = 0; p < P; ++p) {
        acc[mt][p] = floatx4{0.f, 0.f, 0.f, 0.f};
        tot[mt][p] = floatx4{0.f, 0.f, 0.f, 0.f};
      }
    // ranges [r_lo, r_hi) of this split; rnext / bnd: the first non-empty one
    const int r_lo = SPLIT ? kGemmWaves * ks / KS : 0, r_hi = SPLIT ? kGemmWaves * (ks + 1) / KS : kGemmWaves;
    kb0 = NKB * r_lo / kGemmWaves;
    kb1 = NKB * r_hi / kGemmWaves;
    T = (kb1 - kb0) * 8;
    rnext = r_lo + 1;
    bnd = NKB * rnext / kGemmWaves;
    while (bnd == kb0 && rnext < r_hi) bnd = (NKB * ++rnext) / kGemmWaves;
    // wave w moves blocks w, w + 8, ... of a slot's 4 RT: 8 rows x 128 bytes
    // (whole lines of the row-major operand), one 16-byte piece per lane
    // (lane l: row l / 8, piece l % 8 of the swizzled block).  Rows past M
    // repeat row M - 1: finite values whose products are never stored.
#pragma unroll
    for (int i = 0; i < NFB; ++i) {
      const int q = wave + kTileWaves * i;
      const int s = q / (2 * RT), mt = (q >> 1) % RT;
      const int r = (q & 1) * 8 + (lane >> 3), lp = (lane & 7) ^ (r >> 1);
      const int row = row0 + mt * 16 + r;
      const int grow = row < a.M ? row : a.M - 1;
      foff[i] = q < 4 * RT ? (uint32_t)(((size_t)s * a.act_split + (size_t)grow * a.act_stride + (size_t)kb0 * 256 +
                                         lp * 8) * 2)
                           : kOob;
    }
  }

  // Block i of this wave's share of the pair of slices t, t + 1 (t even) of
  // the split into ring slot `slot`; pairs past the split read zeros, so every
  // wave always issues the same loads and the wait counts are constants.
  __device__ __forceinline__ void fill1(int i, int t, int slot) const {
    const uint32_t off = t < T ? foff[i] + (uint32_t)t * 64u : kOob;
    const int q = wave + kTileWaves * i;
    uint8_t* d = &sm.ring[0][0][0][0] + slot * SLOT + q * 1024;
    if ((i + 1) * kTileWaves > 4 * RT) d = q < 4 * RT ? d : &sm.pad[0];
    __builtin_amdgcn_raw_ptr_buffer_load_lds(ract, (__attribute__((address_space(3))) void*)d, 16, off, 0, 0, 0);
  }

  // weight fragment of slice t for this wave's panel p (zeros past the split)
  __device__ __forceinline__ uint4 load_w(int t, int p) const {
    const uint32_t off = t < T ? (uint32_t)((kb0 + (t >> 3)) * kTileBytes + (t & 7) * 1024 + lane * 16) : kOob;
    return NTW ? ld_stream_b128(rw[p], off) : ld_b128<false>(rw[p], off);
  }

  template <int OFF>
  __device__ __forceinline__ static u32x4t ds_read16(uint32_t addr) {
    u32x4t v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
  }

  // both terms' fragments of row tile MT at `base` (slot and k-step)
  template <int MT>
  __device__ __forceinline__ static void read_tile(uint32_t base, u32x4t (&f)[S]) {
    f[0] = ds_read16<MT * 2048>(base);
    f[1] = ds_read16<(RT + MT) * 2048>(base);
  }

  // wait until at most N of this wave's LDS reads are outstanding; the
  // fragments f depend on the wait
  template <int N>
  __device__ __forceinline__ static void lds_wait(u32x4t (&f)[S]) {
    asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(f[0]), "+v"(f[1]) : "n"(N));
  }

  // No fragment read may be in flight where the control flow branches or
  // joins: the compiler takes an asm output as written at once and may copy
  // it to another register there.
  template <int N = NX>
  __device__ __forceinline__ void lds_drain() {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; ++i) lds_wait<0>(x[i]);
    __builtin_amdgcn_sched_barrier(0);
  }

  __device__ __forceinline__ uint32_t part_off(int slot, int mt) const {
    return (uint32_t)(((slot * ptiles + row0 / 16 + mt) * tile_units(P) + wave * P) * 64 + lane) * 16u;
  }

  // The end of a k-range for row tile mt: the partial joins the total (split
  // 0 or no splits) or is published in the range's slot.
  __device__ __forceinline__ void close_tile(int mt) {
#pragma unroll
    for (int p = 0; p < P; ++p) {
      if (!SPLIT || ks == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) tot[mt][p][i] += acc[mt][p][i];
      } else {
        const bool in = row0 / 16 + mt < ptiles;
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4t, acc[mt][p]), rp,
                                               (int)(in ? part_off(rnext - 1, mt) + (uint32_t)p * 1024u : kOob), 0,
                                               kAuxCoh);
      }
      acc[mt][p] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
  }

  // Row tile MT of slice t, J = t % 8 (ring bases b0 of this slice, b1 of the
  // next): its share of the slice's requests, the fragments of the row tile
  // PF ahead, then the MFMAs, the low term first.  Requests are spread over
  // the row tiles: a 1 KB load holds the compute unit's address path for 16
  // clocks, and a wave that issues all of a slice's loads at once waits for
  // the other waves' with its MFMAs behind them.
  template <int J, int MT, bool LAST>
  __device__ __forceinline__ void row_tile(int t, int fslot, uint32_t b0, uint32_t b1) {
    constexpr int I = (J * RT + MT) % NX, N = (J * RT + MT + PF) % NX;
    constexpr int NEXT = MT + PF;
    if constexpr (NEXT < RT) read_tile<NEXT % RT>(b0, x[N]);
    else read_tile<NEXT % RT>(b1, x[N]);
    // the pair's fill blocks alternate with the weights of slice t + D - 1
    constexpr int H = J & 1, F0 = H * NFB / 2, NF = (H + 1) * NFB / 2 - F0, NS = NF + P;
#pragma unroll
    for (int l = NS * MT / RT; l < NS * (MT + 1) / RT; ++l) {
      if (l < NF) fill1(F0 + l, t - H + 2 * DP, fslot);
      else wq[(J + D - 1) % D][l - NF] = load_w(t + D - 1, l - NF);
    }
    lds_wait<2 * PF>(x[I]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int s = S - 1; s >= 0; --s)
        acc[MT][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x[I][s]),
                                                             __builtin_bit_cast(bf16x8, wq[J % D][p]), acc[MT][p], 0, 0, 0);
    if constexpr (LAST && !SPLIT && MT > 0) close_tile(MT - 1);
    __builtin_amdgcn_sched_barrier(0);
  }

  // slice t = 8 (kb - kb0) + J.  At the start of a pair u = t / 2, once every
  // load up to pair u + 1 - DP's has landed (pair u + 1's fill and this
  // pair's weights among them; loads complete in issue order), the barrier
  // publishes the next slot and ends every wave's reads of the previous one,
  // which pair u + DP's fill then overwrites; slice t + D - 1's weights go
  // where slice t - 1's were.
  template <int J, bool LAST, int... MT>
  __device__ __forceinline__ void slice(int t, std::integer_sequence<int, MT...>) {
    wait_vmcnt<(D - 2) / 2 * NL>();
    __builtin_amdgcn_sched_barrier(0);
    if constexpr ((J & 1) == 0) {
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
    }
    const int s1 = slot + 1 == SLOTS ? 0 : slot + 1;
    const int fslot = slot == 0 ? SLOTS - 1 : slot - 1;
    const uint32_t base = lds_ring + (uint32_t)slot * (uint32_t)SLOT;
    const uint32_t b0 = base + (frag_off ^ ((J & 1) ? 64u : 0u));
    const uint32_t b1 = (J & 1) ? lds_ring + (uint32_t)s1 * (uint32_t)SLOT + frag_off : base + (frag_off ^ 64u);
    if constexpr (J & 1) slot = s1;
    (row_tile<J, MT, LAST>(t, fslot, b0, b1), ...);
    if constexpr (J == 7) lds_drain();
    if constexpr (LAST) {
      if constexpr (SPLIT) {
#pragma unroll
        for (int mt = 0; mt < RT; ++mt) close_tile(mt);
      } else {
        close_tile(RT - 1);
      }
      next_range(kb0 + (t >> 3));
    }
  }

  int slot;  // ring slot of the slice in use

  __device__ __forceinline__ void next_range(int kb) {
    do {
      ++rnext;
      bnd = (NKB * rnext) / kGemmWaves;
    } while (bnd == kb + 1 && rnext < kGemmWaves);
  }

  __device__ __forceinline__ void range_end(int kb) {
#pragma unroll
    for (int mt = 0; mt < RT; ++mt) close_tile(mt);
    next_range(kb);
  }

  // Row scales of rows 32 i + tid / 16: this thread takes partials tid % 16,
  // + 16, ... of each row in order, as gemm_row_rinv does.  The first 256 of a
  // row are requested before the ring and summed once the ring's loads are on
  // their way.
  static constexpr int NR = (RT + 1) / 2;
  __device__ __forceinline__ void row_load(int q0, float (&v)[NR][16]) const {
    const Rsrc rs = make_rsrc(a.ssq_in + (size_t)a.m0 * a.n_ssq, (uint32_t)((size_t)a.M * a.n_ssq * 4));
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int r = 32 * i + (tid >> 4), row = row0 + r;
#pragma unroll
      for (int f = 0; f < 16; ++f) {
        const int q = q0 + (tid & 15) + f * 16;
        v[i][f] = ld_f32<false>(rs, (r < RT * 16 && row < a.M && q < a.n_ssq) ? (uint32_t)(row * a.n_ssq + q) * 4u : kOob);
      }
    }
  }
  __device__ __forceinline__ void row_sums(float (&v)[NR][16], float (&ss)[NR]) const {
#pragma unroll
    for (int i = 0; i < NR; ++i) ss[i] = 0.f;
    for (int q0 = 0;; row_load(q0, v)) {
#pragma unroll
      for (int i = 0; i < NR; ++i)
#pragma unroll
        for (int f = 0; f < 16; ++f) ss[i] += v[i][f];
      q0 += 256;
      if (q0 >= a.n_ssq) break;
    }
  }

  // 1/rms of a row from its sixteen threads' sums (all of them get it)
  __device__ __forceinline__ float row_rinv(float s, int row) const {
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) s += __shfl_xor(s, off);
    return row < a.M ? 1.0f / sqrtf(s * a.inv_din + a.eps) : 1.0f;
  }

  template <int... I>
  __device__ __forceinline__ void kblock(int kb, std::integer_sequence<int, I...>) {
    const int t0 = (kb - kb0) * 8;
    (slice<I, false>(t0 + I, std::make_integer_sequence<int, RT>{}), ...);
    if constexpr (!LATE) lds_drain();
    if constexpr (LATE) {
      slice<7, false>(t0 + 7, std::make_integer_sequence<int, RT>{});
      if (kb + 1 == bnd) range_end(kb);
    } else {
      if (kb + 1 == bnd) slice<7, true>(t0 + 7, std::make_integer_sequence<int, RT>{});
      else slice<7, false>(t0 + 7, std::make_integer_sequence<int, RT>{});
    }
  }

  __device__ __forceinline__ void run() {
    // the row scales' loads go first (they are older than the ring's, so they
    // are waited for alone) and are summed once the ring's are on their way
    constexpr bool RINV = KIND != GEMM_O && KIND != GEMM_DOWN && !SPLIT;
    float ss[NR], sv[NR][16];
    if constexpr (RINV) row_load(0, sv);
    __builtin_amdgcn_sched_barrier(0);
    if (T > 0) {
      slot = 0;
      // the first DP pairs of the ring and D - 1 slices of weights, in the
      // order in which slices -2 DP .. -1 would have requested them (the
      // loop's wait counts rely on it)
#pragma unroll
      for (int t = -2 * DP; t < 0; ++t) {
        const int h = t & 1;
#pragma unroll
        for (int j = h * NFB / 2; j < (h + 1) * NFB / 2; ++j) fill1(j, t - h + 2 * DP, (t - h) / 2 + DP);
        __builtin_amdgcn_sched_barrier(0);
        if (t + D - 1 >= 0) {
#pragma unroll
          for (int p = 0; p < P; ++p) wq[t + D - 1][p] = load_w(t + D - 1, p);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (RINV) row_sums(sv, ss);
      __builtin_amdgcn_sched_barrier(0);
      wait_vmcnt<(DP - 1) * NFB + (D - 1) * P>();
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      const uint32_t b0 = lds_ring + frag_off;
      read_tile<0>(b0, x[0]);
      read_tile<1>(b0, x[1]);
      if constexpr (PF > 2) read_tile<2 % RT>(b0, x[2]);
      lds_drain<PF>();
      for (int kb = kb0; kb < kb1; ++kb) kblock(kb, std::make_integer_sequence<int, 7>{});
    }
    if constexpr (SPLIT) {
      if (ks == 0) {
#pragma unroll
        for (int mt = 0; mt < RT; ++mt)
#pragma unroll
          for (int p = 0; p < P; ++p) {
            const bool in = row0 / 16 + mt < ptiles;
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4t, tot[mt][p]), rp,
                                                   (int)(in ? part_off(0, mt) + (uint32_t)p * 1024u : kOob), 0, kAuxCoh);
          }
      }
      // the workgroup ends once the fills past the split have landed in its LDS
      __builtin_amdgcn_s_waitcnt(0);
    } else {
      // the ring is idle once every fill has landed and every wave is past
      // its last read: it becomes the staging blocks
      __builtin_amdgcn_s_waitcnt(0);
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        const int r = 32 * i + (tid >> 4);
        const float ri = RINV ? row_rinv(ss[i], row0 + r) : 1.0f;
        if ((tid & 15) == 0 && r < RT * 16) sm.rinv[r] = ri;
      }
      __syncthreads();
      bool nan_seen = false;
      constexpr int CH = tile_chunk(RT, P);
      {
        floatx4 t[CH][P];
#pragma unroll
        for (int mt = 0; mt < CH; ++mt)
#pragma unroll
          for (int p = 0; p < P; ++p) t[mt][p] = tot[mt][p];
        tile_store<KIND, CH, P>(a, &sm.stage[wave][0][0], t, row0, u0, sm.rinv, lane, nan_seen);
      }
      if constexpr (CH < RT) {
        floatx4 t[RT - CH][P];
#pragma unroll
        for (int mt = CH; mt < RT; ++mt)
#pragma unroll
          for (int p = 0; p < P; ++p) t[mt - CH][p] = tot[mt][p];
        tile_store<KIND, RT - CH, P>(a, &sm.stage[wave][0][0], t, row0 + CH * 16, u0, sm.rinv + CH * 16, lane, nan_seen);
      }
      if (KIND == GEMM_LM && nan_seen) flag_error(a.err, SPADE_DERR_NAN);
    }
  }
};

// Second pass of a k-split launch: workgroup (panel group ug, row tile mt),
// wave w its panels P w .. : split 0's total plus the non-empty ranges of the
// other splits in range order, then the epilogue.
template <int KIND, int P>
struct GemmTileFinish {
  const GemmParams& a;
  GemmTileFinishSmem<P>& sm;

  __device__ __forceinline__ void run(int ug, int mt, int KS, const float* part) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles = (a.M + 15) / 16;
    const size_t item = tile_item_floats(tiles, P);
    const Rsrc rp = make_rsrc(part + (size_t)ug * item, (uint32_t)(item * 4));
    const uint32_t base = (uint32_t)((mt * tile_units(P) + wave * P) * 64 + lane) * 16u;
    const uint32_t step = (uint32_t)(tiles * tile_units(P) * 64) * 16u;  // bytes of a slot
    const int NKB = a.NKB;
    floatx4 t[1][P], x[kGemmWaves - 1][P];
#pragma unroll
    for (int p = 0; p < P; ++p) t[0][p] = __builtin_bit_cast(floatx4, ld_b128<true>(rp, base + 1024u * p));
#pragma unroll
    for (int r = 1; r < kGemmWaves; ++r) {
      const bool use = r >= kGemmWaves / KS && NKB * (r + 1) / kGemmWaves > NKB * r / kGemmWaves;
#pragma unroll
      for (int p = 0; p < P; ++p)
        x[r - 1][p] = __builtin_bit_cast(floatx4, ld_b128<true>(rp, use ? base + step * r + 1024u * p : kOob));
    }
    if (tid < 256) {
      const float ri = gemm_row_rinv(a, mt * 16 + (tid >> 4), tid & 15);
      if ((tid & 15) == 0) sm.rinv[tid >> 4] = ri;
    }
#pragma unroll
    for (int r = 1; r < kGemmWaves; ++r) {
      const bool use = r >= kGemmWaves / KS && NKB * (r + 1) / kGemmWaves > NKB * r / kGemmWaves;
      if (use) {
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
          for (int i = 0; i < 4; ++i) t[0][p][i] += x[r - 1][p][i];
      }
    }
    __syncthreads();
    bool nan_seen = false;
    tile_store<KIND, 1, P>(a, sm.stage[wave], t, mt * 16, ug * tile_units(P) + wave * P, sm.rinv, lane, nan_seen);
  }
};

// Host-side shape of a launch.
inline __host__ __device__ int gemm_tile_unit_groups(int n_units, int p) { return (n_units + tile_units(p) - 1) / tile_units(p); }
inline __host__ __device__ int gemm_tile_row_groups(int M, int rt) { return ((M + 15) / 16 + rt - 1) / rt; }

}  // namespace spade
