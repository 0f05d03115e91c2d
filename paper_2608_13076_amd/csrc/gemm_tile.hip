// Tiled GEMM kernels (device_gemm_tile.h): launches and the choice of tile.
#include "device_gemm_tile.h"

#include <algorithm>
#include <iterator>

namespace spade {
namespace {

// Workgroup b runs on XCD b % 8, which owns panel groups b % 8 + 8 c.  Its
// workgroups go in blocks of up to 4 row groups x every one of its panel
// groups (then k-splits, row groups fastest), so those that run together on
// an XCD share their weight panels and activation rows in its L2.
template <int KIND, int RT, int P, bool SPLIT, bool NTW>
__global__ void __launch_bounds__(kTileThreads) gemm_tile_kernel(GemmParams a, int NRG, int NUG, int KS, float* part) {
  extern __shared__ uint4 lds_dyn[];
  constexpr int RB = 4;
  const int b = (int)blockIdx.x, NC = (NUG + 7) / 8;
  const int per = RB * NC * KS, full = NRG / RB;
  int q = b >> 3, rg0 = full * RB, rbs = NRG - rg0;
  if (q < full * per) {
    rg0 = q / per * RB;
    rbs = RB;
    q %= per;
  } else {
    q -= full * per;
  }
  const int c = q / (rbs * KS);
  q -= c * rbs * KS;
  const int ks = q / rbs, rg = rg0 + q - ks * rbs;
  const int ug = (b & 7) + 8 * c;
  if (ug >= NUG) return;  // uniform, before any barrier
  GemmTile<KIND, RT, P, SPLIT, NTW> t(a, *(GemmTileSmem<RT, P>*)lds_dyn, rg, ug, ks, KS, part);
  t.run();
}

// Second pass of a k-split launch: workgroup (panel group, row tile).
template <int KIND, int P>
__global__ void __launch_bounds__(kTileThreads) gemm_tile_finish_kernel(GemmParams a, int KS, const float* part) {
  __shared__ GemmTileFinishSmem<P> sm;
  const int tiles = (a.M + 15) / 16;
  const int ug = (int)blockIdx.x / tiles, mt = (int)blockIdx.x - ug * tiles;
  GemmTileFinish<KIND, P> f{a, sm};
  f.run(ug, mt, KS, part);
}

template <int KIND, int RT, int P, bool SPLIT, bool NTW>
hipError_t launch_one(const GemmParams& gp, int ks, float* part, hipStream_t st) {
  const void* fn = reinterpret_cast<const void*>(&gemm_tile_kernel<KIND, RT, P, SPLIT, NTW>);
  constexpr uint32_t lds = (uint32_t)sizeof(GemmTileSmem<RT, P>);
  static_assert(lds <= 160 * 1024, "LDS of a compute unit");
  static hipError_t attr = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (attr != hipSuccess) return attr;
  const int nrg = gemm_tile_row_groups(gp.M, RT), nug = gemm_tile_unit_groups(gp.n_units, P);
  hipLaunchKernelGGL((gemm_tile_kernel<KIND, RT, P, SPLIT, NTW>), dim3(8 * ((nug + 7) / 8) * nrg * ks),
                     dim3(kTileThreads), lds, st, gp, nrg, nug, ks, part);
  if constexpr (SPLIT) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((gemm_tile_finish_kernel<KIND, P>), dim3(nug * ((gp.M + 15) / 16)), dim3(kTileThreads), 0, st,
                       gp, ks, (const float*)part);
  }
  return hipGetLastError();
}

// Non-temporal weight loads while at most kTileNtRowGroups workgroups re-read
// a weight tile (batched verification); prefill forwards keep them in L2.
constexpr int kTileNtRowGroups = 4;

template <int KIND, int RT, int P>
hipError_t launch_tile_rp(const GemmParams& gp, int ks, float* part, hipStream_t st) {
  if constexpr (KIND != GEMM_LM)
    if (ks > 1) return launch_one<KIND, RT, P, true, true>(gp, ks, part, st);
  if (gemm_tile_row_groups(gp.M, RT) <= kTileNtRowGroups) return launch_one<KIND, RT, P, false, true>(gp, 1, part, st);
  return launch_one<KIND, RT, P, false, false>(gp, 1, part, st);
}

template <int KIND>
hipError_t launch_tile_kind(const GemmParams& gp, const TileChoice& c, float* part, hipStream_t st) {
  if (c.p == 2) {
    switch (c.rt) {
      case 2: return launch_tile_rp<KIND, 2, 2>(gp, c.ks, part, st);
      case 3: return launch_tile_rp<KIND, 3, 2>(gp, c.ks, part, st);
      case 4: return launch_tile_rp<KIND, 4, 2>(gp, c.ks, part, st);
      case 5: return launch_tile_rp<KIND, 5, 2>(gp, c.ks, part, st);
      case 6: return launch_tile_rp<KIND, 6, 2>(gp, c.ks, part, st);
      case 8: return launch_tile_rp<KIND, 8, 2>(gp, c.ks, part, st);
      default: return launch_tile_rp<KIND, 9, 2>(gp, c.ks, part, st);
    }
  }
  switch (c.rt) {
    case 4: return launch_tile_rp<KIND, 4, 1>(gp, c.ks, part, st);
    case 5: return launch_tile_rp<KIND, 5, 1>(gp, c.ks, part, st);
    case 6: return launch_tile_rp<KIND, 6, 1>(gp, c.ks, part, st);
    case 7: return launch_tile_rp<KIND, 7, 1>(gp, c.ks, part, st);
    default: return launch_tile_rp<KIND, 9, 1>(gp, c.ks, part, st);
  }
}

// The tiles that are built, each with the time one workgroup takes for a 32-k
// slice (us).  Fitted, with the constants of tile_choice, to 490 launches of
// the 7B and 8B projections at 144, 1019 and 2040 rows over every tile and
// k-split (rms error 9%; the picks within 5% of the fastest of each of those
// shapes; an LM head of 128K columns takes a fifth to a quarter more).
struct TileCost {
  int rt, p;
  double slice_us;
};
constexpr TileCost kTileCosts[] = {{2, 2, 0.362}, {3, 2, 0.418}, {4, 2, 0.479}, {5, 2, 0.56},
                                   {6, 2, 0.609}, {8, 2, 0.694}, {9, 2, 0.828}, {4, 1, 0.273},
                                   {5, 1, 0.354}, {6, 1, 0.378}, {7, 1, 0.415}, {9, 1, 0.545}};

}  // namespace

bool tile_built(int rt, int p) {
  return std::any_of(std::begin(kTileCosts), std::end(kTileCosts),
                     [=](const TileCost& t) { return t.rt == rt && t.p == p; });
}

// Tile and k-splits of a launch: the least estimate of
//   rounds of workgroups (one per compute unit at a time, the panel groups of
//   an XCD on its eighth of them)
//     x (slices of the longest k-split x the tile's time per slice + 2 us)
//   + 3 us, and for k-splits 5 us more for the second launch and the
//   published values written and read back at 8 TB/s,
// but no less than the weights at 5.5 TB/s; ties, several tiles below that
// line, go to the least time of the rounds.  Rounds over the whole chip let 20
// panel groups pass for one where four XCDs had 36 workgroups for 32 compute
// units (13B O and down at 144 rows 48 and 97 us, now 39 and 55; 880 rows 150
// and 363, now 89 and 199); ties to the first tile listed took the 33B LM head
// at 33 rows 97 us (now 77).  cap_floats: the published values that fit the workspace; fixed_rt > 0: that tile (with fixed_p);
// fixed_ks > 0: that many splits (one where they do not fit).
TileChoice tile_choice(int kind, int M, int n_units, int NKB, int n_cu, int fixed_rt, int fixed_p, int fixed_ks,
                       size_t cap_floats) {
  const int tiles = (M + 15) / 16;
  const int xcd_cu = std::max(1, n_cu / 8);
  TileChoice best{2, 2, 1, -1.0};
  double best_cu = 0.0;
  for (const TileCost& t : kTileCosts) {
    if (fixed_rt > 0 && (t.rt != fixed_rt || t.p != fixed_p)) continue;
    const int nug = gemm_tile_unit_groups(n_units, t.p), nrg = gemm_tile_row_groups(M, t.rt);
    for (int ks = 1; ks <= 8; ++ks) {
      if (kind == GEMM_LM ? ks > 1 : (fixed_ks > 0 && ks != fixed_ks)) continue;
      const double item = ks > 1 ? (double)nug * tile_item_floats(tiles, t.p) : 0.0;
      if (item > (double)cap_floats) continue;
      int longest = 0, slots = 1;
      for (int s = 0; s < ks; ++s) {
        longest = std::max(longest, NKB * (8 * (s + 1) / ks) / 8 - NKB * (8 * s / ks) / 8);
        if (s > 0) slots += 8 * (s + 1) / ks - 8 * s / ks;
      }
      const long rounds = ((long)((nug + 7) / 8) * nrg * ks + xcd_cu - 1) / xcd_cu;
      const double cu = rounds * (longest * 8 * t.slice_us + 2.0);
      double us = std::max(cu, (double)n_units * NKB * 8192.0 / 5.5e6) + 3.0;
      if (ks > 1) us += 5.0 + item * 4.0 / 8.0 * slots * 2.0 / 8e6;
      if (best.us < 0 || us < best.us - 1e-9 || (us <= best.us + 1e-9 && cu < best_cu - 1e-9)) {
        best = TileChoice{t.rt, t.p, ks, us};
        best_cu = cu;
      }
    }
  }
  if (best.us < 0) return tile_choice(kind, M, n_units, NKB, n_cu, fixed_rt, fixed_p, 1, cap_floats);
  return best;
}

// Published floats that one 256-column panel group of a k-split launch of
// 144 rows needs (the workspace's unit of tile_part).
size_t tile_split_floats() { return tile_item_floats(9, 2); }

hipError_t launch_tile(int kind, const GemmParams& gp, const TileChoice& c, float* part, hipStream_t st) {
  switch (kind) {
    case GEMM_QKV: return launch_tile_kind<GEMM_QKV>(gp, c, part, st);
    case GEMM_O: return launch_tile_kind<GEMM_O>(gp, c, part, st);
    case GEMM_GU: return launch_tile_kind<GEMM_GU>(gp, c, part, st);
    case GEMM_DOWN: return launch_tile_kind<GEMM_DOWN>(gp, c, part, st);
    default: return launch_tile_kind<GEMM_LM>(gp, c, part, st);
  }
}

}  // namespace spade
