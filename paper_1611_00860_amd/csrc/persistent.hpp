// Pieces shared by the two persistent lowerings of the sgemm graph: grouped
// batches (many graphs, one launch) and the streaming graph (argument packs
// pushed while the kernel runs).
//
// Both keep a fixed set of resident workgroups that pull SgemmInternal
// instances (tiles) from a device-side counter -- the persistent-node form
// of Sec. 3.5 -- and both let every sgemm carry its own tile shape, chosen
// from a menu whose shapes share one workgroup size and one LDS size so a
// single kernel can run any of them.
#pragma once

#include <cmath>
#include <cstdint>

#include "device_common.hpp"
#include "host_common.hpp"
#include "hpvm_sgemm.h"
#include "mfma_f32.hpp"
#include "mfma_f32_any.hpp"

namespace hpvm {

struct GroupedShape {
  hpvm_tile tile;
  double cost_per_flop;  // relative cost of a useful flop, for the cost model
  double start;          // a tile's fixed time, in steps of k
};

// The shapes a persistent kernel can run: all use 256 lanes (4 waves).  Fixed
// times from batches of one size on one shape, 768 resident workgroups,
// 512 x 512 x 512 against 512 x 512 x 64: 14, 8.5, 8.5 and 6.5 us a tile.
// Costs per flop: alike within 10% for the three larger shapes there, but a
// batch of 512 log-uniform sgemms gains from larger tiles (less traffic).
static const GroupedShape kGroupedShapes[] = {
    {{128, 128, 16, 64, 64, 2}, 1.00, 58.0},
    {{128, 64, 16, 64, 32, 2}, 1.08, 79.0},
    {{64, 128, 16, 32, 64, 2}, 1.05, 84.0},
    {{64, 64, 16, 32, 32, 2}, 1.30, 113.0},
};
constexpr int kNumGroupedShapes = 4;
constexpr int kGroupedThreads = 256;

// The shapes run the DMA-fed loop for any size (mfma_f32_any.hpp), 16-deep
// slabs in as many stages as the Allocation holds: 48 KB for the grouped
// launch, three workgroups a CU (128 x 128 tiles at 1024^3: 118 TFLOP/s
// against 103 in 32 KB); 36 KB for the stream, whose two resident workgroups
// leave 87 KB of a CU's LDS to the kernels that run beside it.
template <int TM, int TN, int WM, int WN, int NST>
using GroupedAny = AnyShape<TM, TN, 16, WM, WN, false, false, NST, 1>;
constexpr int64_t kGroupedLds = 49152, kStreamLds = 36864;
constexpr int kGroupedBatch = 32;  // elements of C in flight per lane, within 168 registers

template <int64_t LDS, int TM, int TN, int WM, int WN>
__device__ __forceinline__ void grouped_any_tile(const GemmArgs& p, int tm, int tn, char* smem) {
  constexpr int NST = (int)(LDS / GroupedAny<TM, TN, WM, WN, 2>::kStage);
  using S = GroupedAny<TM, TN, WM, WN, NST>;
  static_assert(S::kThreads == kGroupedThreads && S::kLdsBytes <= LDS, "256 lanes, the Allocation fits");
  f32_any_tile<TM, TN, 16, WM, WN, false, false, NST, 1>(
      p, 1, tm, tn, 0, smem,
      [&](const auto& acc, int m0, int n0, int m_own, int n_own, bool whole, int wm0, int wn0, int lane, int q0,
          int q1) {
        any_epilogue<typename S::OA, typename S::OB, false, kDmaUpdate, kGroupedBatch>(
            p, F32DmaOut{}, acc, m0, n0, m_own, n_own, whole, wm0, wn0, lane, 0, q0, q1);
      });
}

// What that loop leaves out (f32_any_fits; it does take k = 0, which the
// persistent kernels pass for alpha = 0): the tile as 64 x 64 tiles of the
// register-staged loop, one after another.
static_assert(F32Tile<64, 64, 16, 32, 32, false, false>::kLdsBytes <= kStreamLds, "LDS");
__device__ __forceinline__ void grouped_odd_tile(const GemmArgs& p, int m0, int n0, int tile_m, int tile_n,
                                                 float* lds) {
  for (int i = m0; i < m0 + tile_m && i < p.m; i += 64)
    for (int j = n0; j < n0 + tile_n && j < p.n; j += 64) {
      f32x16 acc[1][1];
      f32_mainloop<64, 64, 16, 32, 32, false, false>(p, i, j, lds, acc);
      const int wave = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
      store_c<1, 1>(p, acc, i + (wave / 2) * 32, j + (wave % 2) * 32, lane);
    }
}

// Runs tile `local` (row-major over the instance's tile grid) of one sgemm
// with menu shape `shape`, the Allocation of LDS bytes at lds.  Uniform
// across the workgroup.
template <int64_t LDS>
__device__ __forceinline__ void run_shape_tile(int shape, const GemmArgs& p, int tiles_n, int local,
                                               float* lds) {
  const int tm = local / tiles_n, tn = local - (local / tiles_n) * tiles_n;
  char* smem = reinterpret_cast<char*>(lds);
  if (p.n < 4 || p.lda >= kAnyPitch || p.ldb >= kAnyPitch || p.ldc >= kAnyPitch || p.m >= (1 << 30) ||
      p.n >= (1 << 30)) {
    const int tile_m = shape < 2 ? 128 : 64, tile_n = shape == 0 || shape == 2 ? 128 : 64;
    grouped_odd_tile(p, tm * tile_m, tn * tile_n, tile_m, tile_n, lds);
    return;
  }
  switch (shape) {
    case 0: grouped_any_tile<LDS, 128, 128, 32, 128>(p, tm, tn, smem); break;
    case 1: grouped_any_tile<LDS, 128, 64, 32, 64>(p, tm, tn, smem); break;
    case 2: grouped_any_tile<LDS, 64, 128, 32, 64>(p, tm, tn, smem); break;
    default: grouped_any_tile<LDS, 64, 64, 32, 32>(p, tm, tn, smem); break;
  }
}

// Host side ---------------------------------------------------------------

inline int64_t shape_tiles(int64_t m, int64_t n, int shape) {
  if (m == 0 || n == 0) return 0;
  const hpvm_tile& t = kGroupedShapes[shape].tile;
  return ((m + t.tile_m - 1) / t.tile_m) * ((n + t.tile_n - 1) / t.tile_n);
}

// Estimated time of one tile of depth k (in flops of the 128 x 128 shape):
// its padded flops and its fixed time, weighted by the shape's relative cost
// per flop raised to `lambda`, plus `overhead` steps of k of a 128 x 128 tile
// whatever its shape (which favours fewer, larger tiles for shallow
// instances).
inline double tile_cost(int64_t k, int shape, double lambda = 1.0, double overhead = 0.0) {
  const GroupedShape& g = kGroupedShapes[shape];
  return (double)g.tile.tile_m * g.tile.tile_n * ((double)(k > 0 ? k : 0) + g.start) *
             std::pow(g.cost_per_flop, lambda) +
         overhead * 128.0 * 128.0;
}

// Cost model: the shape whose tiles of the instance take the least time.
inline int cost_model_shape(int64_t m, int64_t n, int64_t k, double lambda, double overhead = 0.0) {
  int best = 0;
  double best_cost = 0.0;
  for (int s = 0; s < kNumGroupedShapes; ++s) {
    const double cost = (double)shape_tiles(m, n, s) * tile_cost(k, s, lambda, overhead);
    if (s == 0 || cost < best_cost) {
      best = s;
      best_cost = cost;
    }
  }
  return best;
}

}  // namespace hpvm
