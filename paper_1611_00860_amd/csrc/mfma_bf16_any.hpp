// BF16 / bf16x3 products on FP32 storage for any size and alignment (gfx950).
//
// The feed is that of mfma_f32_any.hpp: FP32 slabs straight from HBM into a
// ring of LDS stages, the last, partial slab of k by element.  The rounding
// to bfloat16 (and bf16x3's split) happens in registers between the LDS
// reads of a step and its MFMAs, as in mfma_bf16_dma.hpp, whose order of
// products this keeps: 16-k steps in ascending k, bf16x3 as lo*hi, hi*lo,
// hi*hi -- the bits of every other lowering of the precision.
#pragma once

#include "mfma_bf16_dma.hpp"
#include "mfma_f32_any.hpp"

namespace hpvm {

// The FP32 values of one side's fragments of a 16-k step.  KC: chunks
// 4 s + 2 h and 4 s + 2 h + 1 of the lane's rows; MN: eight reads, one per k,
// of V adjacent values.
template <typename O, bool KC, int R, int TK>
struct Bf16AnySide {
  static constexpr int kBlocks = O::kBlocks, V = O::V;
  struct Values {
    float v[kBlocks][8];  // [block][slot]
  };
  __device__ __forceinline__ static void read(Values& x, const char* st, int s, int w0, int lane) {
    if constexpr (KC) {
#pragma unroll
      for (int b = 0; b < kBlocks; ++b)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const f32x4 y = *reinterpret_cast<const f32x4*>(
              st + (w0 + 32 * b) * 4 * TK + kc_chunk_off<4 * TK>(lane, 4 * s + 2 * (lane >> 5) + e));
#pragma unroll
          for (int i = 0; i < 4; ++i) x.v[b][4 * e + i] = y[i];
        }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const char* q = st + (16 * s + 8 * (lane >> 5) + j) * R * 4 + (w0 + V * (lane & 31)) * 4;
        if constexpr (V == 1) {
          x.v[0][j] = *reinterpret_cast<const float*>(q);
        } else {
          const typename VecF<V>::type y = *reinterpret_cast<const typename VecF<V>::type*>(q);
#pragma unroll
          for (int b = 0; b < V; ++b) x.v[b][j] = y[b];
        }
      }
    }
  }
};

// A step is a whole sub-slab: all its fragments are read at once, under the
// previous sub-slab's MFMAs, then converted behind them into the one set of
// operands.  (By 16-k steps, a wave alone on its SIMD waited for LDS twice
// per sub-slab: 1000 x 1003 x 777, 64 x 64 tiles, 16.4 us.)
template <typename S, bool X3>
struct MathBf16 {
  using OA = typename S::OA;
  using OB = typename S::OB;
  using SideA = Bf16AnySide<OA, !S::kAt, S::kTm, S::kTk>;
  using SideB = Bf16AnySide<OB, S::kBt, S::kTn, S::kTk>;
  static constexpr int NA = OA::kBlocks, NB = OB::kBlocks, kSteps = 1, KS = S::kTk / 16, P = X3 ? 2 : 1;
  f32x16 acc[NA][NB];
  typename SideA::Values ra[KS];
  typename SideB::Values rb[KS];
  u32x4 ca[KS][P][NA], cb[KS][P][NB];  // converted: [16-k step][hi, lo][block]
  int wm0, wn0, lane;

  __device__ __forceinline__ MathBf16(int wm, int wn, int ln) : wm0(wm), wn0(wn), lane(ln) { zero_acc(acc); }
  __device__ __forceinline__ void read(int, const char* st, int) {
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      SideB::read(rb[s], st + OA::kBytes, s, wn0, lane);
      SideA::read(ra[s], st, s, wm0, lane);
    }
  }
  __device__ __forceinline__ static void convert_block(const float (&v)[8], u32x4& hi, u32x4* lo) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t h = bf16_pair(v[2 * q], v[2 * q + 1]);
      hi[q] = h;
      if constexpr (X3) (*lo)[q] = bf16_lo_pair(v[2 * q], v[2 * q + 1], h);
    }
  }
  __device__ __forceinline__ void first() {
#pragma unroll
    for (int s = 0; s < KS; ++s) {
#pragma unroll
      for (int b = 0; b < NB; ++b) convert_block(rb[s].v[b], cb[s][0][b], &cb[s][P - 1][b]);
#pragma unroll
      for (int a = 0; a < NA; ++a) convert_block(ra[s].v[a], ca[s][0][a], &ca[s][P - 1][a]);
    }
  }
  // Multiplies the converted sub-slab, then converts the one read meanwhile.
  __device__ __forceinline__ void multiply(int) {
    __builtin_amdgcn_sched_barrier(0);
    auto op = [](const u32x4& v) { return __builtin_bit_cast(bf16x8, v); };
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      if constexpr (X3) {
#pragma unroll
        for (int a = 0; a < NA; ++a)
#pragma unroll
          for (int b = 0; b < NB; ++b) {
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op(ca[s][P - 1][a]), op(cb[s][0][b]), acc[a][b], 0, 0,
                                                                0);
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op(ca[s][0][a]), op(cb[s][P - 1][b]), acc[a][b], 0, 0,
                                                                0);
          }
      }
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op(ca[s][0][a]), op(cb[s][0][b]), acc[a][b], 0, 0, 0);
    }
    first();
  }
};

// The smaller waves keep to a third of a SIMD's registers (see
// F32DmaShape::kMinWaves); bf16x3's hi and lo parts leave that to 32 x 32.
template <int WM, int WN, bool X3>
constexpr int kBf16AnyMinWaves = WM * WN <= (X3 ? 32 * 32 : 32 * 64) ? 3 : 1;

// One launch: a workgroup per tile and contraction slice (slice-major),
// XCD-aware tile order.
template <int TM, int TN, int TK, int WM, int WN, bool AT, bool BT, int NST, int KW, bool X3, int MODE>
__global__ void __launch_bounds__((AnyShape<TM, TN, TK, WM, WN, AT, BT, NST, KW>::kThreads))
    __attribute__((amdgpu_waves_per_eu(kBf16AnyMinWaves<WM, WN, X3>))) sgemm_bf16_any(GemmArgs p, F32DmaOut o) {
  extern __shared__ __align__(16) char smem[];
  read_early(p);
  using S = AnyShape<TM, TN, TK, WM, WN, AT, BT, NST, KW>;
  const int tiles = p.tiles_m * p.tiles_n;
  const int z = blockIdx.x / tiles;
  int tm, tn;
  tile_coords(p.tiles_m, p.tiles_n, blockIdx.x - z * tiles, tm, tn);
  any_tile<S, MathBf16<S, X3>>(p, o.splits, tm, tn, z, smem,
                               [&](const auto& acc, int m0, int n0, int m_own, int n_own, bool whole, int wm0,
                                   int wn0, int lane, int q0, int q1) {
                                 any_epilogue<typename S::OA, typename S::OB, BT, MODE>(
                                     p, o, acc, m0, n0, m_own, n_own, whole, wm0, wn0, lane, z, q0, q1);
                               });
}

}  // namespace hpvm
