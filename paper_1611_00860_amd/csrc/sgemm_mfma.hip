// Single-launch MFMA lowerings of the sgemm dataflow graph for CDNA4 (gfx950):
// one kernel launch per SgemmRoot instance, one workgroup per SgemmInternal
// instance (the main loops live in mfma_f32.hpp and mfma_bf16.hpp).
//
// The dynamic instances of SgemmInternal are independent (HPVM report,
// Sec. 2.1), so the tiles may run in any order; the order chosen keeps the
// tiles in flight on one XCD close together so that they share its L2.
#include <algorithm>

#include "device_common.hpp"
#include "internal.hpp"
#include "mfma_f32_any.hpp"
#include "mfma_f32_dma.hpp"
#include "mfma_bf16.hpp"
#include "mfma_bf16_any.hpp"
#include "mfma_bf16_dma.hpp"
#include "mfma_f32.hpp"

namespace hpvm {

// FP32 kernel: v_mfma_f32_32x32x2f32, FP32 operands and accumulation.  The
// register-staged loop remains for the products the DMA-fed one does not
// take (f32_any_fits): an operand of 1 to 3 columns, rows 2^22 floats or
// more apart, or a contraction deeper than kAnyDepth.
template <int TM, int TN, int TK, int WM, int WN, bool AT, bool BT>
__global__ void __launch_bounds__((TM / WM) * (TN / WN) * kWave) sgemm_mfma_f32(GemmArgs p) {
  extern __shared__ __align__(16) float lds[];
  int tm, tn;
  tile_coords(p.tiles_m, p.tiles_n, blockIdx.x, tm, tn);
  f32x16 acc[WM / 32][WN / 32];
  f32_mainloop<TM, TN, TK, WM, WN, AT, BT>(p, tm * TM, tn * TN, lds, acc);
  const int wave = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
  store_c<WM / 32, WN / 32>(p, acc, tm * TM + (wave / (TN / WN)) * WM,
                            tn * TN + (wave % (TN / WN)) * WN, lane);
}

// BF16 kernel (X3 = false) and bf16x3 kernel (X3 = true), register-staged:
// as the FP32 one, for what the DMA-fed loop does not take, and one bf16x3
// tile (Bf16x3WideConfig).
template <int TM, int TN, int TK, int WM, int WN, bool AT, bool BT, bool X3>
__global__ void __launch_bounds__((TM / WM) * (TN / WN) * kWave)
    sgemm_mfma_bf16(GemmArgs p) {
  extern __shared__ __align__(16) char smem[];
  int tm, tn;
  tile_coords(p.tiles_m, p.tiles_n, blockIdx.x, tm, tn);
  f32x16 acc[WM / 32][WN / 32];
  bf16_mainloop<TM, TN, TK, WM, WN, AT, BT, X3>(p, tm * TM, tn * TN, smem, acc);
  const int wave = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
  store_c<WM / 32, WN / 32>(p, acc, tm * TM + (wave / (TN / WN)) * WM,
                            tn * TN + (wave % (TN / WN)) * WN, lane);
}

// Dynamic LDS beyond 64 KiB must be enabled per kernel before its launch.
template <typename Kernel>
static hipError_t allow_lds(Kernel* fn, size_t bytes) {
  if (bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

template <int TM, int TN, int TK, int WM, int WN>
struct F32Config {
  static constexpr int kThreads = (TM / WM) * (TN / WN) * kWave;
  // LDS bytes for the given operand forms (the Allocation node's size).
  static constexpr int64_t lds(bool at, bool bt) {
    return at ? F32Tile<TM, TN, TK, WM, WN, true, false>::kLdsBytes
              : bt ? F32Tile<TM, TN, TK, WM, WN, false, true>::kLdsBytes
                   : F32Tile<TM, TN, TK, WM, WN, false, false>::kLdsBytes;
  }
  static hipError_t launch(const GemmArgs& args, bool at, bool bt, hipStream_t s) {
    GemmArgs a = args;
    a.tiles_m = (a.m + TM - 1) / TM;
    a.tiles_n = (a.n + TN - 1) / TN;
    const dim3 grid((unsigned)(a.tiles_m * a.tiles_n));
    void* kargs[] = {&a};
    void (*fn)(GemmArgs);
    if (!at && !bt) fn = &sgemm_mfma_f32<TM, TN, TK, WM, WN, false, false>;
    else if (at && !bt) fn = &sgemm_mfma_f32<TM, TN, TK, WM, WN, true, false>;
    else if (!at && bt) fn = &sgemm_mfma_f32<TM, TN, TK, WM, WN, false, true>;
    else return hipErrorInvalidValue;
    const size_t bytes = (size_t)lds(at, bt);
    hipError_t e = allow_lds(fn, bytes);
    if (e != hipSuccess) return e;
    return hipLaunchKernel(reinterpret_cast<const void*>(fn), grid, dim3(kThreads), kargs, bytes, s);
  }
};

template <int TM, int TN, int TK, int WM, int WN, bool X3>
struct Bf16Config {
  static constexpr int kThreads = (TM / WM) * (TN / WN) * kWave;
  static constexpr int64_t lds(bool, bool) { return Bf16TileShape<TM, TN, TK, WM, WN, X3>::kLdsBytes; }
  static hipError_t launch(const GemmArgs& args, bool at, bool bt, hipStream_t s) {
    void (*fn)(GemmArgs);
    if (!at && !bt) fn = &sgemm_mfma_bf16<TM, TN, TK, WM, WN, false, false, X3>;
    else if (at && !bt) fn = &sgemm_mfma_bf16<TM, TN, TK, WM, WN, true, false, X3>;
    else if (!at && bt) fn = &sgemm_mfma_bf16<TM, TN, TK, WM, WN, false, true, X3>;
    else return hipErrorInvalidValue;
    return launch_fn(fn, args, s);
  }
  static hipError_t launch_plain(const GemmArgs& args, hipStream_t s) {
    return launch_fn(&sgemm_mfma_bf16<TM, TN, TK, WM, WN, false, false, X3>, args, s);
  }
  static hipError_t launch_fn(void (*fn)(GemmArgs), const GemmArgs& args, hipStream_t s) {
    GemmArgs a = args;
    a.tiles_m = (a.m + TM - 1) / TM;
    a.tiles_n = (a.n + TN - 1) / TN;
    const dim3 grid((unsigned)(a.tiles_m * a.tiles_n));
    void* kargs[] = {&a};
    const size_t bytes = (size_t)lds(false, false);
    hipError_t e = allow_lds(fn, bytes);
    if (e != hipSuccess) return e;
    return hipLaunchKernel(reinterpret_cast<const void*>(fn), grid, dim3(kThreads), kargs, bytes, s);
  }
};

// The DMA-fed loops for any size and alignment (mfma_f32_any.hpp,
// mfma_bf16_any.hpp): TK deep sub-slabs, KW of them per slab, NST stages.  In
// tiles of KW k groups a wave computes a WM x WN block of its group and, after
// the groups' sum, owns WM / KW of its rows.  They replaced register-staged
// loops of the same tiles, which loaded one slab ahead (and element by
// element where an operand was not 16-byte aligned) and waited a memory
// round trip for nearly every slab: 1000 x 1003 x 777, 64 x 64 tiles, 21.6 us
// against 56; 512 x 4096 x 1024 38.5 against 47 (54 under a profiler); BF16
// 1500 x 1100 x 900, 64 x 128 tiles, 17.7 against 30.6.
template <int PREC, int TM, int TN, int TK, int WM, int WN, int NST, int KW>
struct AnyConfig {
  using Shape = AnyShape<TM, TN, TK, WM, WN, false, false, NST, KW>;
  static constexpr int kThreads = Shape::kThreads;
  static constexpr int64_t kLdsBytes = Shape::kLdsBytes;
  template <int MODE>
  static hipError_t run(const GemmArgs& args, int splits, hipStream_t s) {
    GemmArgs a = args;
    a.tiles_m = (a.m + TM - 1) / TM;
    a.tiles_n = (a.n + TN - 1) / TN;
    F32DmaOut o{};
    o.splits = splits;
    void* kargs[] = {&a, &o};
    void (*fn)(GemmArgs, F32DmaOut);
    if constexpr (PREC == HPVM_PREC_FP32) fn = &sgemm_f32_any<TM, TN, TK, WM, WN, false, false, NST, KW, MODE>;
    else fn = &sgemm_bf16_any<TM, TN, TK, WM, WN, false, false, NST, KW, PREC == HPVM_PREC_BF16X3, MODE>;
    hipError_t e = allow_lds(fn, (size_t)kLdsBytes);
    if (e != hipSuccess) return e;
    return hipLaunchKernel(reinterpret_cast<const void*>(fn), dim3((unsigned)(a.tiles_m * a.tiles_n * splits)),
                           dim3(kThreads), kargs, (size_t)kLdsBytes, s);
  }
  static hipError_t launch(const GemmArgs& a, bool at, bool bt, hipStream_t s) {
    // Transposed operands come from the backward only, which gives this entry what
    // its own launch of both products leaves out.
    if (!at && !bt && f32_any_fits(a, false, false)) return run<kDmaUpdate>(a, 1, s);
    if constexpr (PREC == HPVM_PREC_FP32) return F32Config<64, 64, 16, 32, 32>::launch(a, at, bt, s);
    else return Bf16Config<64, 64, 32, 32, 32, PREC == HPVM_PREC_BF16X3>::launch(a, at, bt, s);
  }
  // Contraction slices of a product whose tiles would leave CUs idle (any
  // sizes): doubled while they would, each at least 256 deep, at most 16.
  // FP32, 32 x 32 tiles: up to one workgroup a CU, from k = 2048 on, where
  // the shorter slices save more than the summing launch costs, about 5 us
  // (16 x 4096 x 4096: 128 tiles, 27 us whole, 16 in two slices;
  // 64 x 64 x 4096: 4 tiles, 25 us whole, 7 in 16 slices).  BF16 and bf16x3,
  // 32 x 128 tiles: up to two a CU, from k = 1024 on (16 x 4096 x 4096: 32
  // tiles, 40 us whole, 15.4 in eight or sixteen slices).
  static int splits(int64_t m, int64_t n, int64_t k) {
    constexpr bool f32 = PREC == HPVM_PREC_FP32;
    if (m <= 0 || n < 4 || k < (f32 ? 2048 : 1024)) return 1;
    const int64_t tiles = ((m + TM - 1) / TM) * ((n + TN - 1) / TN);
    int sp = 1;
    while (sp < 16 && tiles * sp < (f32 ? 256 : 512) && k / (2 * sp) >= 256) sp *= 2;
    return sp;
  }
  static int64_t split_bytes(int64_t m, int64_t n, int64_t k) {
    const int sp = splits(m, n, k);
    return sp > 1 ? (int64_t)sp * m * n * (int64_t)sizeof(float) : 0;
  }
  static hipError_t launch_split(const GemmArgs& args, void* workspace, hipStream_t s) {
    const int sp = splits(args.m, args.n, args.k);
    if (sp <= 1 || !f32_any_fits(args, false, false)) return launch(args, false, false, s);
    float* part = static_cast<float*>(workspace);
    GemmArgs a = args;
    a.C = part;
    a.ldc = a.n;
    a.beta = 0.0f;
    hipError_t e = run<kDmaSplit>(a, sp, s);
    if (e != hipSuccess) return e;
    return launch_split_finish(part, sp, args, s);
  }
};

#define HPVM_F32_ENTRY(TM, TN, TK, WM, WN, SUB, NST, KW)                                                \
  {{TM, TN, TK, WM / KW, WN, 2}, HPVM_PREC_FP32, AnyConfig<HPVM_PREC_FP32, TM, TN, SUB, WM, WN, NST, KW>::kThreads,       \
   AnyConfig<HPVM_PREC_FP32, TM, TN, SUB, WM, WN, NST, KW>::kLdsBytes, &AnyConfig<HPVM_PREC_FP32, TM, TN, SUB, WM, WN, NST, KW>::launch}

// C <- alpha * (slice 0 + ... + slice splits-1) + beta * C, the slices
// summed in order, from partial sums [splits][m][n]; beta == 0 never reads
// C.  A lane takes four adjacent outputs of a row (fewer at its end); rows
// may start at any float.
constexpr int kSplitThreads = 256;
__global__ void __launch_bounds__(kSplitThreads)
    sgemm_split_finish(const float* __restrict__ part, int32_t splits, GemmArgs a) {
  const int64_t m = a.m, n = a.n, ldc = a.ldc, ldci = a.ldci;
  const float alpha = a.alpha, beta = a.beta;
  float* C = a.C;
  const float* cin = a.Cin;
  using Vec = LooseF<4>::type;
  const int64_t c4 = (n + 3) / 4, units = m * c4, plane = m * n;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < units; u += stride) {
    const int64_t i = u / c4, j = (u - i * c4) * 4;
    const float* p = part + i * n + j;
    float* c = C + i * ldc + j;
    const float* o = cin + i * ldci + j;
    if (j + 4 <= n) {
      Vec v = *reinterpret_cast<const Vec*>(p);
      for (int z = 1; z < splits; ++z) v += *reinterpret_cast<const Vec*>(p + z * plane);
      if (beta != 0.0f) {
        const Vec old = *reinterpret_cast<const Vec*>(o);
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = fmaf(beta, old[t], alpha * v[t]);
      } else {
        v = alpha * v;
      }
      *reinterpret_cast<Vec*>(c) = v;
    } else {
      for (int t = 0; j + t < n; ++t) {
        float v = p[t];
        for (int z = 1; z < splits; ++z) v += p[z * plane + t];
        v *= alpha;
        c[t] = beta != 0.0f ? fmaf(beta, o[t], v) : v;
      }
    }
  }
}

hipError_t launch_split_finish(const float* part, int32_t splits, const GemmArgs& a, hipStream_t s) {
  GemmArgs args = a;
  const int64_t units = (int64_t)a.m * ((a.n + 3) / 4);
  const unsigned blocks = (unsigned)std::min<int64_t>(2048, (units + kSplitThreads - 1) / kSplitThreads);
  void* fargs[] = {&part, &splits, &args};
  return hipLaunchKernel(reinterpret_cast<const void*>(&sgemm_split_finish), dim3(blocks), dim3(kSplitThreads),
                         fargs, 0, s);
}

// FP32 problems of at least one tile each way with k a multiple of the
// slab, n a multiple of 4, every row 16-byte aligned and no transposed
// operand take the DMA-fed loop of mfma_f32_dma.hpp (edge tiles moved
// inward) with 128-wide wave tiles; any other problem the loop for any size
// with 64 x 128 tiles, the fastest there (4097 x 4099 x 2001: 535 us against
// 545 for 64 x 64 tiles and 609 for the best larger one, 3001 x 2999 x 1001:
// 159 against 155 and 169).
template <int TM, int TN, int TK, int WM, int NST>
struct F32DmaConfig {
  using S = F32DmaShape<TM, TN, TK, WM, 128, false, false, NST>;
  static constexpr int kThreads = S::NW * kWave;
  static hipError_t launch(const GemmArgs& args, bool at, bool bt, hipStream_t s) {
    if (at || bt || !f32_dma_fits_edges<TM, TN, TK>(args, args.C, args.ldc))
      return AnyConfig<HPVM_PREC_FP32, 64, 128, 32, 32, 64, 2, 1>::launch(args, at, bt, s);
    GemmArgs a = args;
    a.tiles_m = (a.m + TM - 1) / TM;
    a.tiles_n = (a.n + TN - 1) / TN;
    GemmArgs unused = a;
    F32DmaOut o{};
    o.splits = 1;
    void* kargs[] = {&a, &unused, &o};
    // Whole tiles take the kernel without edge masks.
    auto* fn = f32_dma_fits<TM, TN, TK>(args, args.C, args.ldc, 1)
                   ? &sgemm_f32_dma<TM, TN, TK, WM, 128, false, false, NST, kDmaUpdate>
                   : &sgemm_f32_dma<TM, TN, TK, WM, 128, false, false, NST, kDmaUpdate, 0, false, true>;
    hipError_t e = allow_lds(fn, (size_t)S::kLdsBytes);
    if (e != hipSuccess) return e;
    return hipLaunchKernel(reinterpret_cast<const void*>(fn), dim3((unsigned)(a.tiles_m * a.tiles_n)),
                           dim3(kThreads), kargs, (size_t)S::kLdsBytes, s);
  }
  // Contraction slices for a whole-tile problem whose tiles would not cover
  // 256 CUs: doubled while they would not, each slice a whole number of
  // slabs and at least 256 deep, at most 16; 1 (no split) when the slices
  // still would not cover them.
  static int splits(int64_t m, int64_t n, int64_t k) {
    if (m <= 0 || n <= 0 || k <= 0 || m % TM || n % TN || k % TK) return 1;
    return dma_split_count((m / TM) * (n / TN), k, TK);
  }
  static int64_t split_bytes(int64_t m, int64_t n, int64_t k) {
    const int sp = splits(m, n, k);
    return sp > 1 ? (int64_t)sp * m * n * (int64_t)sizeof(float) : 0;
  }
  // The slices write raw partial tiles to `workspace` (split_bytes of it,
  // 16-byte aligned), then sgemm_split_finish forms C.  Problems the split
  // does not cover (operands or C not 16-byte units) take launch().
  static hipError_t launch_split(const GemmArgs& args, void* workspace, hipStream_t s) {
    const int sp = splits(args.m, args.n, args.k);
    float* part = static_cast<float*>(workspace);
    if (sp <= 1 || !f32_dma_fits<TM, TN, TK>(args, part, args.n, sp) ||
        !f32_dma_fits<TM, TN, TK>(args, args.C, args.ldc, sp))
      return launch(args, false, false, s);
    GemmArgs a = args;
    a.C = part;
    a.ldc = a.n;
    a.beta = 0.0f;
    a.tiles_m = a.m / TM;
    a.tiles_n = a.n / TN;
    GemmArgs unused = a;
    F32DmaOut o{};
    o.splits = sp;
    void* kargs[] = {&a, &unused, &o};
    auto* fn = &sgemm_f32_dma<TM, TN, TK, WM, 128, false, false, NST, kDmaSplit>;
    hipError_t e = allow_lds(fn, (size_t)S::kLdsBytes);
    if (e != hipSuccess) return e;
    e = hipLaunchKernel(reinterpret_cast<const void*>(fn), dim3((unsigned)(a.tiles_m * a.tiles_n * sp)),
                        dim3(kThreads), kargs, (size_t)S::kLdsBytes, s);
    if (e != hipSuccess) return e;
    return launch_split_finish(part, sp, args, s);
  }
};

#define HPVM_F32_DMA_ENTRY(TM, TN, TK, WM, NST)                                                   \
  {{TM, TN, TK, WM, 128, NST},                                                                    \
   HPVM_PREC_FP32,                                                                                \
   F32DmaConfig<TM, TN, TK, WM, NST>::kThreads,                                                   \
   F32DmaConfig<TM, TN, TK, WM, NST>::S::kLdsBytes,                                               \
   &F32DmaConfig<TM, TN, TK, WM, NST>::launch,                                                    \
   nullptr,                                                                                       \
   nullptr,                                                                                       \
   nullptr,                                                                                       \
   &F32DmaConfig<TM, TN, TK, WM, NST>::split_bytes,                                               \
   &F32DmaConfig<TM, TN, TK, WM, NST>::launch_split}

#define HPVM_F32_SPLIT_ENTRY(TM, TN, TK, WM, WN, SUB, NST, KW)                                          \
  {{TM, TN, TK, WM / KW, WN, 2}, HPVM_PREC_FP32, AnyConfig<HPVM_PREC_FP32, TM, TN, SUB, WM, WN, NST, KW>::kThreads,  \
   AnyConfig<HPVM_PREC_FP32, TM, TN, SUB, WM, WN, NST, KW>::kLdsBytes, &AnyConfig<HPVM_PREC_FP32, TM, TN, SUB, WM, WN, NST, KW>::launch, \
   nullptr, nullptr, nullptr, &AnyConfig<HPVM_PREC_FP32, TM, TN, SUB, WM, WN, NST, KW>::split_bytes,                  \
   &AnyConfig<HPVM_PREC_FP32, TM, TN, SUB, WM, WN, NST, KW>::launch_split}

// Entry 0 is the default for large problems.  The stages of the entries on
// the loop for any size: 24 to 64 KB of slabs, alike in time however they
// are cut (64 x 64 tiles at 1000 x 1003 x 777: two 32-deep slabs 21.9 us,
// four 16-deep 22.4, six 22.4; in two k groups 20.9 and 19.7).  The autotuner
// times in this order, twice: the large tiles end it, so that a slow tile's
// rest does not come before entry 0 (with the 32 x 32 tile last, 3 of 6 tunings
// of 4096^3 and 8192 x 4096 x 2048 took a 128-wide tile, 2% slower).
static const MfmaEntry kF32Menu[] = {
    HPVM_F32_DMA_ENTRY(256, 256, 32, 64, 2),
    HPVM_F32_ENTRY(128, 128, 16, 64, 64, 16, 4, 1),
    HPVM_F32_ENTRY(256, 128, 16, 128, 64, 16, 3, 1),
    HPVM_F32_ENTRY(128, 128, 32, 64, 64, 32, 2, 1),
    HPVM_F32_ENTRY(64, 64, 16, 32, 32, 16, 6, 1),
    HPVM_F32_ENTRY(128, 64, 16, 64, 32, 16, 4, 1),
    HPVM_F32_ENTRY(64, 128, 16, 32, 64, 16, 4, 1),
    HPVM_F32_ENTRY(64, 128, 32, 32, 64, 32, 2, 1),
    HPVM_F32_ENTRY(64, 64, 32, 32, 32, 16, 3, 2),
    HPVM_F32_SPLIT_ENTRY(32, 32, 128, 32, 32, 32, 2, 4),
    HPVM_F32_DMA_ENTRY(256, 256, 16, 64, 4),
    HPVM_F32_DMA_ENTRY(128, 256, 32, 32, 2),
    HPVM_F32_DMA_ENTRY(128, 128, 32, 32, 2),
};

// BF16 and bf16x3 entries on the loop for any size.
#define HPVM_BF16_ENTRY(PREC, TM, TN, TK, WM, WN, SUB, NST)                                               \
  {{TM, TN, TK, WM, WN, 2}, PREC, AnyConfig<PREC, TM, TN, SUB, WM, WN, NST, 1>::kThreads,                 \
   AnyConfig<PREC, TM, TN, SUB, WM, WN, NST, 1>::kLdsBytes, &AnyConfig<PREC, TM, TN, SUB, WM, WN, NST, 1>::launch}
// bf16x3's 256 x 256 tile of eight 128 x 64 waves: the converted slab's hi
// and lo parts do not fit 256 registers beside the accumulators, so aligned
// operands keep the register-staged loop (2048^3: 204 us against 245; with
// scalar loads it takes 233 against 146 at 3001 x 2999 x 1001).
struct Bf16x3WideConfig {
  using Any = AnyConfig<HPVM_PREC_BF16X3, 256, 256, 16, 128, 64, 2, 1>;
  static hipError_t launch(const GemmArgs& a, bool at, bool bt, hipStream_t s) {
    return a.vec_a && a.vec_b && !at && !bt ? Bf16Config<256, 256, 32, 128, 64, true>::launch_plain(a, s)
                                            : Any::launch(a, at, bt, s);
  }
};
#define HPVM_BF16_SPLIT_ENTRY(PREC, TM, TN, TK, WM, WN, SUB, NST)                                         \
  {{TM, TN, TK, WM, WN, 2}, PREC, AnyConfig<PREC, TM, TN, SUB, WM, WN, NST, 1>::kThreads,                 \
   AnyConfig<PREC, TM, TN, SUB, WM, WN, NST, 1>::kLdsBytes, &AnyConfig<PREC, TM, TN, SUB, WM, WN, NST, 1>::launch, \
   nullptr, nullptr, nullptr, &AnyConfig<PREC, TM, TN, SUB, WM, WN, NST, 1>::split_bytes,                  \
   &AnyConfig<PREC, TM, TN, SUB, WM, WN, NST, 1>::launch_split}

// BF16 / bf16x3 products on the FP32 DMA-fed loop (mfma_bf16_dma.hpp):
// problems of at least one tile each way with k a multiple of the slab, n a
// multiple of 4 and 16-byte rows, no transposed operand (edge tiles moved
// inward as in the FP32 loop); any other problem takes the loop for any
// size, on 128 x 256 tiles (64 x 128 for the 128 x 128 entry).  The split
// contraction is the FP32 entries' (same slice rule, same ordered sum).
template <int TM, int TN, int TK, int WM, int WN, int NST, bool X3>
struct Bf16SrcConfig {
  using S = Bf16SrcShape<TM, TN, TK, WM, WN, false, false, NST>;
  static constexpr int kPrec = X3 ? HPVM_PREC_BF16X3 : HPVM_PREC_BF16;
  using Other = typename std::conditional<(TM > 128), AnyConfig<kPrec, 128, 256, 32, 64, 64, 3, 1>,
                                          AnyConfig<kPrec, 64, 128, 32, 32, 64, 3, 1>>::type;
  static constexpr int kThreads = S::NW * kWave;
  static hipError_t launch(const GemmArgs& args, bool at, bool bt, hipStream_t s) {
    if (at || bt || !f32_dma_fits_edges<TM, TN, TK>(args, args.C, args.ldc))
      return Other::launch(args, at, bt, s);
    GemmArgs a = args;
    a.tiles_m = (a.m + TM - 1) / TM;
    a.tiles_n = (a.n + TN - 1) / TN;
    F32DmaOut o{};
    o.splits = 1;
    void* kargs[] = {&a, &o};
    auto* fn = f32_dma_fits<TM, TN, TK>(args, args.C, args.ldc, 1)
                   ? &sgemm_bf16src_dma<TM, TN, TK, WM, WN, false, false, NST, X3, kDmaUpdate>
                   : &sgemm_bf16src_dma<TM, TN, TK, WM, WN, false, false, NST, X3, kDmaUpdate, true>;
    hipError_t e = allow_lds(fn, (size_t)S::kLdsBytes);
    if (e != hipSuccess) return e;
    return hipLaunchKernel(reinterpret_cast<const void*>(fn), dim3((unsigned)(a.tiles_m * a.tiles_n)),
                           dim3(kThreads), kargs, (size_t)S::kLdsBytes, s);
  }
  static int splits(int64_t m, int64_t n, int64_t k) {
    if (m <= 0 || n <= 0 || k <= 0 || m % TM || n % TN || k % TK) return 1;
    return dma_split_count((m / TM) * (n / TN), k, TK);
  }
  static int64_t split_bytes(int64_t m, int64_t n, int64_t k) {
    const int sp = splits(m, n, k);
    return sp > 1 ? (int64_t)sp * m * n * (int64_t)sizeof(float) : 0;
  }
  static hipError_t launch_split(const GemmArgs& args, void* workspace, hipStream_t s) {
    const int sp = splits(args.m, args.n, args.k);
    float* part = static_cast<float*>(workspace);
    if (sp <= 1 || !f32_dma_fits<TM, TN, TK>(args, part, args.n, sp) ||
        !f32_dma_fits<TM, TN, TK>(args, args.C, args.ldc, sp))
      return launch(args, false, false, s);
    GemmArgs a = args;
    a.C = part;
    a.ldc = a.n;
    a.beta = 0.0f;
    a.tiles_m = a.m / TM;
    a.tiles_n = a.n / TN;
    F32DmaOut o{};
    o.splits = sp;
    void* kargs[] = {&a, &o};
    auto* fn = &sgemm_bf16src_dma<TM, TN, TK, WM, WN, false, false, NST, X3, kDmaSplit>;
    hipError_t e = allow_lds(fn, (size_t)S::kLdsBytes);
    if (e != hipSuccess) return e;
    e = hipLaunchKernel(reinterpret_cast<const void*>(fn), dim3((unsigned)(a.tiles_m * a.tiles_n * sp)),
                        dim3(kThreads), kargs, (size_t)S::kLdsBytes, s);
    if (e != hipSuccess) return e;
    return launch_split_finish(part, sp, args, s);
  }
};

#define HPVM_BF16SRC_ENTRY(PREC, X3, TM, TN, TK, WM, WN, NST)                                    \
  {{TM, TN, TK, WM, WN, NST}, PREC, Bf16SrcConfig<TM, TN, TK, WM, WN, NST, X3>::kThreads,         \
   Bf16SrcConfig<TM, TN, TK, WM, WN, NST, X3>::S::kLdsBytes,                                       \
   &Bf16SrcConfig<TM, TN, TK, WM, WN, NST, X3>::launch,                                            \
   nullptr,                                                                                                   \
   nullptr,                                                                                                   \
   nullptr,                                                                                                   \
   &Bf16SrcConfig<TM, TN, TK, WM, WN, NST, X3>::split_bytes,                                       \
   &Bf16SrcConfig<TM, TN, TK, WM, WN, NST, X3>::launch_split}

// Entry 0 is the default for large products.
// bf16x3 takes 16-deep slabs in 4 stages first (8192^3: 2.65 ms against
// 2.87 for 32-deep slabs in 2 stages), BF16 32-deep slabs in 2 stages
// (8192^3: 1.46 ms against 1.51, 4096^3: 0.167 against 0.176; a fifth
// 16-deep stage, all 160 KB of LDS, gave 1.45).
static const MfmaEntry kBf16Menu[] = {
    HPVM_BF16SRC_ENTRY(HPVM_PREC_BF16, false, 256, 256, 32, 64, 128, 2),
    HPVM_BF16SRC_ENTRY(HPVM_PREC_BF16, false, 256, 256, 16, 64, 128, 4),
    HPVM_BF16SRC_ENTRY(HPVM_PREC_BF16, false, 128, 128, 32, 64, 64, 4),
    HPVM_BF16_ENTRY(HPVM_PREC_BF16, 256, 256, 32, 128, 64, 16, 2),
    HPVM_BF16_ENTRY(HPVM_PREC_BF16, 256, 128, 32, 128, 64, 16, 3),
    HPVM_BF16_ENTRY(HPVM_PREC_BF16, 128, 128, 32, 64, 64, 32, 2),
    HPVM_BF16_ENTRY(HPVM_PREC_BF16, 128, 128, 64, 64, 64, 32, 2),
    HPVM_BF16_ENTRY(HPVM_PREC_BF16, 64, 64, 32, 32, 32, 32, 3),
    HPVM_BF16_ENTRY(HPVM_PREC_BF16, 64, 128, 32, 32, 64, 32, 3),
    HPVM_BF16_ENTRY(HPVM_PREC_BF16, 128, 256, 32, 64, 64, 32, 3),
    HPVM_BF16_SPLIT_ENTRY(HPVM_PREC_BF16, 32, 128, 32, 32, 32, 32, 4),
};

static const MfmaEntry kBf16x3Menu[] = {
    HPVM_BF16SRC_ENTRY(HPVM_PREC_BF16X3, true, 256, 256, 16, 128, 128, 4),
    HPVM_BF16SRC_ENTRY(HPVM_PREC_BF16X3, true, 256, 256, 32, 128, 128, 2),
    HPVM_BF16SRC_ENTRY(HPVM_PREC_BF16X3, true, 128, 128, 32, 64, 64, 4),
    {{256, 256, 32, 128, 64, 2}, HPVM_PREC_BF16X3, Bf16Config<256, 256, 32, 128, 64, true>::kThreads,
     Bf16Config<256, 256, 32, 128, 64, true>::lds(false, false), &Bf16x3WideConfig::launch},
    HPVM_BF16_ENTRY(HPVM_PREC_BF16X3, 256, 128, 32, 128, 64, 16, 3),
    HPVM_BF16_ENTRY(HPVM_PREC_BF16X3, 128, 128, 32, 64, 64, 32, 2),
    HPVM_BF16_ENTRY(HPVM_PREC_BF16X3, 64, 64, 32, 32, 32, 32, 3),
    HPVM_BF16_ENTRY(HPVM_PREC_BF16X3, 64, 128, 32, 32, 64, 32, 3),
    HPVM_BF16_ENTRY(HPVM_PREC_BF16X3, 128, 256, 32, 64, 64, 32, 3),
    HPVM_BF16_SPLIT_ENTRY(HPVM_PREC_BF16X3, 32, 128, 32, 32, 32, 32, 4),
};

int mfma_menu(int32_t prec, const MfmaEntry** entries) {
  if (prec == HPVM_PREC_FP32) {
    *entries = kF32Menu;
    return (int)(sizeof(kF32Menu) / sizeof(kF32Menu[0]));
  }
  if (prec == HPVM_PREC_BF16) {
    *entries = kBf16Menu;
    return (int)(sizeof(kBf16Menu) / sizeof(kBf16Menu[0]));
  }
  if (prec == HPVM_PREC_BF16X3) {
    *entries = kBf16x3Menu;
    return (int)(sizeof(kBf16x3Menu) / sizeof(kBf16x3Menu[0]));
  }
  *entries = nullptr;
  return 0;
}

}  // namespace hpvm
