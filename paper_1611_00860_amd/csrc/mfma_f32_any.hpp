// DMA-fed FP32 MFMA loop for any size and alignment (gfx950).
//
// The Allocation node is the ring of LDS stages of mfma_f32_dma.hpp, fed by
// global_load_lds_dwordx4; here nothing has to be a multiple of anything:
//   * a 16-byte transfer needs its global address aligned to 4 bytes only,
//     so rows of any leading dimension are moved as they are;
//   * an operand stored with k contiguous (KC) takes rows past the matrix
//     from its last row, and one stored with m or n contiguous (MN) moves
//     an edge tile inward to end at the edge, or, when the matrix is
//     narrower than the tile, takes columns past it from column 0: what
//     they give is never stored, and every address stays in the matrix;
//   * the last, partial slab of k (all of a short contraction) is loaded
//     element by element into registers before the first transfer, with
//     zeros outside the matrix, and written to its LDS stage when the ring
//     reaches it.  A narrow MN operand whose width is not a multiple of 4
//     has its last slab loaded that way too, since the last 16-byte unit of
//     the matrix's last row would end past the matrix.
// KW > 1 splits each slab's k over KW groups of waves, each with a sub-slab
// of TK of its own; their accumulators are added in group order through
// LDS at the end.  With KW = 1 outputs are summed over k in ascending
// order, with the slots of mfma_f32.hpp, so the bits are those of every
// other FP32 lowering.
#pragma once

#include <type_traits>

#include "device_common.hpp"
#include "hpvm_sgemm.h"
#include "lds_dma.hpp"
#include "mfma_f32.hpp"
#include "mfma_f32_dma.hpp"

namespace hpvm {

// V floats that may sit at any multiple of 4 bytes.
template <int V>
struct LooseF;
template <>
struct LooseF<1> {
  typedef float type;
};
template <>
struct LooseF<2> {
  typedef float type __attribute__((ext_vector_type(2), aligned(4)));
};
template <>
struct LooseF<4> {
  typedef float type __attribute__((ext_vector_type(4), aligned(4)));
};

// One side of the product.  R: the tile's extent on this side, W: a wave's.
template <bool KC, int R, int W, int TK>
struct AnyOperand {
  static constexpr int kBytes = R * TK * 4;  // one sub-slab
  static constexpr int kDma = kBytes / 1024;
  static constexpr int kBlocks = W / 32;
  static constexpr int V = KC ? 4 : kBlocks;      // floats per fragment read
  static constexpr int kFrags = KC ? kBlocks : 4;  // fragment reads per 8-k group
  using Rows = SwizzledRows<4 * TK>;
  static_assert(kDma * 1024 == kBytes && W % 32 == 0, "whole DMA instructions and blocks");
  static_assert(KC || (R <= 256 && (V == 1 || V == 2 || V == 4)), "MN rows of at most one instruction");
  struct Frag {
    float v[V];
  };

  // What this lane moves with instruction q: row r and first column c of
  // its 16 bytes within the sub-slab (KC: an m or n row and a k; MN: a k
  // row and an m or n).
  __device__ static void unit(int lane, int q, int& r, int& c) {
    if constexpr (KC && TK == 32) {
      const int x = (lane >> 3) ^ (q & 1);
      r = q * 8 + x;
      c = ((lane & 7) ^ x) * 4;
    } else if constexpr (KC) {
      const int y = lane >> 3, p = lane & 7, g = (y & 3) ^ ((y >> 2) & 1);
      r = q * 16 + 2 * y + ((p >> 2) & 1);
      c = ((p ^ g) & 3) * 4;
    } else {
      r = q * (256 / R) + lane / (R / 4);
      c = (lane % (R / 4)) * 4;
    }
  }
  // Byte offset of that unit from the tile's corner; `left`: rows (KC) or
  // columns (MN) of the matrix from the corner on.
  __device__ static uint32_t offset(int lane, int q, int left, int64_t ld) {
    int r, c;
    unit(lane, q, r, c);
    if constexpr (KC) r = r < left ? r : left - 1;
    else c = c < left ? c : 0;
    return (uint32_t)(((int64_t)r * ld + c) * 4);
  }
  // The unit's four values of the tail sub-slab at `base`, `depth` values
  // of k deep (<= 0: none), zero outside.
  __device__ static f32x4 tail(const char* base, int lane, int q, int left, int depth, int64_t ld) {
    int r, c;
    unit(lane, q, r, c);
    const int rows = KC ? left : depth, cols = KC ? depth : left;
    const float* p = reinterpret_cast<const float*>(base) + (int64_t)r * ld + c;
    f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
    if (r < rows) {
      if (c + 4 <= cols) {
        const typename LooseF<4>::type w = *reinterpret_cast<const typename LooseF<4>::type*>(p);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = w[e];
      } else {
#pragma unroll
        for (int e = 0; e < 3; ++e)
          if (c + e < cols) v[e] = p[e];
      }
    }
    return v;
  }
  // Fragment j (block for KC, step for MN) of the 8-k group whose chunk
  // offset is foff (KC) or number g (MN).
  __device__ static Frag frag(const char* st, int j, int g, int w0, int lane, int foff) {
    Frag f;
    if constexpr (KC) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(st + (w0 + 32 * j) * 4 * TK + foff);
#pragma unroll
      for (int e = 0; e < 4; ++e) f.v[e] = x[e];
    } else {
      const char* q = st + (8 * g + 4 * (lane >> 5) + j) * R * 4 + (w0 + V * (lane & 31)) * 4;
      if constexpr (V == 1) {
        f.v[0] = *reinterpret_cast<const float*>(q);
      } else {
        const typename VecF<V>::type x = *reinterpret_cast<const typename VecF<V>::type*>(q);
#pragma unroll
        for (int e = 0; e < V; ++e) f.v[e] = x[e];
      }
    }
    return f;
  }
  // Operand of MFMA step p for block b.
  __device__ static float pick(const Frag (&f)[kFrags], int b, int p) {
    if constexpr (KC) return f[b].v[p];
    else return f[p].v[b];
  }
  // Row or column of block b's element x for a wave starting at w0.
  __device__ static int index(int b, int x, int w0) { return KC ? w0 + 32 * b + x : w0 + V * x + b; }
  // The A side's row of accumulator register r is row(a, r, w0) (uniform)
  // plus lane_row(lane).
  __device__ static int row(int b, int r, int w0) { return index(b, acc_row(r, 0), w0); }
  __device__ static int lane_row(int lane) { return (KC ? 4 : 4 * V) * (lane >> 5); }
};

// The deepest slab, and the deepest contraction: k + kAnySlab is an int.
// (With slab_count instead of that sum the loop's code was another, and dB's
// tiles 4 to 6% slower: 4473 x 493 x 2157, dB alone 160 us against 150.)
constexpr int kAnySlab = 128, kAnyDepth = INT32_MAX - kAnySlab;

template <int TM, int TN, int TK, int WM, int WN, bool AT, bool BT, int NST, int KW>
struct AnyShape {
  using OA = AnyOperand<!AT, TM, WM, TK>;
  using OB = AnyOperand<BT, TN, WN, TK>;
  static constexpr int NWN = TN / WN, NWT = (TM / WM) * NWN, NW = NWT * KW;  // waves: per group, in all
  static constexpr int kThreads = NW * kWave;
  static constexpr int kSub = OA::kBytes + OB::kBytes, kStage = KW * kSub;
  static constexpr int64_t kLdsBytes = (int64_t)NST * kStage;
  // A group's waves move that group's sub-slab.
  static constexpr int QA = OA::kDma / NWT, QB = OB::kDma / NWT, Q = QA + QB;
  static constexpr int kSlab = KW * TK;
  // Four FP32 waves of up to 64 x 64 keep to a third of a SIMD's registers
  // (see F32DmaShape::kMinWaves), eight of 32 x 32 to a sixth.
  static constexpr int kMinWaves = WM * WN > 64 * 64 ? 1 : NW == 4 ? 3 : NW == 8 && WM * WN <= 32 * 32 ? 6 : 1;
  static constexpr int kTm = TM, kTn = TN, kTk = TK, kWm = WM, kWn = WN, kNst = NST, kKw = KW;
  static constexpr bool kAt = AT, kBt = BT;
  static_assert(TM % WM == 0 && TN % WN == 0, "wave tiles");
  static_assert(QA * NWT == OA::kDma && QB * NWT == OB::kDma, "DMA instructions split evenly over a group's waves");
  static_assert(KW == 1 || (int64_t)NW * OA::kBlocks * OB::kBlocks * 4096 <= kLdsBytes, "partials fit the ring");
  // The groups share the four row quads (with KW = 8 the first four take one each).
  static_assert(KW == 1 || KW == 2 || KW == 4 || KW == 8, "groups share the four row quads");
  static constexpr int kQuads = KW < 4 ? 4 / KW : 1;
  static_assert((NST - 1) * Q < 64, "vmcnt range");
};

// Waits until at most `slabs` whole slabs of this wave's transfers (Q
// instructions each) are outstanding and its LDS traffic is complete, then
// joins the workgroup barrier.
template <int Q, int MAX>
__device__ __forceinline__ void wait_slabs_barrier(int slabs) {
  if constexpr (MAX > 0) {
    if (slabs >= MAX) {
      dma_wait_barrier<MAX * Q>();
      return;
    }
    wait_slabs_barrier<Q, MAX - 1>(slabs);
  } else {
    dma_wait_barrier<0>();
  }
}

// Outputs of the accumulators' row quads [q0, q1) (quad g of block a: the
// rows acc_row(4 g .. 4 g + 3)).  m_own, n_own: the tile's place in the
// tile grid; only rows in [m_own, m) and columns in [n_own, n) are stored.
template <typename OA, typename OB, bool BT, int MODE, int BATCH = 32, int NA, int NB>
__device__ __forceinline__ void any_epilogue(const GemmArgs& q, const F32DmaOut& o, const f32x16 (&acc)[NA][NB],
                                             int m0, int n0, int m_own, int n_own, bool whole, int wm0, int wn0,
                                             int lane, int z, int q0, int q1) {
  const int64_t plane = (int64_t)q.m * q.ldc;
  const float* cin = q.Cin;
  const int64_t ldci = q.ldci;
  float* out = MODE == kDmaConsume ? o.D : q.C + (MODE == kDmaSplit ? z * plane : 0);
  const int64_t ldo = MODE == kDmaConsume ? o.ldd : q.ldc;
  const float alpha = MODE == kDmaSplit ? 1.0f : q.alpha;
  const bool read_c = MODE != kDmaSplit && q.beta != 0.0f;
  constexpr int V = BT ? 1 : NB;  // adjacent outputs a lane holds
  using Vec = typename LooseF<V>::type;
  const int I = lane & 31;
  // An output's address is its row's (uniform) plus the lane's 32-bit byte
  // offset, so that no address is held per row.
  const int lrow = OA::lane_row(lane);
  auto at = [](const Vec& v, int e) -> float {
    if constexpr (V == 1) return v;
    else return v[e];
  };
  auto put = [](Vec& v, int e, float x) {
    if constexpr (V == 1) v = x;
    else v[e] = x;
  };
  // Up to BATCH elements of C per lane are loaded before any of their outputs
  // is stored (see store_c).
  constexpr int kRows = BATCH / V < 16 ? BATCH / V : 16;  // of a block
  constexpr int kBatch = NA * 16 * V <= BATCH ? NA : BATCH / (16 * V) > 0 ? BATCH / (16 * V) : 1;
  auto store = [&](auto all) {
    constexpr bool kAll = decltype(all)::value;  // the tile owns all its outputs
#pragma unroll
    for (int b0 = 0; b0 < NB; b0 += V) {
      const int col = n0 + OB::index(b0, I, wn0);
      const uint32_t coff = (uint32_t)((lrow * ldci + col) * 4), ooff = (uint32_t)((lrow * ldo + col) * 4);
      Vec bias{};
      if constexpr (MODE == kDmaConsume) {
        if (o.op == HPVM_CONSUMER_BIAS || o.op == HPVM_CONSUMER_BIAS_RELU) {
#pragma unroll
          for (int e = 0; e < V; ++e) put(bias, e, col + e < q.n ? o.bias[col + e] : 0.0f);
        }
      }
#pragma unroll
      for (int ar = 0; ar < NA * 16; ar += kBatch * kRows) {
        const int a0 = ar / 16, r0 = ar % 16;
        Vec c[kBatch][kRows];
        if (read_c) {
#pragma unroll
          for (int a = 0; a < kBatch; ++a)
#pragma unroll
            for (int r = 0; r < kRows; ++r) {
              if (a0 + a >= NA || (r0 + r) / 4 < q0 || (r0 + r) / 4 >= q1) continue;
              const int urow = m0 + OA::row(a0 + a, r0 + r, wm0);
              if constexpr (kAll) {
                c[a][r] = *reinterpret_cast<const Vec*>(
                    reinterpret_cast<const char*>(cin + (int64_t)urow * ldci) + coff);
              } else {  // past the edge: some element of C, not used
                const float* p = cin + (int64_t)(urow + lrow < q.m ? urow + lrow : q.m - 1) * ldci;
#pragma unroll
                for (int e = 0; e < V; ++e) put(c[a][r], e, p[col + e < q.n ? col + e : q.n - 1]);
              }
            }
        }
#pragma unroll
        for (int a = 0; a < kBatch; ++a)
#pragma unroll
          for (int r = 0; r < kRows; ++r) {
            if (a0 + a >= NA || (r0 + r) / 4 < q0 || (r0 + r) / 4 >= q1) continue;
            const int urow = m0 + OA::row(a0 + a, r0 + r, wm0), row = urow + lrow;
            Vec v{};
#pragma unroll
            for (int e = 0; e < V; ++e) {
              float x = alpha * acc[a0 + a][b0 + e][r0 + r];
              if (read_c) x = fmaf(q.beta, at(c[a][r], e), x);
              if constexpr (MODE == kDmaConsume) x = consume_op(o.op, x, at(bias, e), o.lo, o.hi);
              put(v, e, x);
            }
            float* p = reinterpret_cast<float*>(reinterpret_cast<char*>(out + (int64_t)urow * ldo) + ooff);
            if constexpr (kAll) {
              *reinterpret_cast<Vec*>(p) = v;
            } else if (row >= m_own && row < q.m) {
#pragma unroll
              for (int e = 0; e < V; ++e)
                if (col + e >= n_own && col + e < q.n) p[e] = at(v, e);
            }
          }
      }
    }
  };
  if (whole) store(std::true_type{});
  else store(std::false_type{});
}

// The arithmetic of one wave on staged sub-slabs: kSteps steps per sub-slab
// (an even number, or one where the buffer does not matter), each read from
// LDS one step ahead into buffer `buf` and multiplied from it.  MathF32: steps of 8 k, the fragments as read.
template <typename S>
struct MathF32 {
  using OA = typename S::OA;
  using OB = typename S::OB;
  static constexpr int NA = OA::kBlocks, NB = OB::kBlocks, kSteps = S::kTk / 8;
  f32x16 acc[NA][NB];
  typename OA::Frag fa[2][OA::kFrags];
  typename OB::Frag fb[2][OB::kFrags];
  int foff[kSteps], wm0, wn0, lane;

  __device__ __forceinline__ MathF32(int wm, int wn, int ln) : wm0(wm), wn0(wn), lane(ln) {
#pragma unroll
    for (int g = 0; g < kSteps; ++g) foff[g] = OA::Rows::frag(lane, g);
    zero_acc(acc);
  }
  // Step g of the sub-slab at st into buffer buf.
  __device__ __forceinline__ void read(int buf, const char* st, int g) {
#pragma unroll
    for (int j = 0; j < OB::kFrags; ++j) fb[buf][j] = OB::frag(st + OA::kBytes, j, g, wn0, lane, foff[g]);
#pragma unroll
    for (int j = 0; j < OA::kFrags; ++j) fa[buf][j] = OA::frag(st, j, g, wm0, lane, foff[g]);
  }
  // The first step read of all is ready to be multiplied.
  __device__ __forceinline__ void first() {}
  // Multiplies buffer buf; the next step (if any) was read into buf ^ 1.
  __device__ __forceinline__ void multiply(int buf) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(OA::pick(fa[buf], a, q), OB::pick(fb[buf], b, q),
                                                           acc[a][b], 0, 0, 0);
  }
};

// Accumulates tile (tm, tn) over contraction slice z on the whole
// workgroup, with the Allocation at smem (S::kLdsBytes), and hands the
// accumulators to `epilogue(acc, m0, n0, m_own, n_own, whole, wm0, wn0,
// lane, q0, q1)`.  Ends past a barrier with no transfer outstanding and (KW
// = 1) no LDS read pending, so smem may be reused at once.
template <typename S, typename Math, typename Epilogue>
__device__ __forceinline__ void any_tile(const GemmArgs& p, int splits, int tm, int tn, int z, char* smem,
                                         Epilogue epilogue) {
  using OA = typename S::OA;
  using OB = typename S::OB;
  constexpr int NA = OA::kBlocks, NB = OB::kBlocks, KW = S::kKw, NST = S::kNst, TK = S::kTk;
  constexpr int TM = S::kTm, TN = S::kTn, kSteps = Math::kSteps;
  constexpr bool AT = S::kAt, BT = S::kBt;
  static_assert(kSteps == 1 || kSteps % 2 == 0, "a sub-slab's last step uses buffer 1");
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int kw = KW == 1 ? 0 : wave / S::NWT, wt = KW == 1 ? wave : wave % S::NWT;
  const int wm0 = (wt / S::NWN) * S::kWm, wn0 = (wt % S::NWN) * S::kWn;
  // The tile's place, and the corner it is computed from (MN sides of at
  // least one tile move inward).
  const int m_own = tm * TM, n_own = tn * TN;
  const int m0 = AT && p.m >= TM && m_own + TM > p.m ? p.m - TM : m_own;
  const int n0 = !BT && p.n >= TN && n_own + TN > p.n ? p.n - TN : n_own;
  const int m_left = p.m - m0, n_left = p.n - n0;
  // Whole slabs of k (moved by DMA), then at most one partial slab.
  const bool last_by_hand = (AT && p.m < TM && p.m % 4 != 0) || (!BT && p.n < TN && p.n % 4 != 0);
  const int dma_all = (last_by_hand ? p.k - 1 : p.k) / S::kSlab;
  static_assert(S::kSlab <= kAnySlab, "p.k <= kAnyDepth");
  const int all = (p.k + S::kSlab - 1) / S::kSlab;
  const int per = (all + splits - 1) / splits, sbeg = z * per;
  const int slabs = all - sbeg < per ? all - sbeg : per;  // <= 0: this slice is empty
  const int dma = (dma_all < sbeg + slabs ? dma_all : sbeg + slabs) - sbeg;
  const bool has_tail = slabs > 0 && dma < slabs;

  const int64_t astep = (AT ? p.lda : 1) * (int64_t)TK * 4, bstep = (BT ? 1 : p.ldb) * (int64_t)TK * 4;
  // Source of this group's sub-slab of the slice's first slab.
  const char* abase = reinterpret_cast<const char*>(p.A) +
                      (AT ? (int64_t)m0 : (int64_t)m0 * p.lda) * 4 + ((int64_t)sbeg * KW + kw) * astep;
  const char* bbase = reinterpret_cast<const char*>(p.B) +
                      (BT ? (int64_t)n0 * p.ldb : (int64_t)n0) * 4 + ((int64_t)sbeg * KW + kw) * bstep;
  uint32_t aoff[S::QA], boff[S::QB];
#pragma unroll
  for (int j = 0; j < S::QA; ++j) aoff[j] = OA::offset(lane, wt * S::QA + j, m_left, p.lda);
#pragma unroll
  for (int j = 0; j < S::QB; ++j) boff[j] = OB::offset(lane, wt * S::QB + j, n_left, p.ldb);

  const uint32_t lds0 = lds_addr(smem) + kw * S::kSub;
  const char* sub = smem + kw * S::kSub;
  f32x4 ta[S::QA], tb[S::QB];
  if (has_tail) {
    const int depth = p.k - (sbeg + dma) * S::kSlab - kw * TK;
#pragma unroll
    for (int j = 0; j < S::QA; ++j)
      ta[j] = OA::tail(abase + (int64_t)dma * KW * astep, lane, wt * S::QA + j, m_left, depth, p.lda);
#pragma unroll
    for (int j = 0; j < S::QB; ++j)
      tb[j] = OB::tail(bbase + (int64_t)dma * KW * bstep, lane, wt * S::QB + j, n_left, depth, p.ldb);
  }
  // Slab i of the slice into stage st: requested, or for the tail written.
  auto bring = [&](int i, int st) {
    if (i < dma) {
      const uint32_t la = lds0 + st * S::kStage + wt * S::QA * 1024;
      const uint32_t lb = lds0 + st * S::kStage + OA::kBytes + wt * S::QB * 1024;
      const char* a = abase + (int64_t)i * KW * astep;
      const char* b = bbase + (int64_t)i * KW * bstep;
#pragma unroll
      for (int j = 0; j < S::QA; ++j) dma16(la + j * 1024, a, aoff[j]);
#pragma unroll
      for (int j = 0; j < S::QB; ++j) dma16(lb + j * 1024, b, boff[j]);
    } else if (i < slabs) {
      char* la = smem + st * S::kStage + kw * S::kSub + wt * S::QA * 1024 + lane * 16;
      char* lb = smem + st * S::kStage + kw * S::kSub + OA::kBytes + wt * S::QB * 1024 + lane * 16;
#pragma unroll
      for (int j = 0; j < S::QA; ++j) *reinterpret_cast<f32x4*>(la + j * 1024) = ta[j];
#pragma unroll
      for (int j = 0; j < S::QB; ++j) *reinterpret_cast<f32x4*>(lb + j * 1024) = tb[j];
    }
  };

  Math math(wm0, wn0, lane);
  if (slabs > 0) {
#pragma unroll
    for (int i = 0; i < NST - 1; ++i) bring(i, i);
    // Slab 0 has landed once at most the requests after it are outstanding.
    wait_slabs_barrier<S::Q, NST - 2>((dma < NST - 1 ? dma : NST - 1) - 1);
    // The tail's loads are older than slab 0's: their values are used here,
    // so that no wait for them falls between the later requests.
    if (has_tail) {
#pragma unroll
      for (int j = 0; j < S::QA; ++j) asm volatile("" : "+v"(ta[j]));
#pragma unroll
      for (int j = 0; j < S::QB; ++j) asm volatile("" : "+v"(tb[j]));
    }
    math.read(0, sub, 0);
    bring(NST - 1, NST - 1);
    math.first();
  }
  int st = 0;
  for (int s = 0; s < slabs; ++s) {
    const char* cur = sub + st * S::kStage;
#pragma unroll
    for (int g = 0; g + 1 < kSteps; ++g) {
      math.read((g + 1) & 1, cur, g + 1);
      math.multiply(g & 1);
    }
    // Slab s + 1 has landed everywhere and slab s is no longer read: bring
    // slab s + NST into its stage and read slab s + 1's first step under the
    // last step's MFMAs.
    const int nst = st + 1 == NST ? 0 : st + 1;
    const int newest = s + NST < dma ? s + NST : dma;  // DMA slabs requested so far
    wait_slabs_barrier<S::Q, NST - 2>(newest - (s + 2));
    if (s + 1 < slabs) {
      math.read(0, sub + nst * S::kStage, 0);
      bring(s + NST, st);
    }
    math.multiply(1);
    st = nst;
  }
  auto& acc = math.acc;
  const bool whole = m_own + TM <= p.m && n_own + TN <= p.n;
  if constexpr (KW == 1) {
    epilogue(acc, m0, n0, m_own, n_own, whole, wm0, wn0, lane, 0, 4);
  } else {
    // The groups' accumulators meet in LDS (past the loop's last barrier no
    // stage is read or written any more); each group adds a share of the
    // row quads, in group order, and stores it.
    constexpr int kQuads = S::kQuads;
    f32x4* part = reinterpret_cast<f32x4*>(smem);
    auto slot = [&](int grp, int a, int b, int g) {
      return ((((grp * S::NWT + wt) * NA + a) * NB + b) * 4 + g) * kWave + lane;
    };
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          part[slot(kw, a, b, g)] = f32x4{acc[a][b][4 * g], acc[a][b][4 * g + 1], acc[a][b][4 * g + 2],
                                          acc[a][b][4 * g + 3]};
    __syncthreads();
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          if (g / kQuads != kw) continue;
          f32x4 v = part[slot(0, a, b, g)];
#pragma unroll
          for (int w = 1; w < KW; ++w) v += part[slot(w, a, b, g)];
#pragma unroll
          for (int u = 0; u < 4; ++u) acc[a][b][4 * g + u] = v[u];
        }
    epilogue(acc, m0, n0, m_own, n_own, whole, wm0, wn0, lane, kw * kQuads, (kw + 1) * kQuads);
  }
}

template <int TM, int TN, int TK, int WM, int WN, bool AT, bool BT, int NST, int KW, typename Epilogue>
__device__ __forceinline__ void f32_any_tile(const GemmArgs& p, int splits, int tm, int tn, int z, char* smem,
                                             Epilogue epilogue) {
  using S = AnyShape<TM, TN, TK, WM, WN, AT, BT, NST, KW>;
  any_tile<S, MathF32<S>>(p, splits, tm, tn, z, smem, epilogue);
}

// One launch: a workgroup per tile and contraction slice (slice-major),
// XCD-aware tile order.
template <int TM, int TN, int TK, int WM, int WN, bool AT, bool BT, int NST, int KW, int MODE>
__global__ void __launch_bounds__((AnyShape<TM, TN, TK, WM, WN, AT, BT, NST, KW>::kThreads))
    __attribute__((amdgpu_waves_per_eu((AnyShape<TM, TN, TK, WM, WN, AT, BT, NST, KW>::kMinWaves)))) sgemm_f32_any(GemmArgs p, F32DmaOut o) {
  extern __shared__ __align__(16) char smem[];
  read_early(p);
  if constexpr (MODE == kDmaConsume) read_early(o.D, o.ldd, o.bias, o.op, o.lo, o.hi);
  using S = AnyShape<TM, TN, TK, WM, WN, AT, BT, NST, KW>;
  const int tiles = p.tiles_m * p.tiles_n;
  const int z = blockIdx.x / tiles;
  int tm, tn;
  tile_coords(p.tiles_m, p.tiles_n, blockIdx.x - z * tiles, tm, tn);
  f32_any_tile<TM, TN, TK, WM, WN, AT, BT, NST, KW>(
      p, o.splits, tm, tn, z, smem,
      [&](const auto& acc, int m0, int n0, int m_own, int n_own, bool whole, int wm0, int wn0, int lane, int q0,
          int q1) {
        any_epilogue<typename S::OA, typename S::OB, BT, MODE>(p, o, acc, m0, n0, m_own, n_own, whole, wm0, wn0, lane,
                                                               z, q0, q1);
      });
}

// Row pitch (floats) up to which a tile's rows lie within 32-bit byte offsets
// of its corner (at most 256 rows of an operand).
constexpr int64_t kAnyPitch = 1 << 22;

// True when the loop covers the product: something to contract, no deeper than
// kAnyDepth (a backward's m may be), MN operands at least one 16-byte unit wide,
// and pitches within kAnyPitch.
constexpr bool f32_any_fits(const GemmArgs& a, bool at, bool bt) {
  return a.m > 0 && a.n > 0 && a.k > 0 && a.k <= kAnyDepth && a.m < (1 << 30) && a.n < (1 << 30) && (!at || a.m >= 4) && (bt || a.n >= 4) &&
         a.lda < kAnyPitch && a.ldb < kAnyPitch && a.ldc < kAnyPitch && a.ldci < kAnyPitch;
}

}  // namespace hpvm
