// C-ABI layer of the sgemm dataflow-graph library: argument checks, the
// Allocation-size function, structural queries and the root launch.
//
// This file plays the role of the host code the paper's GPU backend emits
// (HPVM report, Sec. 6.3): it unpacks the root node's arguments, computes the
// Allocation node's size before the launch, sets the launch geometry from the
// SgemmInternal / SgemmLeaf instance counts, and enqueues the kernel.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <iterator>
#include <mutex>

#include "device_common.hpp"
#include "hpvm_sgemm.h"
#include "internal.hpp"

namespace hpvm {

namespace {
thread_local char g_error[512] = "";
}

int set_error(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_error, sizeof g_error, fmt, ap);
  va_end(ap);
  return code;
}

int clear_error() {
  g_error[0] = '\0';
  return HPVM_OK;
}

const char* last_error_text() { return g_error; }

int hip_error(hipError_t e, const char* what) {
  return set_error(HPVM_HIP_ERROR, "%s: %s", what, hipGetErrorString(e));
}

// HPVM_FAULT_INJECT=<site> makes the named step report a HIP failure after
// the argument checks, so that error propagation can be exercised without a
// GPU.  Sites: launch, wait, capture.
bool fault_injected(const char* site) {
  const char* v = std::getenv("HPVM_FAULT_INJECT");
  return v && std::strcmp(v, site) == 0;
}

void matrix_extent(const void* p, int64_t rows, int64_t cols, int64_t ld, uintptr_t* lo, uintptr_t* hi) {
  *lo = (uintptr_t)p;
  *hi = (uintptr_t)p + (uintptr_t)(((rows - 1) * ld + cols) * (int64_t)sizeof(float));
}

int check_operands(const char* what, int64_t m, int64_t n, int64_t k, float alpha, const float* A, int64_t lda,
                   const float* B, int64_t ldb, bool* reads_ab) {
  if (m < 0) return set_error(HPVM_INVALID_ARG, "%sargument 1: m = %lld < 0", what, (long long)m);
  if (n < 0) return set_error(HPVM_INVALID_ARG, "%sargument 2: n = %lld < 0", what, (long long)n);
  if (k < 0) return set_error(HPVM_INVALID_ARG, "%sargument 3: k = %lld < 0", what, (long long)k);
  if (m > INT32_MAX || n > INT32_MAX || k > INT32_MAX)
    return set_error(HPVM_UNSUPPORTED, "%ssizes above 2^31 - 1 are not supported", what);
  const bool empty = (m == 0 || n == 0);
  *reads_ab = !empty && k > 0 && alpha != 0.0f;
  if (*reads_ab && !A) return set_error(HPVM_INVALID_ARG, "%sargument 5: A is NULL", what);
  if (lda < (k > 1 ? k : 1))
    return set_error(HPVM_INVALID_ARG, "%sargument 6: lda = %lld < max(1, k)", what, (long long)lda);
  if (*reads_ab && !B) return set_error(HPVM_INVALID_ARG, "%sargument 7: B is NULL", what);
  if (ldb < (n > 1 ? n : 1))
    return set_error(HPVM_INVALID_ARG, "%sargument 8: ldb = %lld < max(1, n)", what, (long long)ldb);
  return HPVM_OK;
}

int check_output(const char* what, int64_t m, int64_t n, int64_t k, const float* A, int64_t lda, const float* B,
                 int64_t ldb, const float* C, int64_t ldc, bool reads_ab, int argno, char name) {
  if (m > 0 && n > 0 && !C) return set_error(HPVM_INVALID_ARG, "%sargument %d: %c is NULL", what, argno, name);
  if (ldc < (n > 1 ? n : 1))
    return set_error(HPVM_INVALID_ARG, "%sargument %d: ld%c = %lld < max(1, n)", what, argno + 1, name + ('a' - 'A'),
                     (long long)ldc);
  if (reads_ab) {
    uintptr_t c0, c1, x0, x1;
    matrix_extent(C, m, n, ldc, &c0, &c1);
    matrix_extent(A, m, k, lda, &x0, &x1);
    const bool oa = c0 < x1 && x0 < c1;
    matrix_extent(B, k, n, ldb, &x0, &x1);
    const bool ob = c0 < x1 && x0 < c1;
    if (oa || ob)
      return set_error(HPVM_INVALID_ARG, "%sargument %d: %c overlaps A or B", what, argno, name);
  }
  return HPVM_OK;
}

int check_gemm_args(const char* what, int64_t m, int64_t n, int64_t k, float alpha, const float* A,
                    int64_t lda, const float* B, int64_t ldb, float beta, const float* C,
                    int64_t ldc, bool* reads_ab) {
  (void)beta;
  const int rc = check_operands(what, m, n, k, alpha, A, lda, B, ldb, reads_ab);
  return rc != HPVM_OK ? rc : check_output(what, m, n, k, A, lda, B, ldb, C, ldc, *reads_ab, 10, 'C');
}

}  // namespace hpvm

namespace {

using hpvm::set_error;

int fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  return set_error(code, "%s", buf);
}

int ok() { return hpvm::clear_error(); }

int hip_fail(hipError_t e, const char* what) { return hpvm::hip_error(e, what); }

bool inject(const char* site) { return hpvm::fault_injected(site); }

bool valid_prec(int32_t prec) {
  return prec == HPVM_PREC_FP32 || prec == HPVM_PREC_BF16 || prec == HPVM_PREC_BF16X3;
}

bool is_literal(const hpvm_tile& t) { return t.leaf_m == 1 && t.leaf_n == 1; }

// Literal lowering: tile_n x tile_m lanes (block_x = tile_n, block_y =
// tile_m), a whole number of wavefronts, at most 1024 lanes; the staged B
// slab is tile_m deep and one buffer.  The untiled one-level graph has the
// same lanes, tile_k = 0 and stages = 0 (no Allocation node).
bool is_flat(const hpvm_tile& t) { return t.stages == 0 && t.tile_k == 0; }
bool literal_ok(const hpvm_tile& t) {
  const int64_t lanes = (int64_t)t.tile_m * t.tile_n;
  return t.tile_m > 0 && t.tile_n > 0 && lanes >= hpvm::kWave && lanes <= 1024 &&
         lanes % hpvm::kWave == 0 && ((t.tile_k == t.tile_m && t.stages == 1) || is_flat(t));
}

const hpvm::MfmaEntry* find_entry(int32_t prec, const hpvm_tile* tile) {
  if (!tile) return hpvm::menu_entry_at(prec, 0);
  return hpvm::find_menu_entry(prec, *tile);
}

// Resolves the lowering for (prec, tile); *entry is null for the literal one.
int resolve(int32_t prec, const hpvm_tile* tile, const hpvm::MfmaEntry** entry, int argno) {
  *entry = nullptr;
  if (tile && is_literal(*tile)) {
    if (prec != HPVM_PREC_FP32)
      return fail(HPVM_UNSUPPORTED, "argument %d: the literal lowering (leaf 1x1) is FP32 only", argno);
    if (!literal_ok(*tile))
      return fail(HPVM_UNSUPPORTED,
                  "argument %d: literal tile %dx%d (k %d, stages %d) needs 64..1024 lanes in whole "
                  "wavefronts, and tile_k == tile_m with one stage, or tile_k = 0 with none (untiled)",
                  argno, tile->tile_m, tile->tile_n, tile->tile_k, tile->stages);
    return HPVM_OK;
  }
  *entry = find_entry(prec, tile);
  if (!*entry) {
    if (tile)
      return fail(HPVM_UNSUPPORTED, "argument %d: tile %dx%dx%d leaf %dx%d stages %d is not compiled for precision %d",
                  argno, tile->tile_m, tile->tile_n, tile->tile_k, tile->leaf_m, tile->leaf_n,
                  tile->stages, prec);
    return fail(HPVM_UNSUPPORTED, "no compiled tile for precision %d", prec);
  }
  return HPVM_OK;
}

int64_t tiles_of(const hpvm_tile& t, int64_t m, int64_t n) {
  return ((m + t.tile_m - 1) / t.tile_m) * ((n + t.tile_n - 1) / t.tile_n);
}
const hpvm::MfmaEntry* f32_mid_entry() {
  return hpvm::find_menu_entry(HPVM_PREC_FP32, hpvm_tile{128, 128, 32, 32, 128, 2});
}
}  // namespace

namespace hpvm {
// A tile's estimated time (microseconds): `start` (launch, the ring's first
// fill, the last epilogue); per 32 of k, `alone` for a tile that has its CU
// to itself, at least `shared` for each of the tiles that one of 256 CUs
// gets; and `more` for each of those after the first, whose prologue and
// epilogue the others hide in part (at short contractions it is most of the
// time: 4096 x 4096 x 16 in 32 x 32 tiles 164 us, in 64 x 128 30).
struct TileTime {
  hpvm_tile tile;
  double start, alone, shared, more;
  bool aligned;  // only where its own loop runs (mfma_f32_dma.hpp, mfma_bf16_dma.hpp)
  bool wide = false;  // too many registers or LDS to run beside an open streaming graph
};
static double tile_time(const TileTime& c, double tiles, double k) {
  const double rounds = std::ceil(tiles / 256.0);
  return c.start + std::max(c.alone, rounds * c.shared) * k / 32.0 + (rounds - 1.0) * c.more;
}

// Where tiles that cannot run beside an open streaming graph may be taken.
// Its two workgroups a CU leave 87 KB of LDS and, per SIMD, 176 registers; a
// kernel that needs more waits until the stream has ended, which a program that
// streams meanwhile cannot wait for.  They are taken where the product gives
// 256 tiles of this size, or of their own if that needs alignment.
constexpr hpvm_tile kWideFrom128{128, 128, 32, 64, 64, 4}, kWideFrom256{256, 256, 32, 64, 128, 2};

// The candidate with the least time, a contraction split that fits split_ws
// (< 0: any) included: the partial sums' traffic at 4 TB/s and the summing
// launch.
static bool least_time(const TileTime* c, int count, int32_t prec, int64_t m, int64_t n, int64_t k, int64_t split_ws,
                       bool large_only, const hpvm_tile& wide_from, hpvm_tile* out, double* estimate) {
  double best = 0.0;
  bool found = false;
  for (; count > 0; --count, ++c) {
    const hpvm_tile& t = c->tile;
    if (c->aligned && (m < t.tile_m || n < t.tile_n || n % 4 || k % t.tile_k)) continue;
    if (large_only && t.tile_m * t.tile_n < 128 * 256) continue;
    if (c->wide && tiles_of(c->aligned ? t : wide_from, m, n) < 256) continue;
    int64_t slices = 1, bytes = 0;
    if (!c->aligned && k >= 1024)  // no entry splits less (AnyConfig::splits)
      bytes = entry_split_bytes(find_menu_entry(prec, t), m, n, k);
    if (bytes > 0 && (split_ws < 0 || split_ws >= bytes)) slices = bytes / (m * n * (int64_t)sizeof(float));
    double time = tile_time(*c, (double)(tiles_of(t, m, n) * slices), (double)k / slices);
    if (slices > 1) time += 4.5 + (double)(bytes + m * n * 4) / 4.0e6;
    if (!found || time < best) {
      best = time;
      *out = t;
      found = true;
    }
  }
  if (estimate) *estimate = best;
  return found;
}

constexpr TileTime kF32Mid{{128, 128, 32, 32, 128, 2}, 9.5, 1.77, 1.77, 5.0, true};
constexpr TileTime kF32Groups[] = {
    {{64, 64, 32, 16, 32, 2}, 5.7, 0.597, 0.498, 2.3, false},
    {{32, 32, 128, 8, 32, 2}, 5.4, 0.141, 0.129, 2.0, false},
};

// Whether a tile whose waves share k in at least as many groups as the
// whole-tile split `t` has slices (so that no sum is longer) is estimated
// faster than that split, with `bytes` of partial sums.  Not asked where that
// has four slices or more in a single round, which it fills evenly.  1536^3,
// two slices in two rounds: 100 us against 76 in 32 x 32 tiles;
// 2048 x 1024 x 512, two in one: 30 against 25 in 64 x 64.
static bool f32_groups_beat_split(const hpvm_tile& t, int64_t m, int64_t n, int64_t k, int64_t bytes,
                                  hpvm_tile* out) {
  const int64_t slices = bytes / (m * n * (int64_t)sizeof(float)), tiles = tiles_of(t, m, n) * slices;
  if (slices >= 4 && tiles <= 256) return false;
  const double area = (double)t.tile_m * t.tile_n / (128.0 * 128.0);
  TileTime c = kF32Mid;
  c.alone *= area;
  c.shared *= area;
  const double split = tile_time(c, (double)tiles, (double)k / slices) + 4.5 + (double)(bytes + m * n * 4) / 4.0e6;
  const TileTime* from = kF32Groups + (slices > 2 ? 1 : 0);  // two groups, four
  double groups = 0.0;
  return slices <= 4 && least_time(from, (int)(std::end(kF32Groups) - from), HPVM_PREC_FP32, m, n, k, 0, false,
                                   kWideFrom256, out, &groups) &&
         groups < split;
}

// FP32.  Fitted to each tile's time over 72 products from 64 x 64 x 1000 to
// 8192 x 8192 x 200; over those the choice is 2% behind the best tile on
// average.  Measured, us, this choice and the next best size of tile:
//   1500 x 1500 x 100: 64 x 64 13.3, 64 x 128 15.2
//   2048 x 2048 x 256: 64 x 128 23.3, 64 x 64 26.4; 2048^3: 128 x 128 128
//   1000 x 1003 x 777: 64 x 64 in two k groups 22.2, in one 23.7
//   512^3: 32 x 32 in four k groups 6.5, 64 x 64 15.0
//   4096^3: 256 x 256 932
bool f32_default_tile(int64_t m, int64_t n, int64_t k, int64_t split_ws, hpvm_tile* out) {
  static const TileTime kCandidates[] = {
      {{256, 256, 32, 64, 128, 2}, 13.0, 6.31, 6.89, 32.0, true, true},
      kF32Mid,
      {{64, 128, 32, 32, 64, 2}, 6.2, 1.09, 0.948, 2.3, false},
      {{64, 128, 16, 32, 64, 2}, 5.7, 1.18, 0.983, 2.3, false},
      {{64, 64, 16, 32, 32, 2}, 4.5, 0.712, 0.541, 1.43, false},
      kF32Groups[0],
      kF32Groups[1],
  };
  return least_time(kCandidates, (int)(sizeof(kCandidates) / sizeof(kCandidates[0])), HPVM_PREC_FP32, m, n, k,
                    split_ws, false, kWideFrom256, out, nullptr);
}

// BF16 and bf16x3, fitted the same way.  These loops move FP32 operands and
// convert them in registers, so a slab's time is that of its transfers, LDS
// reads and conversions, not of its MFMAs.  Measured, us:
//   1024^3: 64 x 64 13.5, 64 x 128 15.5; bf16x3 20.3, 25.4
//   2048 x 2048 x 256: 64 x 128 11.8, 64 x 64 14.1; bf16x3 16.6, 18.5
//   3000 x 3000 x 256: 256 x 256 24.0, 64 x 128 25.3; bf16x3 64 x 128 34.7
//   100 x 3000 x 1500: 32 x 128, split 15.7, 64 x 64 18.0
// bf16x3's 64 x 128 tile has 192 registers.  Products of 256 tiles of 256 x 256
// (bf16x3: of 128 x 128) have never run beside an open stream.
static bool bf16_default_tile(int32_t prec, int64_t m, int64_t n, int64_t k, int64_t split_ws, hpvm_tile* out,
                              double* estimate = nullptr, bool large_only = false) {
  const MfmaEntry* e0 = menu_entry_at(prec, 0);
  if (!e0) return false;
  const TileTime kBf16[] = {
      {e0->tile, 28.0, 0.72, 1.15, 28.0, true, true},
      {{128, 256, 32, 64, 64, 2}, 13.0, 0.9, 0.9, 20.0, false, true},
      {{128, 128, 32, 64, 64, 4}, 10.7, 0.44, 0.44, 11.0, true, true},
      {{64, 128, 32, 32, 64, 2}, 6.0, 0.366, 0.265, 3.0, false},
      {{64, 64, 32, 32, 32, 2}, 4.5, 0.299, 0.182, 1.6, false},
      {{32, 128, 32, 32, 32, 2}, 4.6, 0.327, 0.219, 1.85, false},
  };
  const TileTime kX3[] = {
      {e0->tile, 28.0, 2.4, 2.2, 48.0, true, true},
      {{128, 256, 32, 64, 64, 2}, 14.0, 1.75, 1.75, 20.0, false, true},
      {{128, 128, 32, 64, 64, 4}, 11.0, 0.85, 0.85, 9.6, true, true},
      {{64, 128, 32, 32, 64, 2}, 6.4, 0.664, 0.498, 2.9, false, true},
      {{64, 64, 32, 32, 32, 2}, 4.9, 0.471, 0.316, 1.55, false},
      {{32, 128, 32, 32, 32, 2}, 4.9, 0.509, 0.35, 1.85, false},
  };
  return least_time(prec == HPVM_PREC_BF16X3 ? kX3 : kBf16, (int)(sizeof(kX3) / sizeof(kX3[0])), prec, m, n, k,
                    split_ws, large_only, prec == HPVM_PREC_BF16X3 ? kWideFrom128 : kWideFrom256, out, estimate);
}
}  // namespace hpvm

namespace {

// The DMA-fed whole-tile entry whose split contraction needs the fewest partial sums
// (the deepest slices; the first in menu order on a tie), or null.
const hpvm::MfmaEntry* fewest_slices(int32_t prec, int64_t m, int64_t n, int64_t k, int64_t* bytes) {
  const hpvm::MfmaEntry* best = nullptr;
  int64_t best_bytes = 0;
  for (int i = 0; i < hpvm::menu_size(prec); ++i) {
    const hpvm::MfmaEntry* e = hpvm::menu_entry_at(prec, i);
    if (e->tile.tile_m < 128) continue;
    const int64_t b = hpvm::entry_split_bytes(e, m, n, k);
    if (b > 0 && (!best || b < best_bytes)) {
      best = e;
      best_bytes = b;
    }
  }
  *bytes = best_bytes;
  return best;
}

// Built-in choice of hpvm_sgemm_ws (and of hpvm_sgemm_workspace_bytes) for
// tile == NULL when the autotuner has no entry; ws_bytes: the caller's
// workspace (-1 = as much as needed).  In order:
//  * whole-tile products that even 128 x 128 tiles would not cover the CUs
//    with (BF16 and bf16x3: with k >= 2048; at 1024^3 the 64 x 64 tiles were
//    faster) take the DMA-fed entry that splits the contraction into the
//    deepest slices when the workspace holds its partial sums (BF16
//    512 x 512 x 4096: 0.035 ms against 0.095 on 64 x 64 tiles); with a
//    smaller workspace, hpvm_sgemm's choice;
//  * FP32, and BF16 / bf16x3 products under 2^31 multiply-adds, the tile
//    with the least estimated time, splits that fit the workspace included;
//  * larger BF16 products a staged tile, whose conversion pass is then a
//    small share of the time (8192^3: 1.07 ms against 1.48): the first, of
//    256 x 256, when that gives 256 tiles and is estimated faster than the
//    128 x 128 x 64 tile of 64 x 32 waves (4097 x 4099 x 2001, two rounds of
//    the first: 148 us against 138); bf16x3 ones the DMA-fed 256 x 256 tile
//    then, which converts in its fragment reads (8192^3: 2.71 ms against
//    2.82 staged);
//  * of the rest, and of those with k < 256, the tile with the least
//    estimated time, the staged 128 x 128 one included, where k < 1024
//    (2500 x 2500 x 400 bf16x3: 36 us against 51 staged); for deeper ones
//    the staged, unless 128 x 256 tiles on the FP32 operands are estimated
//    faster, then hpvm_sgemm's choice.  BF16 under 256 tiles of 256 x 256 keeps
//    the staged 128 x 128 tile (64 KB, 88 registers: it runs beside an open
//    stream) also where hpvm_sgemm's choice is faster but could not.
// Returns false for hpvm_sgemm's choice.
bool default_ws_tile(int32_t prec, int64_t m, int64_t n, int64_t k, int64_t ws_bytes, hpvm_tile* out) {
  const bool f32 = prec == HPVM_PREC_FP32, x3 = prec == HPVM_PREC_BF16X3;
  const hpvm::MfmaEntry* mid =
      f32 ? f32_mid_entry() : hpvm::find_menu_entry(prec, hpvm_tile{128, 128, 32, 64, 64, 4});
  if (mid && tiles_of(mid->tile, m, n) < 256 && (f32 || k >= 2048)) {
    int64_t need = 0;
    const hpvm::MfmaEntry* best = fewest_slices(prec, m, n, k, &need);
    if (best && ws_bytes >= 0 && ws_bytes < need) return false;
    if (best) {
      *out = best->tile;
      return true;
    }
  }
  if (f32) return hpvm::f32_default_tile(m, n, k, ws_bytes, out);
  if ((double)m * (double)n * (double)k < 2147483648.0) return hpvm::bf16_default_tile(prec, m, n, k, ws_bytes, out);
  const hpvm::MfmaEntry* staged = nullptr;
  if (!hpvm::staged_k_ok(k) || hpvm::staged_menu(prec, &staged) == 0) return false;
  const hpvm::MfmaEntry* small = hpvm::find_menu_entry(prec, hpvm_tile{128, 128, 64, 64, 32, 3});
  if (!small) return false;
  // Estimates of the staged tiles: launches and the pass over the operands
  // at 4.8 TB/s, then as tile_time.
  const double pass = ((double)m * k + (double)k * n) * (x3 ? 8.0 : 6.0) / 4.8e6, slabs = (double)k / 32.0;
  const double rs = (double)((tiles_of(small->tile, m, n) + 255) / 256);
  const double time_small = 12.0 + pass + rs * slabs * (x3 ? 0.62 : 0.27) + (rs - 1.0) * 6.0;
  const int64_t big_tiles = tiles_of(staged[0].tile, m, n);
  const double rb = (double)((big_tiles + 255) / 256);
  const hpvm::MfmaEntry* e0 = hpvm::menu_entry_at(prec, 0);
  const bool direct0 = x3 && e0 && k % e0->tile.tile_k == 0 && n % 4 == 0;
  const double time_big = direct0 ? 28.0 + rb * slabs * 2.2 + (rb - 1.0) * 48.0
                                  : 26.0 + pass + rb * slabs * (x3 ? 1.9 : 0.85) + (rb - 1.0) * 45.0;
  const bool big = big_tiles >= 256 && k >= 256 && time_big <= time_small;
  if (big && direct0) return false;
  // A workspace too small for the planes: the choice without one.
  if (ws_bytes >= 0 && ws_bytes < hpvm::staged_workspace_bytes(prec, m, n, k)) return false;
  if (!big) {
    double direct = 0.0;
    const bool faster = hpvm::bf16_default_tile(prec, m, n, k, 0, out, &direct, k >= 1024) && direct < time_small;
    if (faster && (x3 || big_tiles >= 256 || out->tile_m * out->tile_n < 128 * 128)) return false;
  }
  *out = big ? staged[0].tile : small->tile;
  return true;
}

// The tile a call with tile == NULL runs.  ws_ok: the call has a workspace
// argument (hpvm_sgemm_ws); ws_bytes: its size, or -1 for "as much as the
// choice needs" (hpvm_sgemm_workspace_bytes asks which tile that is).  In
// order: the autotuned winner (with a workspace the overall one, unless it
// splits the contraction and the workspace cannot hold the partial sums:
// then the winner that needs none), the built-in workspace choice, the tile
// with the least estimated time; false = the menu's entry 0.
int describe_impl(int64_t m, int64_t n, int64_t k, int32_t prec, const hpvm_tile* tile, bool ws_ok,
                  int64_t ws_bytes, hpvm_dfg* out);

bool choose_tile(int32_t prec, int64_t m, int64_t n, int64_t k, bool ws_ok, int64_t ws_bytes, hpvm_tile* out) {
  if (hpvm::tuned_tile(prec, m, n, k, ws_ok, out)) {
    if (!ws_ok || ws_bytes < 0) return true;
    const hpvm::MfmaEntry* e = hpvm::find_menu_entry(prec, *out);
    const int64_t need = std::max(hpvm::entry_split_bytes(e, m, n, k), hpvm::entry_workspace_bytes(e, m, n, k));
    if (need == 0 || ws_bytes >= need) return true;
    return hpvm::tuned_tile(prec, m, n, k, false, out) != 0;
  }
  const hpvm::MfmaEntry* mid = prec == HPVM_PREC_FP32 ? f32_mid_entry() : nullptr;
  if (mid && tiles_of(mid->tile, m, n) < 256) {  // with a workspace or without: the same tile
    int64_t need = 0;
    const hpvm::MfmaEntry* best = fewest_slices(prec, m, n, k, &need);
    if (best && hpvm::f32_groups_beat_split(best->tile, m, n, k, need, out)) return true;
  }
  if (ws_ok && default_ws_tile(prec, m, n, k, ws_bytes, out)) return true;
  return prec == HPVM_PREC_FP32 ? hpvm::f32_default_tile(m, n, k, 0, out)
                                : hpvm::bf16_default_tile(prec, m, n, k, 0, out);
}

}  // namespace

extern "C" {

const char* hpvm_status_string(int status) {
  switch (status) {
    case HPVM_OK: return "HPVM_OK";
    case HPVM_INVALID_ARG: return "HPVM_INVALID_ARG";
    case HPVM_UNSUPPORTED: return "HPVM_UNSUPPORTED";
    case HPVM_HIP_ERROR: return "HPVM_HIP_ERROR";
    case HPVM_WORKSPACE_TOO_SMALL: return "HPVM_WORKSPACE_TOO_SMALL";
    case HPVM_BAD_HANDLE: return "HPVM_BAD_HANDLE";
    case HPVM_QUEUE_FULL: return "HPVM_QUEUE_FULL";
    case HPVM_TIMEOUT: return "HPVM_TIMEOUT";
    case HPVM_STREAM_ENDED: return "HPVM_STREAM_ENDED";
    default: return "HPVM_UNKNOWN_STATUS";
  }
}

const char* hpvm_last_error(void) { return hpvm::last_error_text(); }

int hpvm_alloc_bytes(const hpvm_tile* tile, int32_t prec, int64_t* bytes) {
  if (!tile) return fail(HPVM_INVALID_ARG, "argument 1: tile is NULL");
  if (!valid_prec(prec)) return fail(HPVM_INVALID_ARG, "argument 2: unknown precision %d", prec);
  if (!bytes) return fail(HPVM_INVALID_ARG, "argument 3: bytes is NULL");
  const hpvm::MfmaEntry* e;
  int rc = resolve(prec, tile, &e, 1);
  if (rc != HPVM_OK) return rc;
  *bytes = e ? e->lds_bytes : is_flat(*tile) ? 0 : hpvm::literal_alloc_bytes(tile->tile_n, tile->tile_m);
  return ok();
}

int hpvm_tile_menu(int32_t prec, hpvm_tile* out, int32_t capacity, int32_t* count) {
  if (!valid_prec(prec)) return fail(HPVM_INVALID_ARG, "argument 1: unknown precision %d", prec);
  if (capacity < 0 || (capacity > 0 && !out))
    return fail(HPVM_INVALID_ARG, "argument 3: bad capacity or NULL output");
  if (!count) return fail(HPVM_INVALID_ARG, "argument 4: count is NULL");
  const int n = hpvm::menu_size(prec);
  for (int i = 0; i < n && i < capacity; ++i) out[i] = hpvm::menu_entry_at(prec, i)->tile;
  *count = n;
  return ok();
}

int hpvm_describe(int64_t m, int64_t n, int64_t k, int32_t prec, const hpvm_tile* tile, hpvm_dfg* out) {
  if (m < 0) return fail(HPVM_INVALID_ARG, "argument 1: m = %lld < 0", (long long)m);
  if (n < 0) return fail(HPVM_INVALID_ARG, "argument 2: n = %lld < 0", (long long)n);
  if (k < 0) return fail(HPVM_INVALID_ARG, "argument 3: k = %lld < 0", (long long)k);
  if (!valid_prec(prec)) return fail(HPVM_INVALID_ARG, "argument 4: unknown precision %d", prec);
  if (!out) return fail(HPVM_INVALID_ARG, "argument 6: out is NULL");
  return describe_impl(m, n, k, prec, tile, false, 0, out);
}

int hpvm_describe_ws(int64_t m, int64_t n, int64_t k, int32_t prec, const hpvm_tile* tile,
                     int64_t workspace_bytes, hpvm_dfg* out) {
  if (m < 0) return fail(HPVM_INVALID_ARG, "argument 1: m = %lld < 0", (long long)m);
  if (n < 0) return fail(HPVM_INVALID_ARG, "argument 2: n = %lld < 0", (long long)n);
  if (k < 0) return fail(HPVM_INVALID_ARG, "argument 3: k = %lld < 0", (long long)k);
  if (!valid_prec(prec)) return fail(HPVM_INVALID_ARG, "argument 4: unknown precision %d", prec);
  if (workspace_bytes < 0)
    return fail(HPVM_INVALID_ARG, "argument 6: workspace_bytes = %lld < 0", (long long)workspace_bytes);
  if (!out) return fail(HPVM_INVALID_ARG, "argument 7: out is NULL");
  return describe_impl(m, n, k, prec, tile, true, workspace_bytes, out);
}

}  // extern "C"

namespace {

int describe_impl(int64_t m, int64_t n, int64_t k, int32_t prec, const hpvm_tile* tile, bool ws_ok,
                  int64_t ws_bytes, hpvm_dfg* out) {
  hpvm_tile chosen;
  if (!tile && choose_tile(prec, m, n, k, ws_ok, ws_bytes, &chosen)) tile = &chosen;
  const hpvm::MfmaEntry* e;
  int rc = resolve(prec, tile, &e, 5);
  if (rc != HPVM_OK) return rc;
  const hpvm_tile t = e ? e->tile : *tile;
  std::memset(out, 0, sizeof *out);
  out->root_instances = 1;
  out->splits = 1;
  out->tile = t;
  const int64_t split = ws_ok ? hpvm::entry_split_bytes(e, m, n, k) : 0;
  if (split > 0 && ws_bytes >= split && m > 0 && n > 0 && k > 0)
    out->splits = (int32_t)(split / (m * n * (int64_t)sizeof(float)));
  out->grid_x = (int32_t)((n + t.tile_n - 1) / t.tile_n);
  out->grid_y = (int32_t)((m + t.tile_m - 1) / t.tile_m);
  out->k_slabs = t.tile_k > 0 ? (int32_t)((k + t.tile_k - 1) / t.tile_k) : 0;
  if (e) {
    out->block_x = e->threads;
    out->block_y = 1;
    out->waves = e->threads / hpvm::kWave;
    out->alloc_bytes = e->lds_bytes;
    if (e->launch_staged)
      out->lowering = prec == HPVM_PREC_BF16 ? hpvm::kStagedBf16 : hpvm::kStagedBf16x3;
    else
      out->lowering = prec == HPVM_PREC_FP32 ? hpvm::kMfmaF32
                      : prec == HPVM_PREC_BF16 ? hpvm::kMfmaBf16
                                                : hpvm::kMfmaBf16x3;
  } else {
    out->block_x = t.tile_n;
    out->block_y = t.tile_m;
    out->waves = t.tile_m * t.tile_n / hpvm::kWave;
    out->alloc_bytes = is_flat(t) ? 0 : hpvm::literal_alloc_bytes(t.tile_n, t.tile_m);
    out->lowering = is_flat(t) ? hpvm::kFlat : hpvm::kLiteral;
    if (is_flat(t)) out->k_slabs = 0;
  }
  return ok();
}

}  // namespace

extern "C" {

// The sgemm graph of Sec. 6.1: SgemmRoot (0) creates a 2-D SgemmInternal (1)
// and binds its inputs 0..13 through; SgemmInternal creates Allocation (2)
// and a 2-D SgemmLeaf (3), wires Allocation's outputs 0 and 1 (pointer,
// bytes) to the leaf's inputs 12 and 13 with all-to-all replication (one
// Allocation instance feeds every leaf instance), binds its own inputs 0..11
// to the leaf's 0..11 and its inputs 12, 13 (block_x, block_y) to
// Allocation's 0, 1.
int hpvm_dfg_edges(hpvm_edge* out, int32_t capacity, int32_t* count) {
  if (capacity < 0 || (capacity > 0 && !out))
    return fail(HPVM_INVALID_ARG, "argument 2: bad capacity or NULL output");
  if (!count) return fail(HPVM_INVALID_ARG, "argument 3: count is NULL");
  hpvm_edge table[64];
  int n = 0;
  table[n++] = hpvm_edge{0, 2, 3, 0, 12, 1};
  table[n++] = hpvm_edge{0, 2, 3, 1, 13, 1};
  for (int port = 0; port < 12; ++port) table[n++] = hpvm_edge{1, 1, 3, port, port, 0};
  table[n++] = hpvm_edge{1, 1, 2, 12, 0, 0};
  table[n++] = hpvm_edge{1, 1, 2, 13, 1, 0};
  for (int port = 0; port < 14; ++port) table[n++] = hpvm_edge{1, 0, 1, port, port, 0};
  for (int i = 0; i < n && i < capacity; ++i) out[i] = table[i];
  *count = n;
  return ok();
}

}  // extern "C"

namespace {

// Numbers, in the messages of an entry point's checks, of its output C (the
// leading dimension is the next) and of its precision (the tile, workspace and
// workspace's size are the next three).
struct ArgNos {
  int c, prec;
  char c_name;
};
constexpr ArgNos kSgemmNos{10, 12, 'C'}, kIntoNos{12, 14, 'D'};

// hpvm_sgemm and hpvm_sgemm_ws: `ws_ok` tells whether a workspace argument
// exists.  Cin, ldci: where beta * C is read when that is not C
// (hpvm_sgemm_into, which checked them).
int sgemm_impl(int64_t m, int64_t n, int64_t k, float alpha, const float* A, int64_t lda, const float* B,
               int64_t ldb, float beta, float* C, int64_t ldc, int32_t prec, const hpvm_tile* tile, bool ws_ok,
               void* workspace, int64_t workspace_bytes, void* stream, const float* Cin = nullptr,
               int64_t ldci = 0, const ArgNos& no = kSgemmNos) {
  // Checks in argument order; nothing below touches the device until all pass.
  bool reads_ab = false;
  int rc = hpvm::check_operands("", m, n, k, alpha, A, lda, B, ldb, &reads_ab);
  if (rc == HPVM_OK) rc = hpvm::check_output("", m, n, k, A, lda, B, ldb, C, ldc, reads_ab, no.c, no.c_name);
  if (rc != HPVM_OK) return rc;
  if (!valid_prec(prec)) return fail(HPVM_INVALID_ARG, "argument %d: unknown precision %d", no.prec, prec);
  hpvm_tile tuned;
  if (!tile && choose_tile(prec, m, n, k, ws_ok, workspace ? workspace_bytes : 0, &tuned)) tile = &tuned;
  const hpvm::MfmaEntry* entry;
  rc = resolve(prec, tile, &entry, no.prec + 1);
  if (rc != HPVM_OK) return rc;
  const int64_t need = hpvm::entry_workspace_bytes(entry, m, n, k);
  if (need > 0 && reads_ab) {
    if (!hpvm::staged_k_ok(k))
      return fail(HPVM_UNSUPPORTED, "argument %d: k = %lld is too deep for a tile with stages = 3", no.prec + 1,
                  (long long)k);
    if (!ws_ok)
      return fail(HPVM_UNSUPPORTED, "argument %d: tile with stages = 3 needs a workspace (use hpvm_sgemm_ws)",
                  no.prec + 1);
    if (!workspace) return fail(HPVM_INVALID_ARG, "argument %d: workspace is NULL", no.prec + 2);
    if ((uintptr_t)workspace % 16)
      return fail(HPVM_INVALID_ARG, "argument %d: workspace is not 16-byte aligned", no.prec + 2);
    if (workspace_bytes < need)
      return fail(HPVM_WORKSPACE_TOO_SMALL, "argument %d: workspace has %lld bytes, needs %lld", no.prec + 3,
                  (long long)workspace_bytes, (long long)need);
  }
  const bool empty = (m == 0 || n == 0);
  if (empty) return ok();
  if (inject("launch")) return fail(HPVM_HIP_ERROR, "injected launch failure (HPVM_FAULT_INJECT)");

  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  hipError_t e;
  if (!reads_ab) {
    e = hpvm::launch_scale(C, ldc, m, n, beta, s, Cin, ldci);
    return e == hipSuccess ? ok() : hip_fail(e, "scale launch");
  }
  hpvm::GemmArgs a{};
  a.A = A;
  a.B = B;
  a.C = C;
  a.lda = lda;
  a.ldb = ldb;
  a.ldc = ldc;
  a.m = (int32_t)m;
  a.n = (int32_t)n;
  a.k = (int32_t)k;
  a.alpha = alpha;
  a.beta = beta;
  a.Cin = Cin ? Cin : C;
  a.ldci = Cin ? ldci : ldc;
  a.vec_a = hpvm::vec16(A, lda);
  a.vec_b = hpvm::vec16(B, ldb);
  const int64_t split = ws_ok ? hpvm::entry_split_bytes(entry, m, n, k) : 0;
  if (entry && entry->launch_staged)
    e = entry->launch_staged(a, workspace, s);
  else if (split > 0 && workspace && (uintptr_t)workspace % 16 == 0 && workspace_bytes >= split)
    e = entry->launch_split(a, workspace, s);
  else if (entry)
    e = entry->launch(a, false, false, s);
  else if (is_flat(*tile))
    e = hpvm::launch_flat(a, tile->tile_n, tile->tile_m, s);
  else
    e = hpvm::launch_literal(a, tile->tile_n, tile->tile_m, s);
  return e == hipSuccess ? ok() : hip_fail(e, "sgemm launch");
}

}  // namespace

extern "C" {

int hpvm_sgemm(int64_t m, int64_t n, int64_t k, float alpha, const float* A, int64_t lda, const float* B,
               int64_t ldb, float beta, float* C, int64_t ldc, int32_t prec, const hpvm_tile* tile, void* stream) {
  return sgemm_impl(m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, prec, tile, false, nullptr, 0, stream);
}

int hpvm_sgemm_ws(int64_t m, int64_t n, int64_t k, float alpha, const float* A, int64_t lda, const float* B,
                  int64_t ldb, float beta, float* C, int64_t ldc, int32_t prec, const hpvm_tile* tile,
                  void* workspace, int64_t workspace_bytes, void* stream) {
  return sgemm_impl(m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, prec, tile, true, workspace, workspace_bytes,
                    stream);
}

int hpvm_sgemm_into(int64_t m, int64_t n, int64_t k, float alpha, const float* A, int64_t lda, const float* B,
                    int64_t ldb, float beta, const float* C, int64_t ldc, float* D, int64_t ldd, int32_t prec,
                    const hpvm_tile* tile, void* workspace, int64_t workspace_bytes, void* stream) {
  bool reads_ab = false;
  int rc = hpvm::check_operands("", m, n, k, alpha, A, lda, B, ldb, &reads_ab);
  if (rc != HPVM_OK) return rc;
  const bool reads_c = m > 0 && n > 0 && beta != 0.0f;
  if (reads_c && !C) return fail(HPVM_INVALID_ARG, "argument 10: C is NULL (beta != 0)");
  if (ldc < std::max<int64_t>(n, 1))
    return fail(HPVM_INVALID_ARG, "argument 11: ldc = %lld < max(1, n)", (long long)ldc);
  rc = hpvm::check_output("", m, n, k, A, lda, B, ldb, D, ldd, reads_ab, kIntoNos.c, kIntoNos.c_name);
  if (rc != HPVM_OK) return rc;
  if (reads_c && !(C == D && ldc == ldd)) {
    uintptr_t c0, c1, d0, d1;
    hpvm::matrix_extent(C, m, n, ldc, &c0, &c1);
    hpvm::matrix_extent(D, m, n, ldd, &d0, &d1);
    if (c0 < d1 && d0 < c1) return fail(HPVM_INVALID_ARG, "argument 12: D overlaps C without being C itself");
  }
  return sgemm_impl(m, n, k, alpha, A, lda, B, ldb, beta, D, ldd, prec, tile, true, workspace, workspace_bytes, stream,
                    reads_c ? C : nullptr, ldc, kIntoNos);
}

int hpvm_sgemm_workspace_bytes(int64_t m, int64_t n, int64_t k, int32_t prec, const hpvm_tile* tile,
                               int64_t* bytes) {
  if (m < 0 || n < 0 || k < 0) return fail(HPVM_INVALID_ARG, "sizes must be >= 0");
  if (!valid_prec(prec)) return fail(HPVM_INVALID_ARG, "argument 4: unknown precision %d", prec);
  if (!bytes) return fail(HPVM_INVALID_ARG, "argument 6: bytes is NULL");
  hpvm_tile tuned;
  if (!tile && choose_tile(prec, m, n, k, true, -1, &tuned)) tile = &tuned;
  const hpvm::MfmaEntry* entry;
  int rc = resolve(prec, tile, &entry, 5);
  if (rc != HPVM_OK) return rc;
  *bytes = std::max(hpvm::entry_workspace_bytes(entry, m, n, k), hpvm::entry_split_bytes(entry, m, n, k));
  return ok();
}

int64_t hpvm_sgemm_or_bytes(int64_t m, int64_t n, int64_t k, float alpha, const float* A, int64_t lda, const float* B,
                            int64_t ldb, float beta, float* C, int64_t ldc, int32_t prec, const hpvm_tile* tile,
                            void* stream) {
  int64_t need = 0;
  if (m >= 0 && n >= 0 && k >= 0 && valid_prec(prec)) {
    hpvm_tile tuned;
    const hpvm_tile* t = tile;
    if (!t && choose_tile(prec, m, n, k, true, -1, &tuned)) t = &tuned;
    const hpvm::MfmaEntry* entry;
    if (resolve(prec, t, &entry, 13) == HPVM_OK)
      need = std::max(hpvm::entry_workspace_bytes(entry, m, n, k), hpvm::entry_split_bytes(entry, m, n, k));
  }
  // hpvm_sgemm checks every argument; where it is not to be called, so does this.
  if (need == 0) return hpvm_sgemm(m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, prec, tile, stream);
  bool reads_ab = false;
  const int rc = hpvm::check_gemm_args("", m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, &reads_ab);
  if (rc != HPVM_OK) return rc;
  hpvm::clear_error();
  return need;
}

int hpvm_launch_root(const hpvm_root_in* r, void* stream) {
  if (!r) return fail(HPVM_INVALID_ARG, "argument 1: args is NULL");
  if (r->block_x <= 0 || r->block_y <= 0 || r->grid_x < 0 || r->grid_y < 0)
    return fail(HPVM_INVALID_ARG, "block and grid counts must be positive");
  const int64_t lanes = (int64_t)r->block_x * r->block_y;
  if (lanes > 1024 || lanes % hpvm::kWave)
    return fail(HPVM_UNSUPPORTED, "block_x * block_y = %lld must be a multiple of 64, at most 1024",
                (long long)lanes);
  const int64_t m = (int64_t)r->grid_y * r->block_y;
  const int64_t n = (int64_t)r->grid_x * r->block_x;
  const int64_t k = r->k;
  if (k < 0) return fail(HPVM_INVALID_ARG, "k = %lld < 0", (long long)k);
  // The byte extents stand in for the sizes the paper's runtime copies.
  const int64_t f = (int64_t)sizeof(float);
  if (m > 0 && n > 0) {
    if (k > 0 && r->alpha != 0.0f) {
      if (r->lda < (k > 1 ? k : 1) || r->bytesA < ((m - 1) * r->lda + k) * f)
        return fail(HPVM_INVALID_ARG, "bytesA / lda too small for %lld x %lld", (long long)m, (long long)k);
      if (r->ldb < (n > 1 ? n : 1) || r->bytesB < ((k - 1) * r->ldb + n) * f)
        return fail(HPVM_INVALID_ARG, "bytesB / ldb too small for %lld x %lld", (long long)k, (long long)n);
    }
    if (r->ldc < (n > 1 ? n : 1) || r->bytesC < ((m - 1) * r->ldc + n) * f)
      return fail(HPVM_INVALID_ARG, "bytesC / ldc too small for %lld x %lld", (long long)m, (long long)n);
  }
  hpvm_tile t{r->block_y, r->block_x, r->block_y, 1, 1, 1};
  return hpvm_sgemm(m, n, k, r->alpha, r->A, r->lda > 0 ? r->lda : 1, r->B, r->ldb > 0 ? r->ldb : 1,
                    r->beta, r->C, r->ldc > 0 ? r->ldc : 1, HPVM_PREC_FP32, &t, stream);
}

int hpvm_wait(void* stream) {
  if (inject("wait")) return fail(HPVM_HIP_ERROR, "injected wait failure (HPVM_FAULT_INJECT)");
  hipError_t e = hipStreamSynchronize(reinterpret_cast<hipStream_t>(stream));
  return e == hipSuccess ? ok() : hip_fail(e, "stream synchronize");
}

}  // extern "C"

// ---------------------------------------------------------------------------
// hpvm_sgemm_noalloc: hpvm_sgemm_ws whose workspace is a fixed array of
// device memory that the library's code object carries, so that the call
// itself allocates nothing.  Each device that loads the library holds its
// own copy of the array (at its own address) until the process ends.
// ---------------------------------------------------------------------------
namespace {

// Device-side storage.  On the host this name is only a stand-in for the
// symbol: its device address, per device, comes from hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[HPVM_NOALLOC_SCRATCH_BYTES];

constexpr int kScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_at[kScratchDevices] = {};

// The current device's copy of the array, looked up once per device with
// that device current.
int scratch_of_current_device(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  if (dev < 0 || dev >= kScratchDevices)
    return fail(HPVM_UNSUPPORTED, "device %d: the no-allocation entry point supports devices 0..%d", dev,
                kScratchDevices - 1);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_at[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
    if (!p || (uintptr_t)p % 256) return fail(HPVM_HIP_ERROR, "scratch symbol has no usable device address");
    g_scratch_at[dev] = p;
  }
  *out = g_scratch_at[dev];
  return HPVM_OK;
}

}  // namespace

extern "C" int hpvm_sgemm_noalloc(int64_t m, int64_t n, int64_t k, float alpha, const float* A, int64_t lda,
                                  const float* B, int64_t ldb, float beta, float* C, int64_t ldc, int32_t prec,
                                  const hpvm_tile* tile, void* stream) {
  // Checks in argument order, then the lowering hpvm_sgemm_ws would run with
  // a workspace of HPVM_NOALLOC_SCRATCH_BYTES; nothing touches the device
  // before all of them pass.
  bool reads_ab = false;
  int rc = hpvm::check_gemm_args("", m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, &reads_ab);
  if (rc != HPVM_OK) return rc;
  if (!valid_prec(prec)) return fail(HPVM_INVALID_ARG, "argument 12: unknown precision %d", prec);
  const int64_t cap = HPVM_NOALLOC_SCRATCH_BYTES;
  hpvm_tile chosen;
  const hpvm_tile* t = tile;
  if (!t && choose_tile(prec, m, n, k, true, cap, &chosen)) t = &chosen;
  const hpvm::MfmaEntry* entry;
  rc = resolve(prec, t, &entry, 13);
  if (rc != HPVM_OK) return rc;
  const int64_t need = hpvm::entry_workspace_bytes(entry, m, n, k);
  if (need > cap && reads_ab && m > 0 && n > 0)
    return fail(HPVM_WORKSPACE_TOO_SMALL,
                "argument 13: this tile needs %lld bytes of scratch; the no-allocation entry point has %lld "
                "(use hpvm_sgemm_ws with a workspace of that size)",
                (long long)need, (long long)cap);
  void* ws = nullptr;
  if (reads_ab && m > 0 && n > 0 && (need > 0 || hpvm::entry_split_bytes(entry, m, n, k) > 0)) {
    if (inject("launch")) return fail(HPVM_HIP_ERROR, "injected launch failure (HPVM_FAULT_INJECT)");
    rc = scratch_of_current_device(&ws);
    if (rc != HPVM_OK) return rc;
  }
  return sgemm_impl(m, n, k, alpha, A, lda, B, ldb, beta, C, ldc, prec, t, true, ws, ws ? cap : 0, stream);
}
