"""Slabs of the deepest contractions the entry points take (2^31 - 1): a count
that wraps leaves a loop without slabs, and its output zero.  Checked where the
kernels take it from, in the host compiler (a wrapping sum is no constant)."""
import os
import re
import subprocess

from paper_1611_00860_amd import build

SOURCE = r"""
#include "mfma_bf16_any.hpp"
#include "mfma_f32_any.hpp"
using namespace hpvm;
constexpr bool covers(int k, int slab) {
  const long long n = slab_count(k, slab);
  return n * slab >= k && (n - 1) * slab < k;
}
constexpr bool all(int slab) {
  for (int d = 0; d <= 2 * slab; ++d)
    if (!covers(2147483647 - d, slab) || (d > 0 && !covers(d, slab))) return false;
  return slab_count(0, slab) == 0;
}
static_assert(all(8) && all(16) && all(32) && all(64) && all(128), "slab counts");

// The loop for any size leaves deeper contractions than its own sum holds to the loops that count with slab_count.
constexpr GemmArgs deep(int k) {
  GemmArgs a{};
  a.m = a.n = 8;
  a.lda = a.ldb = a.ldc = a.ldci = 8;
  a.k = k;
  return a;
}
static_assert(f32_any_fits(deep(1), true, false) && f32_any_fits(deep(kAnyDepth), true, false), "up to kAnyDepth");
static_assert(!f32_any_fits(deep(kAnyDepth + 1), true, false) && !f32_any_fits(deep(2147483647), true, false), "");
static_assert(!f32_any_fits(deep(2147483647), false, true) && !f32_any_fits(deep(2147483647), false, false), "");
static_assert(kAnyDepth + kAnySlab == 2147483647, "an int");
static_assert(AnyShape<32, 32, 32, 32, 32, false, true, 2, 4>::kSlab == kAnySlab, "the deepest slab");
"""


def test_slab_counts_of_the_deepest_contractions(tmp_path):
    src = tmp_path / "slabs.hip"
    src.write_text(SOURCE)
    r = subprocess.run([build.HIPCC, "--offload-host-only", "-fsyntax-only", "-std=c++17", "-I", build.INCLUDE, "-I",
                        build.CSRC, str(src)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]


def test_the_other_loops_take_their_slabs_from_it():
    for name in sorted(os.listdir(build.CSRC)):
        with open(os.path.join(build.CSRC, name)) as f:
            text = f.read()
        if name != "mfma_f32_any.hpp":
            assert not re.search(r"\bp\d?\.k \+ [\w:]+ - 1\) / ", text), name
