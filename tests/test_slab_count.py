"""Slabs of the deepest contractions the entry points take (2^31 - 1): a count
that wraps leaves a loop without slabs, and its output zero.  Checked where the
kernels take it from, in the host compiler."""
import os
import re
import subprocess

from paper_1611_00860_amd import build

SOURCE = r"""
#include "mfma_bf16_any.hpp"
#include "mfma_f32_any.hpp"
using hpvm::slab_count;
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
static_assert(hpvm::AnyShape<32, 32, 32, 32, 32, false, true, 2, 4>::kSlab == 128, "the deepest slab");
"""


def test_slab_counts_of_the_deepest_contractions(tmp_path):
    src = tmp_path / "slabs.hip"
    src.write_text(SOURCE)
    r = subprocess.run([build.HIPCC, "--offload-host-only", "-fsyntax-only", "-std=c++17", "-I", build.INCLUDE, "-I",
                        build.CSRC, str(src)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]


def test_every_loop_takes_its_slabs_from_it():
    for name in sorted(os.listdir(build.CSRC)):
        with open(os.path.join(build.CSRC, name)) as f:
            text = f.read()
        assert not re.search(r"\bp\d?\.k \+ [\w:]+ - 1\) / ", text), name
