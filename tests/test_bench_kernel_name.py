"""The kernel that bench.py names for a tile is one the library has."""
import subprocess

import bench
import paper_1611_00860_amd as hp
from paper_1611_00860_amd import _lib


def test_named_kernels_exist():
    symbols = subprocess.run(["nm", "-C", _lib.LIB_PATH], capture_output=True, text=True, check=True).stdout
    names = set()
    for tile in hp.tile_menu("fp32"):
        for m, n, k in [(4096, 4096, 4096), (8192, 4096, 2048), (1000, 1000, 1024), (1000, 1003, 777), (64, 3, 40)]:
            names.add(bench.fp32_kernel_name(tile, m, n, k))
            assert f"hpvm::{bench.fp32_kernel_name(tile, m, n, k)}(" in symbols, (tile, m, n, k)
    # Each tile's own, the aligned tiles' form for edges, the narrow product's.
    aligned = sum(t[4] == 128 for t in hp.tile_menu("fp32"))
    assert len(names) == len(hp.tile_menu("fp32")) + aligned + 1
