"""BF16 products and gradients beside an open streaming graph.

The graph's two workgroups a CU leave 87 KB of LDS.  A kernel that needs more
starts only when the stream has ended, so products of less than 256 tiles of
256 x 256 take tiles that fit, and the staged ones of 2^31 multiply-adds and
more the 64 KB tile; whole-tile ones whose 128 x 128 tiles cover the CUs, of
fewer multiply-adds, and split contractions never did."""
import pytest

import paper_1611_00860_amd as hp

ROOM = 87 * 1024
# Staged or direct, ragged or whole, around 2^31 multiply-adds and both tile limits.
SIZES = [(2048, 4096, 512), (4096, 2048, 512), (1280, 5000, 512), (2000, 2000, 768), (8192, 1024, 1024),
         (8192, 1024, 4096), (768, 10254, 638), (3324, 2176, 60), (2001, 2003, 401), (8128, 416, 896),
         (3999, 4001, 130)]


@pytest.mark.parametrize("m,n,k", SIZES)
def test_default_tile_leaves_room(m, n, k):
    hp.autotune_clear()
    for ws in (1 << 40, 32 << 20, None):
        d = hp.describe(m, n, k, "bf16", workspace_bytes=ws)
        whole = d["tile"][:3] == (128, 128, 32) and d["tile"][5] == 4 and n % 4 == 0 and k % 32 == 0
        if not (whole and (m * n * k < 2 ** 31 or ws != 1 << 40)):
            assert d["alloc_bytes"] <= ROOM, (ws, d["tile"])


@pytest.mark.gpu
def test_products_run_beside_an_open_stream(gpu):
    import time

    import torch

    def finish(what, t0):
        torch.cuda.current_stream().synchronize()
        assert time.time() - t0 < 8, what

    with gpu.SgemmStream(capacity=4, idle_ms=10000):
        for m, n, k in SIZES:
            print(f"case: bf16 beside a stream {m}x{n}x{k}", flush=True)
            A, B, C = (torch.rand(*s, device="cuda") for s in ((m, k), (k, n), (m, n)))
            t0 = time.time()
            gpu.sgemm(A, B, C, 1.0, 0.5, prec="bf16")
            finish((m, n, k), t0)
        for prec, m, n, k in [("bf16", 1991, 1956, 810), ("bf16x3", 1502, 1675, 1055)]:
            print(f"case: {prec} backward beside a stream {m}x{n}x{k}", flush=True)
            A, B, C, G = (torch.rand(*s, device="cuda") for s in ((m, k), (k, n), (m, n), (m, n)))
            t0 = time.time()
            gpu.sgemm_backward(A, B, C, G, 1.0, 0.5, prec=prec)
            finish((prec, m, n, k), t0)
