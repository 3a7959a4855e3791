"""The DMA-fed FP32 loop for any size and alignment, at the sizes where it can
go wrong: integer inputs, so every sum is exact in any order and the result
must equal the oracle's bit for bit; rows are padded with NaN, which a value
taken from outside a matrix would spread."""
import numpy as np
import pytest

import oracle
from gpu_util import to_dev, to_host
from paper_1611_00860_amd import inputs

pytestmark = pytest.mark.gpu

# Columns: one 16-byte unit, a partial one, a tile and one more or less of
# it; depths: inside a slab, whole slabs, one over, one short.
SIZES = [(1, 4, 1), (3, 5, 31), (4, 3, 33), (33, 31, 96), (63, 66, 100), (65, 127, 64), (127, 65, 257), (130, 129, 95),
         (257, 259, 130), (5, 300, 511)]


def run(hp, A, B, C, alpha, beta, tile, pad, misalign):
    import torch

    dA, dB, dC = (to_dev(x, pad, misalign) for x in (A, B, C))
    hp.sgemm(dA, dB, dC, alpha, beta, tile=tile)
    torch.cuda.synchronize()
    return to_host(dC)


@pytest.mark.parametrize("m,n,k", SIZES)
@pytest.mark.parametrize("pad,misalign", [(0, False), (3, True)])
def test_any_size_integers(gpu, m, n, k, pad, misalign):
    A, B, C = inputs.sgemm_operands(m, n, k, seed=m + n + k, dist="int")
    ref = oracle.sgemm(A, B, C, 1.0, -2.0)
    for tile in [None] + [t for t in gpu.tile_menu("fp32") if t[4] != 128]:
        print(f"case: {m}x{n}x{k} pad {pad} misalign {misalign} tile {tile}", flush=True)
        got = run(gpu, A, B, C, 1.0, -2.0, tile, pad, misalign)
        assert np.array_equal(got, ref), tile
    nan_c = np.full_like(C, np.nan)
    got = run(gpu, A, B, nan_c, 1.0, 0.0, None, pad, misalign)
    assert np.array_equal(got, oracle.sgemm(A, B, None, 1.0, 0.0))


@pytest.mark.parametrize("m,n,k", [(16, 520, 2048), (33, 35, 2051), (64, 64, 4096), (1, 5, 9000)])
def test_ragged_split_contraction_integers(gpu, m, n, k):
    """Shallow outputs over a long contraction run in slices with a workspace (and whole without one)."""
    A, B, C = inputs.sgemm_operands(m, n, k, seed=k, dist="int")
    product = A.astype(np.float64) @ B.astype(np.float64)
    assert gpu.workspace_bytes(m, n, k, "fp32") > 0 and np.abs(product).max() < 2 ** 24
    print(f"case: split {m}x{n}x{k}", flush=True)
    for pad, misalign in ((0, False), (1, True)):
        got = run(gpu, A, B, C, 1.0, 2.0, None, pad, misalign)
        assert np.array_equal(got, product + 2.0 * C.astype(np.float64))
        got = run(gpu, A, B, np.full_like(C, np.nan), 1.0, 0.0, None, pad, misalign)
        assert np.array_equal(got, product)


@pytest.mark.parametrize("m,n,k", [(33, 35, 37), (64, 128, 64), (130, 67, 129), (5, 260, 300), (257, 3, 66), (70, 90, 2)])
@pytest.mark.parametrize("pad,misalign", [(0, False), (3, True)])
def test_any_size_backward_integers(gpu, m, n, k, pad, misalign):
    """Both gradients, dC_in and both scalars, every FP32 tile, each alone and
    together: exact on integers (all sums stay below 2^24)."""
    import torch

    A, B, C, G = (np.clip(x, -2, 2) for x in inputs.backward_operands(m, n, k, seed=m + n + k, dist="int"))
    a, b, c, g = (x.astype(np.float64) for x in (A, B, C, G))
    ref = {"dA": 2 * (g @ b.T), "dB": 2 * (a.T @ g), "dC_in": -1 * g, "dalpha": (g * (a @ b)).sum(),
           "dbeta": (g * c).sum()}
    assert max(np.abs(v).max() for v in ref.values()) < 2 ** 24
    dev = [to_dev(x, pad, misalign) for x in (A, B, C, G)]
    for tile in [None] + gpu.backward_menu("fp32"):
        print(f"case: backward {m}x{n}x{k} pad {pad} misalign {misalign} tile {tile}", flush=True)
        for need in (("dA", "dB", "dC_in", "dalpha", "dbeta"), ("dA",), ("dB", "dbeta"), ("dalpha",), ("dA", "dB")):
            got = gpu.sgemm_backward(*dev, 2.0, -1.0, need=need, tile=tile)
            torch.cuda.synchronize()
            for name in need:
                assert np.array_equal(to_host(got[name]), ref[name]), (tile, need, name)


@pytest.mark.parametrize("m,n,k", [(33, 35, 37), (64, 128, 64), (130, 67, 129), (5, 260, 300), (257, 3, 66), (70, 90, 2)])
@pytest.mark.parametrize("prec", ["bf16", "bf16x3"])
def test_any_size_backward_integers_bf16(gpu, prec, m, n, k):
    """The same for the fused BF16 and bf16x3 tiles (integers to 2 are exact in
    bfloat16, their lo parts zero)."""
    import torch

    A, B, C, G = (np.clip(x, -2, 2) for x in inputs.backward_operands(m, n, k, seed=m + n + k, dist="int"))
    a, b, c, g = (x.astype(np.float64) for x in (A, B, C, G))
    ref = {"dA": 2 * (g @ b.T), "dB": 2 * (a.T @ g), "dC_in": -1 * g, "dalpha": (g * (a @ b)).sum(),
           "dbeta": (g * c).sum()}
    assert max(np.abs(v).max() for v in ref.values()) < 2 ** 24
    for pad, misalign in ((0, False), (3, True)):
        dev = [to_dev(x, pad, misalign) for x in (A, B, C, G)]
        for tile in [None] + [t for t in gpu.backward_menu(prec) if t[5] == 2 and t[4] != 128]:
            print(f"case: backward {prec} {m}x{n}x{k} pad {pad} tile {tile}", flush=True)
            for need in (("dA", "dB", "dC_in", "dalpha", "dbeta"), ("dA",), ("dB", "dbeta"), ("dalpha",), ("dA", "dB")):
                got = gpu.sgemm_backward(*dev, 2.0, -1.0, prec=prec, need=need, tile=tile)
                torch.cuda.synchronize()
                for name in need:
                    assert np.array_equal(to_host(got[name]), ref[name]), (tile, need, name)


@pytest.mark.parametrize("prec", ["bf16", "bf16x3"])
@pytest.mark.parametrize("m,n,k", [(16, 520, 2048), (33, 35, 2051), (64, 64, 1024), (1, 5, 9000)])
def test_ragged_split_contraction_integers_bf16(gpu, prec, m, n, k):
    """The 32 x 128 tile's slices, through a workspace and as one launch."""
    import torch

    A, B, C = (np.clip(x, -2, 2) for x in inputs.sgemm_operands(m, n, k, seed=m + k, dist="int"))
    ref = oracle.sgemm(A, B, C, 1.0, -2.0)
    for pad, misalign in ((0, False), (3, True)):
        for workspace in (None, False):
            print(f"case: split {prec} {m}x{n}x{k} pad {pad} workspace {workspace}", flush=True)
            dA, dB, dC = (to_dev(x, pad, misalign) for x in (A, B, C))
            gpu.sgemm(dA, dB, dC, 1.0, -2.0, prec=prec, tile=(32, 128, 32, 32, 32, 2), workspace=workspace)
            torch.cuda.synchronize()
            assert np.array_equal(to_host(dC), ref)


def test_grouped_narrow_instances_replayed(gpu):
    """Instances narrower than a 16-byte transfer beside ragged and whole ones;
    every run and every replay starts from a cleared tile counter."""
    import torch

    sizes = [(33, 3, 70), (5, 2, 9), (64, 1, 31), (130, 67, 129), (257, 300, 40), (128, 128, 64), (3, 4, 1)]
    ops = [inputs.sgemm_operands(m, n, k, seed=i, dist="int") for i, (m, n, k) in enumerate(sizes)]
    refs = [oracle.sgemm(A, B, C, 1.0, -2.0) for A, B, C in ops]
    As, Bs, Cs = ([to_dev(o[j], 3, True) for o in ops] for j in range(3))
    plan = gpu.GroupedPlan(As, Bs, Cs, [1.0] * len(sizes), [-2.0] * len(sizes))
    graph = plan.capture()
    for run in (plan.run, graph.launch, graph.launch, plan.run, graph.launch):
        for c, o in zip(Cs, ops):
            c.copy_(torch.from_numpy(o[2]))
        print(f"case: grouped narrow {run.__qualname__}", flush=True)
        run()
        torch.cuda.synchronize()
        for c, ref, size in zip(Cs, refs, sizes):
            assert np.array_equal(to_host(c), ref), size


@pytest.mark.parametrize("prec", ["fp32", "bf16", "bf16x3"])
def test_small_products_run_beside_an_open_stream(gpu, prec):
    """An open streaming graph holds part of every CU until it idles out: the
    default tiles of products that give fewer than 256 tiles of 128 x 128 fit
    in the rest."""
    import time

    import torch

    with gpu.SgemmStream(capacity=4, idle_ms=10000):
        t0 = time.time()
        for m, n, k in [(128, 128, 128), (200, 7000, 512), (1500, 1100, 300), (300, 300, 2048)]:
            print(f"case: beside a stream {prec} {m}x{n}x{k}", flush=True)
            A, B, C, G = (to_dev(x) for x in inputs.backward_operands(m, n, k, seed=3))
            gpu.sgemm(A, B, C, 1.0, 0.5, prec=prec)
            torch.cuda.current_stream().synchronize()
            if m * n * k < 2 ** 28:
                gpu.sgemm_backward(A, B, C, G, 1.0, 0.5, prec=prec)
                torch.cuda.current_stream().synchronize()
        assert time.time() - t0 < 8
