"""Rows 2^22 floats and more apart, which the DMA-fed loop for any size leaves to
the register-staged ones, and one float less, where its 32-bit offsets within
a tile reach furthest.  Integer inputs: exact in any order."""
import numpy as np
import pytest

import oracle
from gpu_util import to_host
from paper_1611_00860_amd import inputs

pytestmark = pytest.mark.gpu

FAR = 1 << 22
PITCHES = [FAR - 1, FAR, FAR + 4]


def far(x, pitch):
    """x on the GPU with rows `pitch` floats apart, NaN between them (or as it is)."""
    import torch

    t = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    if not pitch:
        return t
    r, c = x.shape
    flat = torch.full(((r - 1) * pitch + c,), float("nan"), device="cuda")
    view = flat.as_strided((r, c), (pitch, 1))
    view.copy_(t)
    return view


@pytest.mark.parametrize("pitch", PITCHES)
@pytest.mark.parametrize("prec", ["fp32", "bf16", "bf16x3"])
def test_sgemm(gpu, prec, pitch):
    import torch

    m, n, k = 70, 66, 37
    A, B, C = (np.clip(x, -2, 2) for x in inputs.sgemm_operands(m, n, k, seed=7, dist="int"))
    ref = oracle.sgemm(A, B, C, 1.0, -2.0)
    small = (64, 64, 16, 32, 32, 2) if prec == "fp32" else (64, 64, 32, 32, 32, 2)
    wide = next(t for t in gpu.tile_menu(prec) if t[5] == 2 and t[0] == 128 and t[1] == 128)
    for which in ("A", "B", "C", "ABC"):
        for tile in (None, small, wide):
            print(f"case: {prec} pitch {pitch} of {which} tile {tile}", flush=True)
            a, b, c = (far(x, pitch if name in which else 0) for name, x in zip("ABC", (A, B, C)))
            gpu.sgemm(a, b, c, 1.0, -2.0, prec=prec, tile=tile)
            torch.cuda.synchronize()
            assert np.array_equal(to_host(c), ref), (which, tile)


def test_furthest_offset_of_a_tile(gpu):
    """256 rows a float less than 2^22 apart: the last one starts 16 KB under 4 GB from the tile's corner."""
    import torch

    A, B, C = inputs.sgemm_operands(257, 40, 33, seed=8, dist="int")
    tile = next(t for t in gpu.tile_menu("fp32") if t[:2] == (256, 128) and t[5] == 2)
    print(f"case: furthest offset tile {tile}", flush=True)
    c = far(C, FAR - 1)
    gpu.sgemm(far(A, FAR - 1), far(B, 0), c, 1.0, -2.0, tile=tile)
    torch.cuda.synchronize()
    assert np.array_equal(to_host(c), oracle.sgemm(A, B, C, 1.0, -2.0))


@pytest.mark.parametrize("pitch", PITCHES)
def test_consumer_grouped_and_stream(gpu, pitch):
    import torch

    m, n, k = 70, 66, 37
    A, B, C = inputs.sgemm_operands(m, n, k, seed=9, dist="int")
    ref = oracle.sgemm(A, B, C, 1.0, -2.0)
    for which in ("A", "B", "C", "ABC"):
        print(f"case: consumer, grouped, stream pitch {pitch} of {which}", flush=True)
        a, b, c = (far(x, pitch if name in which else 0) for name, x in zip("ABC", (A, B, C)))
        d = gpu.sgemm_consumer(a, b, c, 1.0, -2.0, op="relu", D=far(np.zeros_like(C), pitch if which == "C" else 0))
        torch.cuda.synchronize()
        assert np.array_equal(to_host(d), np.maximum(ref, 0))
        plan = gpu.GroupedPlan([a], [b], [c], [1.0], [-2.0])
        plan.run()
        torch.cuda.synchronize()
        assert np.array_equal(to_host(c), ref)
        c.copy_(torch.from_numpy(C))
        torch.cuda.synchronize()
        with gpu.SgemmStream(capacity=2) as stream:
            stream.push(a, b, c, 1.0, -2.0)
            stream.pop()
        assert np.array_equal(to_host(c), ref)


@pytest.mark.parametrize("pitch", PITCHES)
@pytest.mark.parametrize("prec", ["fp32", "bf16", "bf16x3"])
def test_backward(gpu, prec, pitch):
    import torch

    m, n, k = 70, 66, 37
    host = [np.clip(x, -2, 2) for x in inputs.backward_operands(m, n, k, seed=10, dist="int")]
    a, b, c, g = (x.astype(np.float64) for x in host)
    ref = {"dA": 2 * (g @ b.T), "dB": 2 * (a.T @ g), "dC_in": -1 * g, "dalpha": (g * (a @ b)).sum(),
           "dbeta": (g * c).sum()}
    odd = (64, 64, 16, 32, 32, 2) if prec == "fp32" else (64, 64, 32, 32, 32, 2)
    for which in ("A", "B", "G", "ABG"):
        dev = [far(x, pitch if name in which else 0) for name, x in zip("ABCG", host)]
        for need in (("dA", "dB", "dC_in", "dalpha", "dbeta"), ("dA", "dB"), ("dalpha",)):
            for tile in (None, odd):
                print(f"case: backward {prec} pitch {pitch} of {which} need {need} tile {tile}", flush=True)
                got = gpu.sgemm_backward(*dev, 2.0, -1.0, prec=prec, need=need, tile=tile)
                torch.cuda.synchronize()
                for name in need:
                    assert np.array_equal(to_host(got[name]), ref[name]), (which, need, tile, name)
