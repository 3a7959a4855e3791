"""hpvm_sgemm_backward with outputs over its inputs: the gradients of the call
on matrices of their own, whatever the tile.  Integer inputs, so every sum is
exact in any order and any tile."""
import ctypes

import numpy as np
import pytest

from gpu_util import to_dev, to_host
from paper_1611_00860_amd import _lib, inputs

pytestmark = pytest.mark.gpu

# Which output lies on which input.
ONE_PASS_EACH = [("C",), ("A",), ("B",), ("C", "A"), ("C", "B"), ("Cin", "A"), ("Cin", "B")]
BOTH = [("A", "B"), ("C", "A", "B")]


def reference(A, B, C, G):
    a, b, c, g = (x.astype(np.float64) for x in (A, B, C, G))
    ref = {"dA": 2 * (g @ b.T), "dB": 2 * (a.T @ g), "dC": -1 * g, "dalpha": (g * (a @ b)).sum(),
           "dbeta": (g * c).sum()}
    assert max(np.abs(v).max() for v in ref.values()) < 2 ** 24
    return ref


def call(gpu, host, over, prec, tile, scalars=True, pad=0, misalign=False):
    """The five outputs with dA on A ("A"), dB on B ("B"), dC_in on G ("C") or C_in ("Cin")."""
    import torch

    (m, k), n = host[0].shape, host[1].shape[1]
    A, B, C, G = (to_dev(x, pad, misalign) for x in host)
    new = lambda t: torch.full(t.shape, float("nan"), device="cuda")
    out = {"dA": A if "A" in over else new(A), "dB": B if "B" in over else new(B),
           "dC": G if "C" in over else C if "Cin" in over else new(G)}
    scal = torch.full((2,), float("nan"), device="cuda")
    ws = torch.empty(max(gpu.backward_workspace_bytes(m, n, k, prec, tile), 16), dtype=torch.uint8, device="cuda")
    args = []
    for t in (A, B, C, G, out["dA"], out["dB"], out["dC"]):
        args += [t.data_ptr(), t.stride(0)]
    t = ctypes.byref(_lib.Tile(*tile)) if tile else None
    rc = _lib.load().hpvm_sgemm_backward(m, n, k, 2.0, -1.0, *args, scal.data_ptr() if scalars else None,
                                         scal.data_ptr() + 4 if scalars else None, gpu.PREC[prec], t, ws.data_ptr(),
                                         ws.numel(), torch.cuda.current_stream().cuda_stream)
    assert rc == 0, gpu.last_error()
    torch.cuda.synchronize()
    got = {name: to_host(x) for name, x in out.items()}
    if scalars:
        got["dalpha"], got["dbeta"] = (float(x) for x in scal)
    return got


def check(gpu, host, ref, over, prec, tile, **kw):
    print(f"case: backward {prec} {host[0].shape} n {host[1].shape[1]} outputs on {over} tile {tile} {kw}", flush=True)
    got = call(gpu, host, over, prec, tile, **kw)
    for name, x in got.items():
        assert np.array_equal(x, ref[name]), (over, tile, name)


@pytest.mark.parametrize("prec", ["fp32", "bf16", "bf16x3"])
@pytest.mark.parametrize("m,n,k", [(130, 67, 129), (5, 3, 64), (256, 512, 256), (700, 900, 500)])
def test_outputs_over_inputs(gpu, prec, m, n, k):
    host = [np.clip(x, -1, 1) for x in inputs.backward_operands(m, n, k, seed=m + n, dist="int")]
    ref = reference(*host)
    for tile in [None] + list(gpu.backward_menu(prec)):
        for over in ONE_PASS_EACH:
            check(gpu, host, ref, over, prec, tile)
        if tile and tile[5] == 3:
            for over in BOTH:
                check(gpu, host, ref, over, prec, tile)
    for over in ONE_PASS_EACH:
        check(gpu, host, ref, over, prec, None, scalars=False, pad=3, misalign=True)


@pytest.mark.parametrize("prec,m,n,k", [("fp32", 1024, 1024, 1024), ("fp32", 256, 512, 256), ("bf16", 300, 3000, 500),
                                        ("bf16x3", 300, 3000, 500), ("bf16", 128, 2048, 64)])
def test_both_gradients_in_place_without_a_tile(gpu, prec, m, n, k):
    """No order of separate launches serves dA on A with dB on B: the call takes a tile that reads copies."""
    host = [np.clip(x, -1, 1) for x in inputs.backward_operands(m, n, k, seed=m + n, dist="int")]
    ref = reference(*host)
    for over in BOTH + ONE_PASS_EACH:
        check(gpu, host, ref, over, prec, None)


@pytest.mark.parametrize("prec", ["fp32", "bf16", "bf16x3"])
def test_grad_c_over_the_products_operands(gpu, prec):
    """dC_in where A or B was (m = n = k): written once nothing reads that any more."""
    import torch

    host = [np.clip(x, -1, 1) for x in inputs.backward_operands(320, 320, 320, seed=9, dist="int")]
    ref = reference(*host)
    for tile in [None] + list(gpu.backward_menu(prec)):
        for where in (0, 1):
            print(f"case: backward {prec} dC_in over operand {where} tile {tile}", flush=True)
            mats = [to_dev(x) for x in host]
            dA, dB = torch.empty_like(mats[0]), torch.empty_like(mats[1])
            scal = torch.empty(2, device="cuda")
            ws = torch.empty(max(gpu.backward_workspace_bytes(320, 320, 320, prec, tile), 16), dtype=torch.uint8,
                             device="cuda")
            args = []
            for t in (*mats, dA, dB, mats[where]):
                args += [t.data_ptr(), 320]
            t = ctypes.byref(_lib.Tile(*tile)) if tile else None
            rc = _lib.load().hpvm_sgemm_backward(320, 320, 320, 2.0, -1.0, *args, scal.data_ptr(), scal.data_ptr() + 4,
                                                 gpu.PREC[prec], t, ws.data_ptr(), ws.numel(),
                                                 torch.cuda.current_stream().cuda_stream)
            assert rc == 0, gpu.last_error()
            torch.cuda.synchronize()
            for x, name in ((dA, "dA"), (dB, "dB"), (mats[where], "dC")):
                assert np.array_equal(to_host(x), ref[name]), (tile, where, name)
            assert float(scal[0]) == ref["dalpha"] and float(scal[1]) == ref["dbeta"]
