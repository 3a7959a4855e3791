"""One FP32 gradient alone where one of m and n is small: its tile is not the one
both gradients together would take.  Integer inputs: exact in any order."""
import numpy as np
import pytest

from gpu_util import to_dev, to_host
from paper_1611_00860_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k", [(3000, 20, 130), (20, 3001, 130), (9, 2050, 300), (2047, 5, 64)])
@pytest.mark.parametrize("pad,misalign", [(0, False), (3, True)])
def test_single_gradients_integers(gpu, m, n, k, pad, misalign):
    import torch

    host = [np.clip(x, -2, 2) for x in inputs.backward_operands(m, n, k, seed=m + n, dist="int")]
    a, b, _, g = (x.astype(np.float64) for x in host)
    ref = {"dA": 2 * (g @ b.T), "dB": 2 * (a.T @ g), "dC_in": -1 * g}
    dev = [to_dev(x, pad, misalign) for x in host]
    for need in (("dA",), ("dB",), ("dA", "dC_in"), ("dB", "dC_in"), ("dA", "dB")):
        print(f"case: backward {m}x{n}x{k} need {need} pad {pad}", flush=True)
        got = gpu.sgemm_backward(*dev, 2.0, -1.0, need=need)
        torch.cuda.synchronize()
        for name in need:
            assert np.array_equal(to_host(got[name]), ref[name]), (need, name)
