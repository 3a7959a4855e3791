"""hpvm_sgemm_into: the bits of the in-place call on a copy of C, for every
lowering, with C read from rows of another length and alignment than D's."""
import pytest

from gpu_util import to_dev
from paper_1611_00860_amd import HpvmError, inputs

pytestmark = pytest.mark.gpu

# Whole tiles, edges moved inward, ragged, split contractions, k = 0.
SIZES = [(256, 256, 128), (260, 132, 96), (130, 67, 129), (5, 3, 7), (256, 256, 2048), (33, 35, 2051), (48, 20, 0)]


@pytest.mark.parametrize("m,n,k", SIZES)
@pytest.mark.parametrize("prec", ["fp32", "bf16", "bf16x3"])
def test_into_equals_in_place_on_a_copy(gpu, m, n, k, prec):
    import torch

    A, B, C = inputs.sgemm_operands(m, n, k, seed=m + n + k)
    dA, dB = to_dev(A), to_dev(B)
    tiles = [None] + list(gpu.tile_menu(prec))
    if prec == "fp32":
        tiles += [(16, 16, 16, 1, 1, 1), (16, 16, 0, 1, 1, 0)]
    for tile in tiles:
        for pad, misalign in ((0, False), (3, True)):
            for alpha, beta in ((0.7, 0.3), (0.0, -2.0), (0.7, 0.0)):
                print(f"case: {m}x{n}x{k} {prec} tile {tile} pad {pad} alpha {alpha} beta {beta}", flush=True)
                dC = to_dev(C, pad, misalign)
                want = dC.clone()
                gpu.sgemm(dA, dB, want, alpha, beta, prec=prec, tile=tile)
                got = torch.full((m, n), float("nan"), device="cuda")
                gpu.sgemm_into(dA, dB, dC, got, alpha, beta, prec=prec, tile=tile)
                assert torch.equal(got, want)
                assert torch.equal(dC, to_dev(C))


def test_into_aliases(gpu):
    """C may be an operand or D itself; any other overlap with D is refused."""
    import torch

    A, B, C = (to_dev(x) for x in inputs.sgemm_operands(96, 96, 96, seed=5))
    want = gpu.sgemm(A, B, A.clone(), 0.7, 0.3)
    assert torch.equal(gpu.sgemm_into(A, B, A, torch.empty_like(A), 0.7, 0.3), want)
    want = gpu.sgemm(A, B, C.clone(), 0.7, 0.3)
    assert torch.equal(gpu.sgemm_into(A, B, C, C, 0.7, 0.3), want)
    big = torch.zeros(97, 96, device="cuda")
    with pytest.raises(HpvmError):
        gpu.sgemm_into(A, B, big[1:], big[:96], 0.7, 0.3)
    with pytest.raises(HpvmError):
        gpu.sgemm_into(A, B, C, A, 0.7, 0.3)
