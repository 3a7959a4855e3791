"""CPU model of how the any-size DMA-fed loop (mfma_f32_any.hpp) fills its LDS
stages: every 16-byte transfer of every lane stays inside its matrix, and
what the matrix cores then read is the matrix, zero past the end of k."""
import numpy as np
import pytest

LANES = np.arange(64)


def unit(kc, R, TK, q):
    """Row and first column, in the sub-slab, of each lane's unit of instruction q."""
    if kc and TK == 32:
        x = (LANES >> 3) ^ (q & 1)
        return q * 8 + x, ((LANES & 7) ^ x) * 4
    if kc:
        y, p = LANES >> 3, LANES & 7
        g = (y & 3) ^ ((y >> 2) & 1)
        return q * 16 + 2 * y + ((p >> 2) & 1), ((p ^ g) & 3) * 4
    return q * (256 // R) + LANES // (R // 4), (LANES % (R // 4)) * 4


def lds_position(kc, TK, row, k):
    """LDS float that a fragment read takes for (row, k) of a KC sub-slab (the SwizzledRows layouts)."""
    block, r, c = row // 32 * 32, row % 32, k // 4
    if TK == 32:
        at = (r ^ ((r >> 3) & 1)) * 128 + ((c ^ (r & 7)) << 4)
    else:
        g = ((r >> 1) & 3) ^ ((r >> 3) & 1)
        at = (r >> 1) * 128 + (((((r & 1) << 2) | c) ^ g) << 4)
    return block * TK + at // 4 + k % 4


@pytest.mark.parametrize("kc", [True, False])
@pytest.mark.parametrize("R,TK,KW", [(32, 32, 1), (64, 32, 1), (128, 32, 1), (32, 32, 4), (64, 32, 2), (128, 16, 1)])
def test_stages_hold_the_matrix_and_no_access_leaves_it(kc, R, TK, KW):
    rng = np.random.default_rng(R + TK + KW)
    sizes = [1, 2, 3, 4, 5, 6, 7, 31, 33, R - 1, R, R + 1, R + 2, 2 * R + 3]
    for extent in sorted(set(sizes)):
        if not kc and extent < 4:
            continue  # the loop does not take such a product
        for depth in (1, 2, 3, 4, 5, TK - 1, TK, TK + 1, KW * TK, KW * TK + 2, 3 * KW * TK - 1):
            for pad in (0, 1):
                rows, cols = (extent, depth) if kc else (depth, extent)
                ld = cols + pad
                flat = rng.uniform(1, 2, (rows - 1) * ld + cols).astype(np.float32)  # the whole allocation
                slab = KW * TK
                by_hand = not kc and extent < R and extent % 4 != 0
                dma = (depth - 1 if by_hand else depth) // slab
                slabs = -(-depth // slab)
                assert slabs - dma in (0, 1)
                for t in range(-(-extent // R)):
                    own = t * R
                    corner = extent - R if not kc and extent >= R and own + R > extent else own
                    left = extent - corner
                    for s in range(slabs):
                        for kw in range(KW):
                            k0 = s * slab + kw * TK
                            base = corner * ld + k0 if kc else k0 * ld + corner
                            lds = np.full(R * TK, np.nan, np.float32)
                            for q in range(R * TK * 4 // 1024):
                                r, c = unit(kc, R, TK, q)
                                if s < dma:
                                    if kc:
                                        r = np.where(r < left, r, left - 1)
                                    else:
                                        c = np.where(c < left, c, 0)
                                    at = base + r * ld + c
                                    assert at.min() >= 0 and at.max() + 4 <= flat.size
                                    v = flat[at[:, None] + np.arange(4)]
                                else:
                                    rr, cc = np.broadcast_arrays(r[:, None], c[:, None] + np.arange(4))
                                    inside = (rr < left) & (cc < depth - k0) if kc else \
                                        (rr < depth - k0) & (cc < left)
                                    at = np.where(inside, base + rr * ld + cc, 0)
                                    assert at.min() >= 0 and at.max() < flat.size
                                    v = np.where(inside, flat[at], 0)
                                lds[q * 256:(q + 1) * 256] = v.reshape(-1)
                            # What a fragment read finds at (index i of the side, k).
                            i, k = np.meshgrid(np.arange(min(R, left)), np.arange(TK), indexing="ij")
                            pos = np.vectorize(lambda a, b: lds_position(kc, TK, a, b))(i, k) if kc else k * R + i
                            got = lds[pos]
                            inside = k < depth - k0
                            at = np.where(inside, base + (i * ld + k if kc else k * ld + i), 0)
                            assert np.array_equal(got, np.where(inside, flat[at], 0)), (extent, depth, pad, t, s)


@pytest.mark.parametrize("m,n,k", [(1, 4, 1), (128, 128, 128), (16, 4096, 4096), (33, 35, 2051), (1000, 1003, 777),
                                   (512, 4096, 1024), (3001, 2999, 1001), (64, 64, 2047), (5, 3, 4096),
                                   (1536, 1536, 1536), (2048, 1024, 512), (1280, 1280, 1280), (1024, 1024, 1024),
                                   (1024, 1536, 2048), (640, 640, 4096), (2048, 1024, 8192)])
def test_fp32_choice_agrees_with_its_workspace(m, n, k):
    """With no tile: the workspace asked for is what the described slices fill, a
    shorter one gives a choice that fits it, and none gives hpvm_sgemm's."""
    import paper_1611_00860_amd as hp

    hp.autotune_clear()
    need = hp.workspace_bytes(m, n, k, "fp32")
    d = hp.describe(m, n, k, "fp32", workspace_bytes=need)
    assert need == (4 * m * n * d["splits"] if d["splits"] > 1 else 0)
    assert d == hp.describe(m, n, k, "fp32", workspace_bytes=1 << 40)
    plain = hp.describe(m, n, k, "fp32")
    assert plain["splits"] == 1 and plain == hp.describe(m, n, k, "fp32", workspace_bytes=0)
    assert (need > 0) == (d["splits"] > 1)
    if need:
        short = hp.describe(m, n, k, "fp32", workspace_bytes=need - 1)
        assert 4 * m * n * short["splits"] < need or short["splits"] == 1
