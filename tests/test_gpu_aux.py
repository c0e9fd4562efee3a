"""The helper kernels of the searches' output check at the sizes where their
work splits: the comparison (one partial result per block, 16-byte and scalar
loads, remainders, NaN and infinities) and the check product (three tile
sizes, ragged edges, few rows and many columns)."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gt():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1909_10616_amd import gemmtune
    gemmtune.lib()
    return gemmtune


def _expected(c, r):
    """max|c − r| / max|r| from fp32 differences; the largest |r| skips NaN."""
    with np.errstate(invalid="ignore"):
        d = np.abs(c - r)
    if np.isnan(d).any():
        return math.nan
    md, mr = float(d.max()), float(np.nanmax(np.abs(r)))
    return (0.0 if md == 0 else math.inf) if mr == 0 else md / mr


# one thread's share and its neighbours, one block's, and more than the most
# blocks (1024 of 4096 elements) with a remainder of 1, 2 and 3
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 255, 1023, 4095, 4096, 4097, 65537, (1 << 22) - 1,
                               (1 << 22) + 3])
@pytest.mark.parametrize("offsets", [(0, 0), (1, 0), (1, 1), (4, 8)])
def test_compare_at_block_and_alignment_edges(gt, n, offsets):
    rng = np.random.default_rng(n)
    r = rng.standard_normal(n + 16).astype(np.float32)
    c = r + (1e-4 * rng.standard_normal(n + 16)).astype(np.float32)
    co, ro = offsets
    for where in sorted({0, n // 2, n - 1}):
        for side, value in ((None, 0.0), ("c", np.nan), ("c", np.inf), ("c", 7.0), ("r", np.nan),
                            ("r", -9.0)):
            cc, rr = c.copy(), r.copy()
            if side == "c":
                cc[co + where] = value
            elif side == "r":
                rr[ro + where] = value
            cd, rd = torch.from_numpy(cc).cuda(), torch.from_numpy(rr).cuda()
            want = _expected(cc[co:co + n], rr[ro:ro + n])
            for f in (gt.gt_compare, gt.gt_compare_noalloc):
                got = f(cd[co:co + n], rd[ro:ro + n])
                assert got == want or (math.isnan(got) and math.isnan(want)), (where, side, value)


# tile edges of each tile size (32, 64 and 128 outputs a side; 384 tiles or
# more pick the larger), one row or column past them, and K around a chunk of
# 16 and below it
REFERENCE = [(1, 1, 1), (31, 33, 15), (32, 32, 16), (33, 31, 17), (65, 1, 33),
             (1024, 1536, 5), (1024, 1472, 6), (1217, 1281, 19), (1281, 1217, 16),
             (2048, 3072, 3), (2048, 2944, 2), (2433, 2561, 18), (2561, 2433, 1),
             # few rows and many columns: a whole group of rows and part of one, K
             # around a round of 8 loads, and the sizes past which the tiles take over
             (1, 65536, 1), (4, 65537, 7), (5, 65791, 8), (8, 65793, 9), (9, 65536, 64),
             (16, 65537, 17), (9, 65536, 65), (17, 65536, 8), (8, 65535, 16)]


@pytest.mark.parametrize("kmajor", [False, True])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", REFERENCE)
def test_reference_product_at_tile_edges(gt, orc, shape, dtype, kmajor):
    """Small integers, exact in any order: every element equals the oracle's."""
    from workloads import make_inputs, raw_bytes
    M, N, K = shape
    A, B = make_inputs(M, N, K, dtype, 17, "smallint")
    ref = orc.gemm(raw_bytes(A), raw_bytes(B), M, N, K, dtype)
    Ad = (A.t().contiguous() if kmajor else A).cuda()
    C = torch.full((M, N), float("nan"), device="cuda")
    gt.gt_reference_gemm(Ad, B.cuda(), C, a_kmajor=kmajor)
    assert np.array_equal(C.cpu().numpy().astype(np.float64), ref)


@pytest.mark.parametrize("offset", [0, 1, 2, 3])
@pytest.mark.parametrize("rows,cols", [(1, 1), (1, 3), (3, 5), (4, 64), (5, 255), (3, 1025)])
def test_split_k_clears_exactly_c(gt, rows, cols, offset):
    """C full of NaN at every 4-byte alignment, sizes with every remainder
    mod 4: a split-K product clears and fills C and nothing around it."""
    K = 16
    cfg = ((rows, 1, 1, 1), (2, 2, 1, 4), (cols, 1, 1, 1), 0)
    A, B = torch.ones(rows, K, device="cuda"), torch.ones(K, cols, device="cuda")
    buf = torch.full((rows * cols + 16,), float("nan"), device="cuda")
    C = buf[4 + offset:4 + offset + rows * cols].view(rows, cols)
    gt.gemm_run(cfg, A, B, C)
    assert (C == K).all()
    assert int(torch.isnan(buf).sum()) == 16
