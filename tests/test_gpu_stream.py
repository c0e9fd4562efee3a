"""The generic path's two kernels: the one whose wavefronts read their own
operands, at block sizes below and above the MFMA's, K ends inside a step, K
splits, several wavefronts and both layouts, and the one with shared stages,
which takes what the other does not. Small integers (exact in any order)
against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

from workloads import make_inputs, raw_bytes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gt():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1909_10616_amd import gemmtune
    gemmtune.lib()
    return gemmtune


# M levels, N levels, K levels, MFMA, and which of (row-major, K-major) the rule
# sends there ("r", "k"); grids of 3 and 5 tiles so that edges are not aligned
BF16 = [
    # blocks of 8 and 4 (an MFMA tile half or a quarter full), single and repeated
    (((3, 1, 1, 8), (5, 1, 1, 8), (45, 1, 1, 16), 16), "rk"),
    (((3, 1, 2, 8), (5, 1, 4, 8), (11, 1, 1, 8), 32), "rk"),
    (((3, 1, 4, 4), (5, 1, 2, 4), (9, 1, 2, 8), 16), "rk"),
    (((3, 2, 1, 16), (5, 1, 1, 32), (3, 1, 1, 16), 16), "rk"),
    # K of less than one step, one step, a step and a bit, and the prefetch depths
    *[(((3, 1, 1, 16), (5, 1, 1, 16), (k, 1, 1, 8), 16), "rk") for k in (3, 4, 5, 9, 15, 16, 17, 33, 35)],
    *[(((3, 1, 1, 32), (5, 1, 1, 32), (k, 1, 1, 8), 32), "rk") for k in (1, 2, 3, 7, 8, 9)],
    # several wavefronts and MFMA tiles, blocks above the MFMA's size
    (((3, 2, 2, 32), (5, 2, 2, 32), (9, 1, 2, 16), 32), "k"),
    (((3, 2, 1, 64), (5, 4, 1, 32), (5, 1, 1, 64), 16), "k"),
    (((3, 1, 1, 128), (5, 1, 1, 32), (5, 1, 2, 16), 16), "k"),
    (((3, 1, 1, 32), (5, 1, 8, 16), (5, 1, 2, 16), 16), "k"),
    # K splits in stages of one step and of several
    (((3, 2, 1, 32), (5, 2, 1, 32), (3, 4, 1, 32), 32), "k"),
    (((3, 1, 1, 8), (5, 1, 1, 16), (5, 2, 2, 32), 16), "rk"),
]
F32 = [
    (((3, 1, 1, 8), (5, 1, 1, 8), (k, 1, 1, 4), 0), "rk") for k in (1, 3, 4, 5, 15, 16, 17, 33)
] + [
    (((3, 1, 2, 2), (5, 1, 1, 1), (9, 1, 1, 4), 0), "rk"),
    (((3, 2, 2, 4), (5, 4, 1, 8), (7, 1, 2, 4), 0), "rk"),
    (((3, 1, 1, 32), (5, 1, 1, 32), (7, 1, 1, 4), 0), "rk"),
    (((3, 1, 1, 8), (5, 1, 4, 16), (3, 1, 1, 1), 0), "k"),       # K = 3
    (((3, 2, 1, 8), (5, 1, 1, 16), (3, 4, 1, 16), 0), "rk"),      # split K
]
# shared stages: more than 8 wavefronts, rows or blocks no 16-byte load fits,
# stages shorter than a step, one stage and several, K splits
GENERIC = [
    ("bf16", ((3, 4, 1, 16), (5, 4, 1, 16), (7, 1, 2, 16), 16), "rk"),
    ("bf16", ((3, 1, 1, 16), (5, 1, 1, 2), (7, 1, 1, 16), 16), "r"),
    ("bf16", ((3, 1, 1, 2), (5, 1, 1, 16), (7, 1, 1, 8), 16), "k"),
    ("bf16", ((3, 1, 1, 8), (5, 2, 1, 16), (3, 1, 1, 1), 16), "k"),
    ("bf16", ((3, 1, 4, 32), (3, 1, 4, 32), (1, 1, 1, 8), 16), "rk"),
    ("bf16", ((3, 1, 4, 32), (3, 1, 4, 32), (3, 2, 1, 8), 16), "rk"),
    ("f32", ((3, 4, 1, 16), (5, 4, 1, 8), (7, 1, 2, 4), 0), "rk"),
    ("f32", ((3, 1, 1, 8), (5, 1, 1, 8), (3, 1, 1, 1), 0), "r"),
    ("f32", ((3, 2, 1, 8), (5, 2, 1, 8), (3, 4, 1, 2), 0), "rk"),
    ("f32", ((2, 1, 16, 8), (2, 1, 2, 8), (3, 1, 2, 4), 0), "r"),
]
CASES = [("stream", "bf16", c, lay == "k") for c, w in BF16 for lay in w] + \
        [("stream", "f32", c, lay == "k") for c, w in F32 for lay in w] + \
        [("generic", d, c, lay == "k") for d, c, w in GENERIC for lay in w]


@pytest.mark.parametrize("kernel,dtype,cfg,kmajor", CASES,
                         ids=[f"{g}-{d}-{'k' if k else 'r'}-{i}" for i, (g, d, _, k) in enumerate(CASES)])
def test_generic_path_bit_exact(gt, orc, kernel, dtype, cfg, kmajor):
    m, n, k, mf = cfg
    cfg = (m, k, n, mf)
    M, N, K = (int(np.prod(x)) for x in (m, n, k))
    info = gt.lower(cfg, M, N, K, gt.dtype_code(dtype) | (gt.A_KMAJOR if kmajor else 0))
    assert info["kernel"] == kernel, (cfg, info)
    A, B = make_inputs(M, N, K, dtype, 29, "smallint")
    ref = orc.gemm(raw_bytes(A), raw_bytes(B), M, N, K, dtype)
    Ad = (A.t().contiguous() if kmajor else A).cuda()
    C = torch.full((M, N), float("nan"), device="cuda")
    gt.gemm_run(cfg, Ad, B.cuda(), C, a_kmajor=kmajor)
    assert np.array_equal(C.cpu().numpy().astype(np.float64), ref), info


def test_infinities_stay_in_their_rows_and_columns(gt):
    """Blocks that leave an MFMA tile part empty and a K end inside a step
    read clamped rows, columns and k: an infinity in A's last row or B's last
    column reaches that row or column of C only."""
    M, N, K = 24, 40, 24
    cfg = ((3, 1, 1, 8), (3, 1, 1, 8), (5, 1, 1, 8), 16)
    A, B = (torch.rand(s, device="cuda").add_(0.5).to(torch.bfloat16) for s in ((M, K), (K, N)))
    A[M - 1, K - 1] = float("inf")
    B[K - 1, N - 1] = float("inf")
    C = torch.empty(M, N, device="cuda")
    gt.gemm_run(cfg, A, B, C)
    assert torch.isinf(C[M - 1]).all() and torch.isinf(C[:, N - 1]).all()
    assert torch.isfinite(C[:M - 1, :N - 1]).all()
