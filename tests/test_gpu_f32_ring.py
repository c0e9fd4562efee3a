"""The fp32 ring kernel at the edges of its schedule and layouts, small
integers (every order of the sums exact) against the oracle, bit for bit."""
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


# (M levels, N levels) of one workgroup tile and its K stages: (kLoop, split, sub, blk)
CASES = [
    # K of one, two, three, four and many stages, at every stage depth
    *[((2, 2, 1, 32), (2, 2, 1, 32), (k, 1, 1, d), 0) for k in (1, 2, 3, 4, 9) for d in (8, 16, 32, 64)],
    *[((2, 2, 1, 16), (2, 2, 1, 16), (k, 1, 1, d), 0) for k in (1, 2, 3, 7) for d in (16, 32, 64)],
    # more wavefronts than a stage of one operand has loads
    ((1, 8, 1, 16), (2, 1, 1, 16), (5, 1, 1, 16), 0),
    ((2, 1, 1, 16), (1, 8, 1, 16), (5, 1, 1, 16), 0),
    ((1, 4, 1, 16), (1, 2, 1, 16), (6, 1, 2, 16), 0),
    # panels of 64, 128, 256, 512 and 1024 columns, one wavefront and more
    ((2, 1, 1, 16), (1, 1, 4, 16), (4, 1, 2, 16), 0),
    ((2, 2, 1, 16), (1, 2, 8, 16), (4, 1, 2, 16), 0),
    ((2, 1, 1, 16), (1, 1, 16, 16), (4, 1, 2, 16), 0),
    ((2, 1, 1, 16), (1, 1, 32, 16), (3, 1, 1, 16), 0),
    ((2, 2, 1, 16), (1, 2, 32, 16), (3, 1, 1, 16), 0),
    ((2, 1, 1, 16), (1, 1, 64, 16), (3, 1, 1, 16), 0),
    ((1, 1, 32, 16), (2, 1, 1, 16), (3, 1, 1, 16), 0),
    ((1, 1, 64, 16), (2, 2, 1, 16), (3, 1, 1, 16), 0),
    ((1, 1, 16, 32), (2, 1, 1, 32), (3, 1, 1, 8), 0),
    # 9 to 32 loads of an operand a stage, and a stage that fills LDS alone
    ((1, 1, 8, 16), (2, 1, 1, 32), (5, 1, 4, 16), 0),
    ((1, 1, 2, 32), (1, 1, 4, 32), (5, 1, 2, 32), 0),
    ((2, 2, 4, 32), (1, 2, 4, 32), (3, 1, 2, 32), 0),
    # split K (atomics), with as many stages a slice as the ring, fewer and more
    *[((2, 2, 1, 32), (2, 2, 1, 32), (k, 4, 1, 32), 0) for k in (1, 2, 3, 5)],
]


@pytest.mark.parametrize("kmajor", [False, True])
@pytest.mark.parametrize("case", CASES, ids=[str(c[:3]).replace(" ", "") for c in CASES])
def test_ring_bit_exact(gt, orc, case, kmajor):
    m, n, k, mf = case
    M, N, K = (int(np.prod(x)) for x in (m, n, k))
    info = gt.lower((m, k, n, mf), M, N, K, gt.F32 | (gt.A_KMAJOR if kmajor else 0))
    assert info["fast"] == 1 and info["ring"] >= 1, info
    A, B = make_inputs(M, N, K, "f32", 23, "smallint")
    ref = orc.gemm(raw_bytes(A), raw_bytes(B), M, N, K, "f32")
    Ad = (A.t().contiguous() if kmajor else A).cuda()
    C = torch.full((M, N), float("nan"), device="cuda")
    gt.gemm_run((m, k, n, mf), Ad, B.cuda(), C, a_kmajor=kmajor)
    assert np.array_equal(C.cpu().numpy().astype(np.float64), ref), info


def test_offsets_past_32_bits(gt):
    """A of 5 GiB: a tile's rows lie further than 2^32 bytes apart, so the
    loads step 64-bit addresses. Entries in {-1, 0, 1}: every sum is exact,
    and the product equals the check product bit for bit."""
    M, N, K = 256, 32, 5 << 20
    g = torch.Generator(device="cuda").manual_seed(3)
    A = torch.randint(-1, 2, (M, K), generator=g, device="cuda", dtype=torch.int8).float()
    B = torch.randint(-1, 2, (K, N), generator=g, device="cuda", dtype=torch.int8).float()
    cfg = ((1, 4, 2, 32), (K // 32 // 256, 256, 1, 32), (1, 1, 1, 32), 0)
    assert gt.lower(cfg, M, N, K, "f32")["fast"] == 1
    C, R = torch.full((M, N), float("nan"), device="cuda"), torch.empty(M, N, device="cuda")
    gt.gemm_run(cfg, A, B, C)
    gt.gt_reference_gemm(A, B, R)
    assert torch.equal(C, R)
