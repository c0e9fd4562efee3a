"""The ring kernel (fp32, bf16) at the edges of its schedule and layouts, small
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


# bf16 stages the evenly shared kernel does not take: uneven shares, more loads
# than it holds, 4 to 7 of them, one-stage and two-stage rings, the MFMA sizes
BF16 = [
    *[((2, 8, 1, 16), (2, 1, 1, 32), (k, 1, 1, 32), 16) for k in (1, 2, 5, 9, 17)],
    *[((2, 8, 1, 16), (2, 1, 1, 32), (k, 1, 2, 32), 16) for k in (1, 3, 9)],
    ((2, 8, 1, 16), (2, 1, 1, 16), (5, 1, 4, 32), 16),
    ((2, 1, 1, 16), (2, 8, 1, 16), (5, 1, 1, 32), 16),
    *[((2, 1, 1, 32), (2, 1, 1, 32), (k, 1, 8, 16), 32) for k in (1, 2, 3, 9)],
    ((2, 1, 2, 16), (2, 1, 2, 16), (5, 1, 4, 32), 16),
    ((2, 1, 1, 32), (2, 1, 8, 16), (5, 1, 2, 32), 16),
    ((2, 1, 1, 32), (2, 1, 4, 32), (5, 1, 2, 16), 32),
    ((2, 2, 2, 32), (2, 2, 1, 32), (9, 1, 2, 32), 32),       # 6 loads a wavefront
    ((2, 1, 4, 32), (2, 2, 1, 32), (4, 1, 2, 32), 16),       # 8 of A and 4 of B
    ((2, 2, 1, 32), (2, 1, 8, 32), (5, 1, 2, 16), 32),   # 2 of A and 8 of B
    ((1, 4, 2, 32), (1, 2, 4, 32), (3, 1, 4, 32), 16),       # one stage fills LDS
    ((2, 1, 1, 32), (1, 1, 16, 32), (3, 1, 1, 16), 32),      # a panel of 512 columns
    ((2, 1, 1, 16), (1, 1, 64, 16), (3, 1, 1, 32), 16),      # … of 1024
    *[((2, 8, 1, 16), (2, 1, 1, 32), (k, 4, 1, 32), 16) for k in (1, 2, 5)],
]
# wavefront tiles whose fragments are streamed, one wavefront and more, K of one
# to many stages, every stage depth
WIDE = [((1, 1, tm, 16), (2, 1, tn, 16), (k, 1, 1, d))
        for tm, tn in ((1, 16), (16, 1), (1, 32), (32, 1), (2, 16), (16, 2), (4, 8), (8, 4), (1, 64), (64, 1),
                       (2, 32), (32, 2), (4, 16), (16, 4)) for k, d in ((1, 64), (2, 32), (3, 64), (7, 32))] + \
       [((1, 2, 4, 16), (2, 2, 8, 16), (5, 1, 1, 64)), ((2, 2, 16, 16), (1, 4, 1, 16), (5, 1, 1, 32)),
        ((1, 1, 2, 16), (1, 2, 32, 16), (9, 1, 1, 32)), ((2, 1, 32, 16), (1, 1, 1, 16), (3, 2, 1, 32))]
CASES += [(m, n, (*k[:3], max(k[3] >> s, 16)), 0) for m, n, k in WIDE for s in (0, 1)
          if (np.prod(m[1:]) + np.prod(n[1:])) * (k[3] >> s) * 4 <= 163840]
BF16 += [(m, n, k, 16) for m, n, k in WIDE]
ALL = [("f32", c, km) for c in CASES for km in (False, True)] + [("bf16", c, False) for c in BF16]


@pytest.mark.parametrize("dtype,case,kmajor", ALL,
                         ids=[f"{d}-{'k' if k else 'r'}-{i}" for i, (d, _, k) in enumerate(ALL)])
def test_ring_bit_exact(gt, orc, dtype, case, kmajor):
    m, n, k, mf = case
    M, N, K = (int(np.prod(x)) for x in (m, n, k))
    info = gt.lower((m, k, n, mf), M, N, K, gt.dtype_code(dtype) | (gt.A_KMAJOR if kmajor else 0))
    assert info["kernel"] == "ring" and info["ring"] >= 1, info
    A, B = make_inputs(M, N, K, dtype, 23, "smallint")
    ref = orc.gemm(raw_bytes(A), raw_bytes(B), M, N, K, dtype)
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
    assert gt.lower(cfg, M, N, K, "f32")["kernel"] == "ring"
    C, R = torch.full((M, N), float("nan"), device="cuda"), torch.empty(M, N, device="cuda")
    gt.gemm_run(cfg, A, B, C)
    gt.gt_reference_gemm(A, B, R)
    assert torch.equal(C, R)


def _small_integers(shape, seed):
    """Entries in {-1, 0, 1}, drawn in pieces."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    out = torch.empty(shape, device="cuda")
    flat = out.view(-1)
    for i in range(0, flat.numel(), 1 << 28):
        n = min(1 << 28, flat.numel() - i)
        flat[i:i + n] = torch.randint(-1, 2, (n,), generator=g, device="cuda", dtype=torch.int8)
    return out


def test_rows_of_one_load_past_32_bits(gt):
    """An instruction that covers 32 rows of an A with 2^28-byte rows (8 GiB):
    its lanes lie further than 2^32 bytes apart. The sums of the slices, in
    {-1, 0, 1} products, are exact in any order."""
    M, N, K = 32, 32, 1 << 26
    A, B = _small_integers((M, K), 5), _small_integers((K, N), 6)
    cfg = ((1, 1, 1, 32), (K // 8 // 256, 256, 1, 8), (1, 1, 1, 32), 0)
    info = gt.lower(cfg, M, N, K, "f32")
    assert info["kernel"] == "ring" and info["ring"] >= 2
    C = torch.full((M, N), float("nan"), device="cuda")
    gt.gemm_run(cfg, A, B, C)
    R = torch.zeros(M, N, device="cuda", dtype=torch.float64)
    for k in range(0, K, 1 << 22):
        R += torch.mm(A[:, k:k + (1 << 22)].contiguous(), B[k:k + (1 << 22)]).double()
    assert torch.equal(C.double(), R)


def test_rows_of_one_panel_load_past_32_bits(gt):
    """The same of a B with 2^29-byte rows (16 GiB), 16 of them an instruction."""
    M, N, K = 16, 1 << 27, 32
    A, B = _small_integers((M, K), 7), _small_integers((K, N), 8)
    cfg = ((1, 1, 1, 16), (2, 1, 1, 16), (N // 16, 1, 1, 16), 0)
    info = gt.lower(cfg, M, N, K, "f32")
    assert info["kernel"] == "ring" and info["ring"] == 2
    C, R = torch.full((M, N), float("nan"), device="cuda"), torch.empty(M, N, device="cuda")
    gt.gemm_run(cfg, A, B, C)
    gt.gt_reference_gemm(A, B, R)
    assert torch.equal(C, R)
