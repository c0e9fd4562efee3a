"""The work this framework is measured on.

Each case is one call a user's program makes through the Python binding: a
tuned product (`gemm_run`, A row-major or, for the perceptron layer Y = WᵀX,
K-major), the plain check product (`gt_reference_gemm`), or a whole G-BFS
search (`tune_gbfs`). Configurations are written as the factors of M, K and N
from the outermost level inwards, as the search reports them.
"""
from __future__ import annotations

import math

import torch

from paper_1909_10616_amd import gemmtune as gt

# (M, N, K) of 4096×11008×4096: no drawn product is larger
LARGEST_RUN = 4096 * 11008 * 4096
# a drawn check product is at most 4096³, a drawn ragged product 1360·1200·720
LARGEST_REFERENCE = 4096 ** 3
LARGEST_RAGGED = 1360 * 1200 * 720


def _run(name, dtype, M, N, K, m, k, n, mfma=0, kmajor=False, dist="normal"):
    return {"name": name, "kind": "run", "dtype": dtype, "M": M, "N": N, "K": K, "m": m, "k": k,
            "n": n, "mfma": mfma, "kmajor": kmajor, "dist": dist}


def listed():
    return [
        # the smallest product of the workload list: one launch, latency
        _run("run256_f32", "f32", 256, 256, 256, "16,1,16", "4,1,64", "8,2,16", dist="uniform"),
        # ordinary fp32 products with the configurations the searches end on
        _run("run1024_f32", "f32", 1024, 1024, 1024, "16,2,1,32", "16,1,16,4", "16,2,1,32",
             dist="uniform"),
        _run("run2048_f32", "f32", 2048, 2048, 2048, "32,1,1,64", "64,1,8,4", "16,4,1,32"),
        # the perceptron layer Y = WᵀX of the paper's protocol, W given K×M
        _run("perceptron1024_f32", "f32", 1024, 1024, 1024, "16,2,1,32", "16,64", "16,2,1,32",
             kmajor=True, dist="uniform"),
        # the same layer in bf16 at the hand-made start configuration
        _run("perceptron2048_bf16", "bf16", 2048, 2048, 2048, "16,2,2,32", "64,1,2,16",
             "16,2,2,32", 32, kmajor=True),
        # the headline product and an MLP's up-projection (N's odd factor 43)
        _run("run4096_bf16", "bf16", 4096, 4096, 4096, "16,2,2,64", "128,1,1,32", "16,4,2,32", 16,
             dist="normal_sqrtk"),
        _run("mlp4096x11008x4096_bf16", "bf16", 4096, 11008, 4096, "16,2,1,128", "128,1,1,32",
             "43,4,2,32", 16, dist="normal002"),
        # a small batch against a square weight, K split four ways
        _run("skinny64x4096x4096_bf16", "bf16", 64, 4096, 4096, "1,2,1,32", "8,4,2,64",
             "64,4,1,16", 16, dist="normal002"),
        # one GPU's eighth of the headline product
        _run("slab512x4096x4096_bf16", "bf16", 512, 4096, 4096, "4,2,2,32", "64,1,4,16",
             "64,2,1,32", 32, dist="normal_sqrtk"),
        # a ragged product: odd factors leave blocks of 16 in every dimension
        _run("ragged1360x1200x720_bf16", "bf16", 1360, 1200, 720, "85,1,1,16", "45,1,1,16",
             "75,1,1,16", 16),
        # the product every search checks its candidates against
        {"name": "reference4096_bf16", "kind": "reference", "dtype": "bf16", "M": 4096, "N": 4096,
         "K": 4096, "kmajor": False, "dist": "normal_sqrtk"},
        # a whole search: the 1024³ fp32 workload with its budget, every
        # candidate timed and checked
        {"name": "search1024_f32", "kind": "search", "dtype": "f32", "M": 1024, "N": 1024,
         "K": 1024, "budget": 200, "dist": "uniform"},
    ]


def _extent(rng, lo, hi, unit):
    """A multiple of `unit` in [lo, hi], spread over the logarithm; half of
    them powers of two times unit, the others with an odd factor."""
    v = 2.0 ** rng.uniform(math.log2(lo / unit), math.log2(hi / unit))
    if rng.random() < 0.5:
        return unit * 2 ** round(math.log2(v))
    return unit * max(1, min(hi // unit, round(v)))


def _split(extent, tile, waves, blk):
    return f"{extent // tile},{waves},{tile // (waves * blk)},{blk}"


def _tiled(rng, dtype, M, N, K, kmajor):
    """A configuration of the kind the searches end on: tiles that give about
    one workgroup or more per compute unit (the most tiles where none do),
    16 to 128 accumulators per lane, K split only where tiles are few."""
    size = 2 if dtype == "bf16" else 4
    choices = []
    for BM in (32, 64, 128, 256):
        for BN in (32, 64, 128, 256):
            if M % BM or N % BN:
                continue
            for wm, wn in ((1, 1), (1, 2), (2, 1), (2, 2), (2, 4), (4, 2)):
                acc = BM * BN // (64 * wm * wn)
                if BM // wm < 16 or BN // wn < 16 or not 4 <= acc <= 128:
                    continue
                choices.append((BM, BN, wm, wn))
    tiles = lambda c: (M // c[0]) * (N // c[1])  # noqa: E731
    full = [c for c in choices if 192 <= tiles(c) <= 1024]
    if not full:
        most = max(tiles(c) for c in choices)
        full = [c for c in choices if tiles(c) == most] if most < 192 else \
            [c for c in choices if tiles(c) == min(tiles(x) for x in choices if tiles(x) >= 192)]
    BM, BN, wm, wn = c = rng.choice(full)
    mfma = rng.choice((16, 32)) if dtype == "bf16" else 0
    if BM // wm < 32 or BN // wn < 32:
        mfma = 16 if dtype == "bf16" else 0
    low = 32 if mfma == 32 else 16
    blk_m = rng.choice([b for b in (16, 32, 64) if low <= b <= BM // wm])
    blk_n = rng.choice([b for b in (16, 32, 64) if low <= b <= BN // wn])
    BK = rng.choice([b for b in ((32, 64, 128) if dtype == "bf16" else (32, 64))
                     if K % b == 0 and (BM + BN) * b * size <= 81920])
    split = rng.choice((2, 4)) if tiles(c) <= 64 and K % (4 * BK) == 0 else 1
    if kmajor and dtype == "f32":   # the paper's levels: K in two
        k = f"{K // BK},{BK}"
    else:
        sub = rng.choice((1, 2)) if BK >= 64 else 1
        k = f"{K // (BK * split)},{split},{sub},{BK // sub}"
    return _split(M, BM, wm, blk_m), k, _split(N, BN, wn, blk_n), mfma


def draw(rng):
    """Another case of the listed ranges (no name): mostly products, some of
    them K-major or ragged, some check products."""
    kind = rng.choice(["run"] * 6 + ["kmajor"] * 3 + ["ragged"] * 2 + ["reference"])
    dtype = rng.choice(["f32", "bf16"])
    dist = rng.choice(["uniform", "normal", "normal_sqrtk", "normal002"])
    if kind == "reference":
        while True:
            M, N, K = (_extent(rng, 64, 4096, 8) + rng.choice((0, 0, 1, 3)) for _ in range(3))
            if M * N * K <= LARGEST_REFERENCE:
                break
        return {"kind": "reference", "dtype": dtype, "M": M, "N": N, "K": K,
                "kmajor": rng.random() < 0.3, "dist": dist}
    if kind == "ragged":
        while True:
            M, N, K = (((2 * rng.randrange(1, 64) + 1) << rng.choice((3, 4, 4, 5)))
                       for _ in range(3))
            if 100 ** 3 <= M * N * K <= LARGEST_RAGGED:
                break
        low = lambda v: v & -v  # noqa: E731
        m, k, n = (f"{v // low(v)},1,1,{low(v)}" for v in (M, K, N))
        return {"kind": "run", "dtype": dtype, "M": M, "N": N, "K": K, "m": m, "k": k, "n": n,
                "mfma": 16 if dtype == "bf16" else 0, "kmajor": rng.random() < 0.3, "dist": dist}
    top = 4096 if kind == "kmajor" or dtype == "f32" else 11008
    while True:
        M, N, K = _extent(rng, 64, 4096, 64), _extent(rng, 256, top, 64), _extent(rng, 256, 4096, 64)
        if 256 ** 3 <= M * N * K <= (LARGEST_RUN if kind == "run" and dtype == "bf16" else 2560 ** 3):
            break
    m, k, n, mfma = _tiled(rng, dtype, M, N, K, kind == "kmajor")
    return {"kind": "run", "dtype": dtype, "M": M, "N": N, "K": K, "m": m, "k": k, "n": n,
            "mfma": mfma, "kmajor": kind == "kmajor", "dist": dist}


def _values(shape, dist, K, generator):
    """The distributions of the framework's own workloads."""
    if dist == "uniform":
        return torch.rand(shape, generator=generator, device="cuda") * 2.0 - 1.0
    v = torch.randn(shape, generator=generator, device="cuda")
    return v * {"normal": 1.0, "normal_sqrtk": 1.0 / math.sqrt(K), "normal002": 0.02}[dist]


def _inputs(case, seed):
    M, N, K = case["M"], case["N"], case["K"]
    g = torch.Generator(device="cuda").manual_seed(seed)
    t = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    A = _values((K, M) if case.get("kmajor") else (M, K), case["dist"], K, g).to(t)
    B = _values((K, N), case["dist"], K, g).to(t)
    return A, B


def prepare(case, seed):
    A, B = _inputs(case, seed)
    state = {"kind": case["kind"], "A": A, "B": B, "kmajor": bool(case.get("kmajor")),
             "C": torch.empty(case["M"], case["N"], device="cuda")}
    if case["kind"] == "run":
        levels = [tuple(int(f) for f in case[x].split(",")) for x in ("m", "k", "n")]
        state["cfg"] = (*levels, case["mfma"])
    elif case["kind"] == "search":
        d = (4, 4, 4)
        coord = case["dtype"] == "bf16"
        state["space"] = gt.Space(case["M"], case["N"], case["K"], d, case["dtype"], coord)
        state["s0"] = gt.hand_start(case["M"], case["N"], case["K"], d, coord)
        state["budget"] = case["budget"]
        state["ref"] = torch.empty_like(state["C"])
    return state


def run(state):
    A, B, C = state["A"], state["B"], state["C"]
    if state["kind"] == "run":
        return gt.gemm_run(state["cfg"], A, B, C, a_kmajor=state["kmajor"])
    if state["kind"] == "reference":
        return gt.gt_reference_gemm(A, B, C, a_kmajor=state["kmajor"])
    found = gt.tune_gbfs(state["space"], budget=state["budget"], s0=state["s0"], A=A, B=B, C=C,
                         c_ref=state["ref"])
    # the last candidate's product, the check product, and how the search went
    return {"C": C, "ref": state["ref"], "timed": found["timed"], "failed": found["failed"]}


def work(case):
    M, N, K = case["M"], case["N"], case["K"]
    size = 2 if case["dtype"] == "bf16" else 4
    one = {"bytes": (M * K + K * N) * size + 4 * M * N, "flops": 2 * M * N * K}
    if case["kind"] != "search":
        return one
    # every candidate runs once to warm up and ten times timed, and its output
    # is read beside the check product's; the check product itself runs once
    launches = 11 * case["budget"] + 1
    return {"bytes": launches * one["bytes"] + case["budget"] * 8 * M * N,
            "flops": launches * one["flops"]}


def tolerance(case):
    """fp32 sums in another order (both input types accumulate in fp32): two
    orders of the same product differ by up to 6e-7 at K = 1024 and, growing
    with the root of K, 1.2e-6 at K = 4096; about four times that."""
    return {"rel": 4e-6}


def exact(case, seed):
    A, B = _inputs(case, seed)
    A = A.t() if case.get("kmajor") else A
    C = torch.mm(A.double().contiguous(), B.double())
    if case["kind"] == "search":
        return {"C": C, "ref": C, "timed": None, "failed": None}
    return C
