"""A CPU model of the generic path whose wavefronts read their own operands:
every global address inside its operand, every piece of LDS inside the
launch's, and the transposing reads finding the elements each MFMA lane
needs, over seeded samples of the launches the rule sends there. The rule and
the index formulas are restated here."""
import os
import random

import numpy as np
import pytest

from test_kernel_model import bswz, levels

LANE = np.arange(64)


@pytest.fixture(scope="module")
def gt():
    from paper_1909_10616_amd import gemmtune
    if not os.path.exists(gemmtune.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    gemmtune.lib()
    return gemmtune


def serves(L, info, M, N, K, bf16, akm):
    size, KL = (2, 8) if bf16 else (4, 4)
    KS = KL * (64 // L["I"])
    WM, WN = L["WM"], L["WN"]
    if info["fast"] or L["W"] > 8 or L["TM"] + L["TN"] > 10 or (L["kSplit"] > 1 and L["BK"] % KS):
        return False
    if K >= 1 << 31 or max(KS * M if akm else WM * K, KS * N) * size >= 1 << 32:
        return False
    if not akm and K % KL:
        return False
    if not bf16:
        return True
    if WN % 8 or N % 8 or L["blkN"] % 4:
        return False
    if akm and (WM % 8 or M % 8 or L["blkM"] % 4):
        return False
    return L["W"] * KS * (max(WM, WN) if akm else WN) * 2 <= info["lds_bytes"]


def in_tile(t, l, I, blk):
    tpb = max(blk // I, 1)
    return (t // tpb) * blk + np.minimum((t % tpb) * I + l, blk - 1)


def panel_bf16(I, TX, width, ld, blk):
    """(k row, byte offset from the step's origin, LDS byte, first and second
    read byte) of each lane and load of a [k][x] panel."""
    KS, cw = 8 * (64 // I), width // 8
    i16, g16 = LANE & 15, LANE >> 4
    kgrp = (g16 >> 1) if I == 32 else g16
    ncol = (16 * (g16 & 1) if I == 32 else 0) + 4 * (i16 & 3)
    bs = np.vectorize(lambda k: bswz(int(k), cw))
    out = []
    for t in range(TX):
        c = np.minimum(LANE + 64 * t, KS * cw - 1)
        k, x = c // cw, c % cw
        kr = kgrp * 8 + (i16 >> 2)
        col = np.minimum(in_tile(t, 0, I, blk) + ncol, width - 4)
        get = (kr * cw + ((col >> 3) ^ bs(kr))) * 16 + (col & 4) * 2
        out.append((k, (k * ld + x * 8) * 2, (k * cw + (x ^ bs(k))) * 16, get, get + cw * 64))
    return out


def check_panel_reads(I, TX, width, blk):
    """The panel in LDS as (k, x) of every 2-byte word, and what the lanes'
    transposing reads hand each MFMA lane."""
    KS = 8 * (64 // I)
    held = np.full((KS * width, 2), -1)
    loads = panel_bf16(I, TX, width, 1 << 20, blk)
    for k, off, put, _, _ in loads:
        for e in range(8):
            held[put // 2 + e] = np.stack([k, (off // 2 + e) % (1 << 20)], 1)
    assert held.min() >= 0
    tpb = max(blk // I, 1)
    for t, (_, _, _, get0, get1) in enumerate(loads):
        for h, get in enumerate((get0, get1)):
            assert get.min() >= 0 and get.max() + 8 <= KS * width * 2
            for lane in range(64):
                g16, l = lane >> 4, lane & 15
                inl = lane % I                     # row or column in the MFMA tile
                if (t % tpb) * I + inl >= blk:
                    continue                       # not stored
                for j in range(4):
                    src = 16 * g16 + 4 * j + (l >> 2)
                    k, x = held[get[src] // 2 + (l & 3)]
                    assert k == lane // I * 8 + 4 * h + j
                    assert x == (t // tpb) * blk + (t % tpb) * I + inl


@pytest.mark.parametrize("I", [16, 32])
def test_panel_reads(I):
    for blk in (4, 8, 16, 32, 64, 128):
        for rep in (1, 2, 4, 8):
            TX, width = rep * -(-blk // I), rep * blk
            if TX <= 9 and width % 8 == 0:
                check_panel_reads(I, TX, width, blk)


def check_stream(L, info, M, N, K, bf16, akm):
    """One launch: the last whole and partial steps of the first and last
    workgroup, slice and wavefront stay inside the operands and the LDS."""
    size = 2 if bf16 else 4
    I, KL = L["I"], 8 if bf16 else 4
    KS = KL * (64 // I)
    run = K if L["kSplit"] == 1 else L["BK"]
    skip = 0 if L["kSplit"] == 1 else (L["kSplit"] - 1) * L["BK"]
    runs = 1 if L["kSplit"] == 1 else L["kLoop"]
    per, left = divmod(run, KS)
    assert left == 0 or L["kSplit"] == 1
    for gm, gn, z in ((0, 0, 0), (L["gridM"] - 1, L["gridN"] - 1, L["kSplit"] - 1)):
        for w in {0, L["W"] - 1}:
            wm, wn = w % L["wavesM"], w // L["wavesM"]
            row0, col0 = gm * L["BM"] + wm * L["WM"], gn * L["BN"] + wn * L["WN"]
            # the last whole step, and the partial one
            last = z * L["BK"] + (runs - 1) * (run + skip)
            for k, kv in ([(last + (per - 1) * KS, KS)] if per else []) + ([(last + per * KS, left)] if left else []):
                for x0, ld, X, TX, width, blk, step_rows in (
                        (col0, N, N, L["TN"], L["WN"], L["blkN"], True),
                        (row0, M if akm else K, M, L["TM"], L["WM"], L["blkM"], akm)):
                    for t in range(TX):
                        if not step_rows:      # row-major A
                            rows, kk = in_tile(t, LANE % I, I, blk), LANE // I * KL
                            off = np.where(kk < kv, rows * K + kk, 0)
                            at, words = x0 * K + k + off, KL
                            assert off.max() * size < 1 << 32 and at.max() + words <= M * K
                        elif bf16:
                            kr, off, put, _, _ = panel_bf16(I, TX, width, ld, blk)[t]
                            off = np.where(kr < kv, off, 0)
                            at = k * ld + x0 + off // 2
                            assert off.max() < 1 << 32 and at.max() + 8 <= K * X
                            assert ((at * 2) % 16 == 0).all()
                            assert put.max() + 16 <= KS * width * 2
                        else:
                            kr = LANE // I * 4 + np.arange(4)[:, None]
                            off = np.where(kr < kv, kr * ld + in_tile(t, LANE % I, I, blk), 0)
                            at = k * ld + x0 + off
                            assert off.max() * 4 < 1 << 32 and at.max() < K * X
                        assert at.min() >= 0
    if bf16:
        assert L["W"] * KS * (max(L["WM"], L["WN"]) if akm else L["WN"]) * 2 <= info["lds_bytes"]


SPACES = [(1360, 1200, 720, "bf16", False), (1360, 1200, 720, "bf16", True), (1000, 1000, 1000, "bf16", False),
          (1000, 1000, 1000, "f32", False), (1000, 1000, 1000, "f32", True), (2048, 2048, 2048, "bf16", True),
          (96, 80, 48, "bf16", False), (130, 74, 36, "f32", False), (4096, 4096, 4096, "bf16", False)]


@pytest.mark.parametrize("space", SPACES)
def test_addresses_of_lowered_launches(gt, space):
    M, N, K, dt, akm = space
    bf16 = dt == "bf16"
    sp = gt.Space(M, N, K, (4, 4, 4), dt, bf16, a_kmajor=akm)
    rng = random.Random(M + K + akm)
    seen = tries = 0
    while seen < 120 and tries < 20000:
        tries += 1
        c = sp.unrank(rng.randrange(sp.size()))
        if not sp.legit(c):
            continue
        info = gt.lower(c, M, N, K, gt.dtype_code(dt) | (gt.A_KMAJOR if akm else 0))
        L = levels(c)
        assert (info["kernel"] == "stream") == serves(L, info, M, N, K, bf16, akm), (c, info)
        if info["kernel"] != "stream":
            continue
        seen += 1
        check_stream(L, info, M, N, K, bf16, akm)
    assert seen >= 20, (seen, tries)
