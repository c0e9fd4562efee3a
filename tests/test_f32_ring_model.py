"""A CPU model of the fp32 ring kernel: where its direct loads put each
element of a stage in LDS, what its fragment reads find there, how far its
global addresses reach, and the order of loads, waits, barriers and reads of
its ring, over every kernel shape and over the launches the lowering chooses.
The model restates the kernel's index formulas; it shares no code with it."""
import itertools
import os
import random

import numpy as np
import pytest

LDS_MAX = 163840
LANE = np.arange(64)


@pytest.fixture(scope="module")
def gt():
    from paper_1909_10616_amd import gemmtune
    if not os.path.exists(gemmtune.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    gemmtune.lib()
    return gemmtune


def fswz(row, cpr):
    return (row >> (0 if cpr >= 8 else 1 if cpr == 4 else 2)) & (min(cpr, 8) - 1)


def share_rows(w, nw, BM, cpr, ld):
    """A wavefront's loads of a row-major A: per instruction its slot in the
    stage (units of 64 chunks) and the lanes' element offsets from the stage's
    origin."""
    cnt = ((BM * cpr >> 6) - w + nw - 1) // nw
    pos = ((LANE % cpr) ^ fswz(LANE // cpr, cpr)) * 4
    out = []
    for b in range(w, w + cnt * nw, nw):
        r = (b << 6) // cpr
        out.append((b, (r + LANE // cpr) * ld + (pos ^ (((r & 4) << 2) if cpr == 16 else 0))))
    return out


def flip_panel(I, CW):
    return I == 16 and CW in (8, 16)


def share_panels(w, nw, panels, I, W, BK, ld):
    """The same of a [k][n] operand in panels of W columns."""
    CW = W // 4
    npp = BK * CW // 64
    panel, b0, db = w % panels, w // panels, nw // panels
    cnt = (npp - b0 + db - 1) // db
    pos = LANE if CW >= 64 else LANE % CW
    row = LANE * 0 if CW >= 64 else LANE // CW
    pos = (pos ^ (row & 4) if flip_panel(I, CW) else pos) * 4
    out = []
    for b in range(b0, b0 + cnt * db, db):
        r, first = (b << 6) // CW, (b << 6) % CW
        x = ((r & 4) << 2) if flip_panel(I, CW) and CW == 16 else 0
        out.append((panel * npp + b, (r + row) * ld + panel * W + first * 4 + (pos ^ x)))
    return out


def loads(I, TM, TN, cpr, wavesM, wavesN, ak, lda, ldb):
    """Every load of a stage: (wavefront, slot, element offsets), A's and B's."""
    nw, BK = wavesM * wavesN, cpr * 4
    A, B = [], []
    for w in range(nw):
        A += [(w, *t) for t in (share_panels(w, nw, wavesM, I, TM * I, BK, lda) if ak
                                else share_rows(w, nw, wavesM * TM * I, cpr, lda))]
        B += [(w, *t) for t in share_panels(nw - 1 - w, nw, wavesN, I, TN * I, BK, ldb)]
    return A, B


def stage(I, TM, TN, cpr, wavesM, wavesN, ak):
    """A slot of the ring as arrays of the (outer, k) each 4-byte word holds,
    filled by every instruction of the stage; returns the arrays, A's and B's
    sizes in instructions."""
    BM, BN, BK = wavesM * TM * I, wavesN * TN * I, cpr * 4
    pa, pt = BM * cpr >> 6, (BM + BN) * cpr >> 6
    outer = np.full(pt * 256, -1)
    kk = np.full(pt * 256, -1)
    ld = 1 << 20   # a leading dimension that separates rows from columns
    A, B = loads(I, TM, TN, cpr, wavesM, wavesN, ak, ld, ld)
    for side, base, n, trans in ((A, 0, pa, not ak), (B, pa, pt - pa, False)):
        assert sorted(p for _, p, _ in side) == list(range(n))   # each slot once
        for _, p, off in side:
            words = (base + p) * 256 + LANE[:, None] * 4 + np.arange(4)
            e = off[:, None] + np.arange(4)
            r, c = e // ld, e % ld
            outer[words], kk[words] = (r, c) if trans else (c, r)
    assert outer.min() >= 0 and kk.min() >= 0 and kk.max() < BK
    assert outer[:pa * 256].max() < BM and outer[pa * 256:].max() < BN
    return outer, kk, pa, pt


SHAPES = [(I, TM, TN, cpr) for I in (16, 32) for cpr in (2, 4, 8, 16) if cpr >= 64 // I
          for TM, TN in itertools.product((1, 2, 4, 8, 16), repeat=2) if TM * TN * I * I // 64 <= 256]


@pytest.mark.parametrize("ak", [False, True])
def test_reads_find_what_the_loads_wrote(ak):
    for I, TM, TN, cpr in SHAPES:
        G = 64 // I
        grp, l0 = LANE // I, LANE % I
        for wavesM, wavesN in ((1, 1), (2, 1), (1, 2), (4, 2)):
            BK, WM, WN = cpr * 4, TM * I, TN * I
            if (wavesM * WM + wavesN * WN) * BK * 4 > LDS_MAX:
                continue
            outer, kk, pa, pt = stage(I, TM, TN, cpr, wavesM, wavesN, ak)
            assert len(set(zip(outer[:pa * 256], kk[:pa * 256]))) == pa * 256
            assert len(set(zip(outer[pa * 256:], kk[pa * 256:]))) == (pt - pa) * 256

            def panel_read(wi, t, W, cs, q):
                col = t * I + l0
                if flip_panel(I, W // 4):
                    col = col ^ ((grp & 1) << 4)
                return wi * BK * W + grp * 4 * W + col + (cs * G * 4 + q) * W

            for wm, wn, cs, q in itertools.product(range(wavesM), range(wavesN), range(cpr // G),
                                                   range(4)):
                k = (cs * G + grp) * 4 + q
                for t in range(TM):
                    if ak:
                        w = panel_read(wm, t, WM, cs, q)
                    else:
                        w = ((wm * WM + t * I + l0) * cpr * 4
                             + (((fswz(l0, cpr) ^ grp) ^ (cs * G)) * 4) + q)
                    assert (outer[w] == wm * WM + t * I + l0).all() and (kk[w] == k).all()
                for t in range(TN):
                    w = pa * 256 + panel_read(wn, t, WN, cs, q)
                    assert (outer[w] == wn * WN + t * I + l0).all() and (kk[w] == k).all()


def replay(ns, kLoop, NCS, na, nb, most):
    """One wavefront's loads, waits, barriers and reads, in program order; a
    load that moves nothing is ("load", None). na, nb: its loads of A and B;
    most: the most of either that any wavefront has."""
    ev, cnt = [], na + nb
    if ns == 1:
        for l in range(kLoop):
            ev += [("load", l)] * cnt + [("wait", 0), ("bar",), ("read", l), ("bar",)]
        return ev
    NH = 0 if most > 8 else 8 if most > 4 else 4 if most > 2 else 2

    def window(s):
        if NH == 0 and s < kLoop:
            ev.extend([("load", s)] * cnt)
        return s

    def group(st, u):
        for i in range(NH):
            for n, k in ((na, 2 * i), (nb, 2 * i + 1)):
                if k * 4 * NCS // (2 * NH) == u:
                    ev.append(("load", st if i < n and st < kLoop else None))

    npro = min(ns - 1, kLoop)
    for l in range(npro):
        ev.extend([("load", l)] * cnt)
    ev.extend([("wait", (npro - 1) * cnt), ("bar",)])
    st = window(ns - 1)
    ev.append(("read", 0))
    for q in range(4):
        group(st, q)
    for l in range(kLoop):
        for cs in range(NCS - 1):
            ev.append(("read", l))
            for q in range(4):
                group(st, 4 + 4 * cs + q)
        more = l + 1 < kLoop
        if more:
            ev.extend([("wait", 0 if ns == 2 else 2 * NH or (cnt if l + 2 < kLoop else 0)), ("bar",)])
            if NCS >= 2:
                ev.append(("read", l + 1))
        st = window(l + ns)
        for q in range(4):
            group(st, q)
        if NCS == 1 and more:
            ev.append(("read", l + 1))
    return ev


@pytest.mark.parametrize("ns", [1, 2, 3])
def test_ring_order(ns):
    """Every load is issued once, into a slot whose stage every wavefront has
    read (a barrier between), and has landed, a barrier before its first
    read, for wavefronts with fewer loads than others too."""
    for kLoop, NCS, most in itertools.product((1, 2, 3, 4, 7, 8, 20), (1, 2, 4, 8),
                                              (1, 2, 3, 4, 5, 8, 9, 16, 33)):
        for na, nb in {(most, most), (most, 0), (0, most), (most - 1, most), (most, most // 2)}:
            if ns > 1 and ns > kLoop:
                continue
            cnt = na + nb
            issued, ready, last_read, bars, landed = [], set(), {}, 0, set()
            for e in replay(ns, kLoop, NCS, na, nb, most):
                if e[0] == "load":
                    if e[1] is not None:
                        assert e[1] < kLoop
                        if e[1] >= ns:
                            assert last_read[e[1] - ns] < bars
                    issued.append(e[1])
                elif e[0] == "wait":
                    done = issued[:len(issued) - e[1]] if e[1] else issued
                    landed |= {s for s in set(done) if done.count(s) == cnt}
                elif e[0] == "bar":
                    bars += 1
                    ready |= landed
                else:
                    assert cnt == 0 or e[1] in ready
                    last_read[e[1]] = bars
            assert all(issued.count(s) == cnt for s in range(kLoop))


@pytest.mark.parametrize("akm", [False, True])
@pytest.mark.parametrize("space", [(1024, 1024, 1024), (192, 320, 128), (2048, 4096, 96),
                                   (96, 11008, 1 << 20)])
def test_lowered_launches_stay_in_bounds(gt, space, akm):
    """The launches the lowering chooses: the ring fits LDS and K, the
    operands' last tile and stage are reached and not passed, and a lane's
    offset from an instruction's origin fits 32 bits."""
    from test_kernel_model import levels
    M, N, K = space
    sp = gt.Space(M, N, K, (4, 4, 4), "f32", False, a_kmajor=akm)
    rng = random.Random(M + N + akm)
    code = gt.dtype_code("f32") | (gt.A_KMAJOR if akm else 0)
    seen = tries = 0
    while seen < 150 and tries < 400000:
        tries += 1
        c = sp.unrank(rng.randrange(sp.size()))
        if not sp.legit(c):
            continue
        info = gt.lower(c, M, N, K, code)
        if not info["fast"]:
            continue
        seen += 1
        L = levels(c)
        I, TM, TN, cpr, ns = info["I"], info["TM"], info["TN"], info["BK"] // 4, info["ring"]
        BM, BN, BK = info["BM"], info["BN"], info["BK"]
        assert 1 <= ns <= min(3, L["kLoop"]) and info["lds_bytes"] == ns * (BM + BN) * BK * 4 <= LDS_MAX
        lda = M if akm else K
        gm, gn, last = L["gridM"] - 1, L["gridN"] - 1, (L["kLoop"] * L["kSplit"] - 1) * BK
        orgA = last * M + gm * BM if akm else gm * BM * K + last
        orgB = last * N + gn * BN
        A, B = loads(I, TM, TN, cpr, L["wavesM"], L["wavesN"], akm, lda, N)
        for side, org, size in ((A, orgA, M * K), (B, orgB, K * N)):
            assert min(off.min() for _, _, off in side) == 0
            assert org + max(off.max() for _, _, off in side) + 4 == size, c
            # 32-bit byte offsets from the stage's origin, or the wide form
            wide = max(BK * M if akm else BM * K, BK * N) >= 1 << 30
            assert wide or max(off.max() for _, _, off in side) * 4 < 1 << 32
    assert seen >= 100, (seen, tries)


@pytest.mark.parametrize("dims,fast", [((256, 256, 1 << 24), 1), ((256, 256, 1 << 25), 0),
                                       ((256, 1 << 24, 256), 1), ((256, 1 << 25, 256), 0)])
def test_extents_whose_lane_offsets_would_wrap_take_the_generic_path(gt, dims, fast):
    M, N, K = dims
    cfg = ((M // 64, 2, 1, 32), (K // 32, 1, 1, 32), (N // 64, 2, 1, 32), 0)
    assert gt.lower(cfg, M, N, K, "f32")["fast"] == fast
