"""A CPU model of the ring kernel (fp32, and bf16 stages that the evenly
shared direct-load kernel does not take): where its direct loads put each
element of a stage in LDS, what its fragment reads find there, how far its
global addresses reach, and the order of loads, waits, barriers and reads of
its ring, over every kernel shape and over the launches the lowering chooses.
The model restates the kernel's index formulas; it shares no code with it."""
import functools
import itertools
import os
import random

import numpy as np
import pytest

from test_kernel_model import bswz, swz

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


def flip_panel(I, C):
    return I == 16 and C in (8, 16)


def planes(bf16, I, cpr):
    return bf16 and I == 16 and cpr // 4 >= 2


def share(w, nw, blocks, insts):
    b0, db = w // blocks, nw // blocks
    return w % blocks, range(b0, b0 + (insts - b0 + db - 1) // db * db, db)


def row_loads(w, nw, BM, cpr, ld, bf16, I):
    """A wavefront's loads of a row-major A: per instruction its slot in the
    stage (units of 64 chunks) and the lanes' element offsets from the stage's
    origin."""
    vec = 8 if bf16 else 4
    out = []
    for b in share(w, nw, 1, BM * cpr >> 6)[1]:
        s = b << 6
        if planes(bf16, I, cpr):
            p, inn = divmod(s, 4 * BM)
            q = swz(inn + LANE)
            out.append((b, (q >> 2) * ld + (p * 4 + (q & 3)) * vec))
        else:
            row = s // cpr + LANE // cpr
            out.append((b, row * ld + ((LANE % cpr) ^ fswz(row, cpr)) * vec))
    return out


def panel_loads(w, nw, panels, I, W, BK, ld, bf16):
    """The same of a [k][n] operand in panels of W columns."""
    vec = 8 if bf16 else 4
    C = W // vec
    insts = BK * C // 64
    panel, bs = share(w, nw, panels, insts)
    out = []
    for b in bs:
        s = b << 6
        k = s // C + (LANE * 0 if C >= 64 else LANE // C)
        pos = s % C + LANE if C >= 64 else LANE % C
        x = np.array([bswz(int(v), C) for v in k]) if bf16 else (k & 4 if flip_panel(I, C) else 0 * k)
        out.append((panel * insts + b, k * ld + panel * W + (pos ^ x) * vec))
    return out


def loads(I, TM, TN, cpr, wavesM, wavesN, ak, lda, ldb, bf16=False):
    """Every load of a stage: (wavefront, slot, element offsets), A's and B's."""
    nw, BK = wavesM * wavesN, cpr * (8 if bf16 else 4)
    A, B = [], []
    for w in range(nw):
        A += [(w, *t) for t in (panel_loads(w, nw, wavesM, I, TM * I, BK, lda, bf16) if ak
                                else row_loads(w, nw, wavesM * TM * I, cpr, lda, bf16, I))]
        B += [(w, *t) for t in panel_loads(nw - 1 - w, nw, wavesN, I, TN * I, BK, ldb, bf16)]
    return A, B


def stage(I, TM, TN, cpr, wavesM, wavesN, ak, bf16):
    """A slot of the ring as arrays of the (outer, k) each element of it holds,
    filled by every instruction of the stage; returns the arrays and A's size
    in elements."""
    vec = 8 if bf16 else 4
    BM, BN, BK = wavesM * TM * I, wavesN * TN * I, cpr * vec
    pa, pt = BM * cpr >> 6, (BM + BN) * cpr >> 6
    outer = np.full(pt * 64 * vec, -1)
    kk = np.full(pt * 64 * vec, -1)
    ld = 1 << 20   # a leading dimension that separates rows from columns
    A, B = loads(I, TM, TN, cpr, wavesM, wavesN, ak, ld, ld, bf16)
    for side, base, n, trans in ((A, 0, pa, not ak), (B, pa, pt - pa, False)):
        assert sorted(p for _, p, _ in side) == list(range(n))   # each slot once
        for _, p, off in side:
            words = (base + p) * 64 * vec + LANE[:, None] * vec + np.arange(vec)
            e = off[:, None] + np.arange(vec)
            r, c = e // ld, e % ld
            outer[words], kk[words] = (r, c) if trans else (c, r)
    assert outer.min() >= 0 and kk.min() >= 0 and kk.max() < BK
    na = pa * 64 * vec
    assert outer[:na].max() < BM and outer[na:].max() < BN
    assert len(set(zip(outer[:na], kk[:na]))) == na
    assert len(set(zip(outer[na:], kk[na:]))) == len(outer) - na
    return outer, kk, na


SHAPES = [(I, TM, TN, cpr) for I in (16, 32) for cpr in (2, 4, 8, 16) if cpr >= 64 // I
          for TM, TN in itertools.product((1, 2, 4, 8, 16), repeat=2) if TM * TN * I * I // 64 <= 256]


@functools.lru_cache(maxsize=None)
def check_reads(bf16, ak, I, TM, TN, cpr, wavesM, wavesN):
    """Every fragment read of every wavefront finds the element its MFMA lane
    needs."""
    vec = 8 if bf16 else 4
    G = 64 // I
    grp, l0 = LANE // I, LANE % I
    i16, g16 = LANE & 15, LANE >> 4
    BK, WM, WN, BM = cpr * vec, TM * I, TN * I, wavesM * TM * I
    outer, kk, na = stage(I, TM, TN, cpr, wavesM, wavesN, ak, bf16)

    def panel_read(wi, t, W, cs, q):      # fp32
        col = t * I + l0
        if flip_panel(I, W // 4):
            col = col ^ ((grp & 1) << 4)
        return wi * BK * W + grp * 4 * W + col + (cs * G * 4 + q) * W

    for wm, wn, cs in itertools.product(range(wavesM), range(wavesN), range(cpr // G)):
        for t in range(TM):
            row = wm * WM + t * I + l0
            for q in range(4 if not bf16 else 8):
                k = (cs * G + grp) * vec + q
                if ak:
                    w = panel_read(wm, t, WM, cs, q)
                elif planes(bf16, I, cpr):
                    w = (cs * 4 * BM + swz((row << 2) + grp)) * 8 + q
                else:
                    w = (row * cpr + ((fswz(l0, cpr) ^ grp) ^ (cs * G))) * vec + q
                assert (outer[w] == row).all() and (kk[w] == k).all()
        for t in range(TN):
            want = wn * WN + t * I + l0
            if not bf16:
                for q in range(4):
                    w = na + panel_read(wn, t, WN, cs, q)
                    assert (outer[w] == want).all() and (kk[w] == (cs * G + grp) * 4 + q).all()
                continue
            # the transposing read: lane l of a 16-lane group gets, as its
            # j-th value, element l & 3 of what lane 4j + (l >> 2) addresses
            C = WN // 8
            kr = (g16 >> 1 if I == 32 else g16) * 8 + (i16 >> 2)
            col = t * I + (16 * (g16 & 1) if I == 32 else 0) + 4 * (i16 & 3)
            x = np.array([bswz(int(v), C) for v in kr])
            at = na + wn * BK * WN + (kr * C + ((col >> 3) ^ x)) * 8 + (col & 4)
            for hh, j in itertools.product(range(2), range(4)):
                w = at[16 * g16 + 4 * j + (i16 >> 2)] + (cs * G * 8 + 4 * hh) * WN + (LANE & 3)
                assert (outer[w] == want).all()
                assert (kk[w] == cs * G * 8 + (LANE // I) * 8 + 4 * hh + j).all()


@pytest.mark.parametrize("bf16,ak", [(False, False), (False, True), (True, False)])
def test_reads_find_what_the_loads_wrote(bf16, ak):
    for I, TM, TN, cpr in SHAPES:
        for wavesM, wavesN in ((1, 1), (2, 1), (1, 2), (4, 2)):
            if (wavesM * TM + wavesN * TN) * I * cpr * 16 <= LDS_MAX:
                check_reads(bf16, ak, I, TM, TN, cpr, wavesM, wavesN)


def replay(ns, kLoop, NCS, na, nb, most, SG, streams):
    """One wavefront's loads, waits, barriers and reads, in program order; a
    load that moves nothing is ("load", None). na, nb: its loads of A and B;
    most: the most of either that any wavefront has; streams: the form that
    reads a chunk-step's fragments while it multiplies them."""
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
            for n, at in ((na, i * NCS * SG // NH), (nb, (2 * i + 1) * NCS * SG // (2 * NH))):
                if u < 0 or at == u:
                    ev.append(("load", st if i < n and st < kLoop else None))

    def wait(l):
        if NH == 0:
            ev.append(("wait", max(min(ns - 2, kLoop - 2 - l), 0) * cnt))
        else:
            ev.append(("wait", (ns - 2) * 2 * NH))

    for l in range(ns - 1):
        group(window(l), -1)
    wait(-1)
    ev.append(("bar",))
    if streams:
        for l in range(kLoop):
            st = window(l + ns - 1)
            for cs in range(NCS):
                ev.append(("read", l))
                for g in range(SG):
                    ev.append(("read", l))
                    group(st, SG * cs + g)
            if l + 1 < kLoop:
                wait(l)
                ev.append(("bar",))
        return ev
    st = window(ns - 1)
    ev.append(("read", 0))
    for g in range(SG):
        group(st, g)
    for l in range(kLoop):
        for cs in range(NCS - 1):
            ev.append(("read", l))
            for g in range(SG):
                group(st, SG + SG * cs + g)
        more = l + 1 < kLoop
        if more:
            wait(l)
            ev.append(("bar",))
            if NCS >= 2:
                ev.append(("read", l + 1))
        st = window(l + ns)
        for g in range(SG):
            group(st, g)
        if NCS == 1 and more:
            ev.append(("read", l + 1))
    return ev


@functools.lru_cache(maxsize=None)
def check_order(ns, kLoop, NCS, na, nb, most, SG, streams):
    cnt = na + nb
    issued, ready, last_read, bars, landed = [], set(), {}, 0, set()
    for e in replay(ns, kLoop, NCS, na, nb, most, SG, streams):
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


@pytest.mark.parametrize("streams", [False, True])
@pytest.mark.parametrize("ns", range(1, 9))
def test_ring_order(ns, streams):
    """Every load is issued once, into a slot whose stage every wavefront has
    read (a barrier between), and has landed, a barrier before its first
    read, for wavefronts with fewer loads than others too."""
    for SG, kLoop, NCS, most in itertools.product((1, 2, 4), (1, 2, 3, 4, 7, 8, 20), (1, 2, 4, 8),
                                              (1, 2, 3, 4, 5, 8, 9, 16, 33)):
        for na, nb in {(most, most), (most, 0), (0, most), (most - 1, most), (most, most // 2)}:
            check_order(ns, kLoop, NCS, na, nb, most, SG, streams)


def check_bounds(L, info, M, N, K, bf16, akm):
    """The ring fits LDS and K, the operands' last tile and stage are reached
    and not passed, offsets fit 32 bits unless the loads step 64-bit
    addresses. Returns the loads of a stage."""
    size, vec = (2, 8) if bf16 else (4, 4)
    I, TM, TN, cpr, ns = info["I"], info["TM"], info["TN"], info["BK"] // vec, info["ring"]
    BM, BN, BK = info["BM"], info["BN"], info["BK"]
    assert 1 <= ns <= (8 if bf16 else 3) and (info["dl"] or ns <= L["kLoop"])
    assert info["lds_bytes"] == ns * (BM + BN) * BK * size <= LDS_MAX
    lda = M if akm else K
    gm, gn, last = L["gridM"] - 1, L["gridN"] - 1, (L["kLoop"] * L["kSplit"] - 1) * BK
    orgA = last * M + gm * BM if akm else gm * BM * K + last
    orgB = last * N + gn * BN
    A, B = loads(I, TM, TN, cpr, L["wavesM"], L["wavesN"], akm, lda, N, bf16)
    for side, org, end in ((A, orgA, M * K), (B, orgB, K * N)):
        assert min(off.min() for _, _, off in side) == 0
        assert org + max(off.max() for _, _, off in side) + vec == end, info
        wide = max(BK * M if akm else BM * K, BK * N) * size >= 1 << 32
        assert wide or max(off.max() for _, _, off in side) * size < 1 << 32
    return A, B


def check_ring(L, info, M, N, K, bf16, akm):
    """One launch of the ring kernel: its addresses, its reads of LDS and the
    order of each of its wavefronts."""
    A, B = check_bounds(L, info, M, N, K, bf16, akm)
    I, TM, TN, cpr = info["I"], info["TM"], info["TN"], info["BK"] // (8 if bf16 else 4)
    check_reads(bf16, akm, I, TM, TN, cpr, L["wavesM"], L["wavesN"])
    nw, NCS = L["W"], cpr // (64 // I)
    acc = TM * TN * I * I // 64
    spare = 32 if not bf16 and cpr == 16 and acc == 256 else 80
    streams = I == 16 and acc + 9 * (TM + TN) + spare > (512 if acc + 96 > 256 else 256)
    SG = min(TM * TN, 4) if bf16 else 4
    most = max(-(-info[x] * cpr // (64 * nw)) for x in ("BM", "BN"))
    for w in range(nw):
        na, nb = (sum(1 for v, _, _ in side if v == w) for side in (A, B))
        assert max(na, nb) <= most
        wide = max(info["BK"] * M if akm else info["BM"] * K, info["BK"] * N) * (2 if bf16 else 4) >= 1 << 32
        # the schedule repeats from one turn of the ring to the next
        check_order(info["ring"], min(L["kLoop"], 20), NCS, na, nb, 9 if wide else most, SG, streams)


@pytest.mark.parametrize("dt,akm", [("f32", False), ("f32", True), ("bf16", False)])
@pytest.mark.parametrize("space", [(1024, 1024, 1024), (192, 320, 128), (2048, 4096, 96),
                                   (96, 11008, 1 << 20)])
def test_lowered_launches_stay_in_bounds(gt, space, dt, akm):
    """The launches the lowering chooses: the ring fits LDS and K, the
    operands' last tile and stage are reached and not passed, and offsets fit
    32 bits unless the wide form takes them."""
    from test_kernel_model import levels
    M, N, K = space
    bf16 = dt == "bf16"
    sp = gt.Space(M, N, K, (4, 4, 4), dt, bf16, a_kmajor=akm)
    rng = random.Random(M + N + akm)
    code = gt.dtype_code(dt) | (gt.A_KMAJOR if akm else 0)
    seen = tries = 0
    while seen < 120 and tries < 400000:
        tries += 1
        c = sp.unrank(rng.randrange(sp.size()))
        if not sp.legit(c):
            continue
        info = gt.lower(c, M, N, K, code)
        if not info["fast"]:
            continue
        seen += 1
        L = levels(c)
        if info["kernel"] == "ring":
            check_ring(L, info, M, N, K, bf16, akm)
        else:       # the evenly shared loads reach the same places
            check_bounds(L, info, M, N, K, bf16, akm)
    assert seen >= 80, (seen, tries)


@pytest.mark.parametrize("dt,dims", [
    ("f32", (256, 256, 1 << 25)), ("f32", (256, 256, 1 << 26)), ("f32", (256, 1 << 26, 256)),
    ("f32", (256, 1 << 27, 256)), ("bf16", (256, 256, 1 << 26)), ("bf16", (256, 256, 1 << 27))])
def test_extents_whose_lane_offsets_would_wrap_stay_on_the_ring(gt, dt, dims):
    """16 rows of A, or the 8 rows of a 32-column fp32 panel, reach 2^32 bytes:
    the loads there step a 64-bit address per lane, so no extent leaves the
    fast path."""
    M, N, K = dims
    cfg = ((M // 64, 2, 1, 32), (K // 32, 1, 1, 32), (N // 64, 2, 1, 32), 32 if dt == "bf16" else 0)
    info = gt.lower(cfg, M, N, K, dt)
    assert info["fast"] == 1 and info["ring"] >= 2


@pytest.mark.parametrize("bf16,ak", [(False, False), (False, True), (True, False)])
def test_stepped_loads_equal_the_numbered_ones(bf16, ak):
    """The loads issued at once add a step from one to the next; here their
    places are worked out by the same steps and compared with each load's own."""
    vec = 8 if bf16 else 4
    ld = 1 << 36       # rows far beyond 32 bits
    for I, TM, TN, cpr in SHAPES:
        BK = cpr * vec
        for wavesM, wavesN in ((1, 1), (2, 1), (1, 2), (4, 2)):
            nw, BM = wavesM * wavesN, wavesM * TM * I
            for w in range(nw):
                for panels, W, ww in ((wavesN, TN * I, nw - 1 - w),) + (((wavesM, TM * I, w),) if ak else ()):
                    C = W // vec
                    RI, IR = max(64 // C, 1), max(C // 64, 1)
                    panel, bs = share(ww, nw, panels, BK * C // 64)
                    db, b, got = nw // panels, ww // panels, []
                    k = b // IR * RI + (LANE * 0 if C >= 64 else LANE // C)
                    at = panel * W + k * ld
                    for _ in bs:
                        x = np.array([bswz(int(v), C) for v in k]) if bf16 else (k & 4 if flip_panel(I, C) else 0 * k)
                        pos = (b % IR * 64 + LANE if C >= 64 else LANE % C) ^ x
                        got.append((panel * (BK * C // 64) + b, at + pos * vec))
                        b += db
                        at = at + (db * RI * ld if IR == 1 else (b // IR - k) * ld)
                        k = k + db * RI if IR == 1 else 0 * k + b // IR
                    want = panel_loads(ww, nw, panels, I, W, BK, ld, bf16)
                    assert [g[0] for g in got] == [g[0] for g in want]
                    assert all((g[1] == v[1]).all() for g, v in zip(got, want))
                if not ak:
                    b, got = w, []
                    s = (b << 6) + LANE
                    for _ in share(w, nw, 1, BM * cpr >> 6)[1]:
                        if planes(bf16, I, cpr):
                            q = swz(s % (4 * BM))
                            off = (q >> 2) * ld + s // (4 * BM) * 4 * vec + (q & 3) * vec
                        else:
                            row = s // cpr
                            off = row * ld + ((s % cpr) ^ fswz(row, cpr)) * vec
                        got.append((b, off))
                        b, s = b + nw, s + (nw << 6)
                    want = row_loads(w, nw, BM, cpr, ld, bf16, I)
                    assert [g[0] for g in got] == [g[0] for g in want]
                    assert all((g[1] == v[1]).all() for g, v in zip(got, want))
