"""CPU models of the layouts of the two convolutions on the BF16 matrix instructions
(paper_2512_18863_amd/csrc/conv_fwd_reg.hip and conv_adj.hip), with FP64 numbers in place
of the BF16 pieces: where the taps' pieces lie in LDS (two copies of rows of equal length),
the run of every lane and where it is moved off the taps, the spare row read ahead, the
matrix instruction's lanes, row shifts, column groups, row and column chunks with and
without carried registers, zeros around the strips; the adjoint's window, its equal pieces,
the (group, tap row) pairs of each wavefront and the products of smaller tiles.

Every LDS and global address is checked against its buffer.  Operands are sums of NP
independent random pieces and the reference is the sum of the six piece convolutions that
the kernels take (BF16: one), so that a lost, doubled or misplaced piece shows.  Outputs
equal the direct convolution to FP64 rounding (1e-11 of the largest)."""
import os
import re

import numpy as np
import pytest

QB, GW = 2, 32
CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2512_18863_amd", "csrc")
MAXH, OFF, W = 31, 40, 41
PAIRS = {1: [(0, 0)], 3: [(2, 0), (0, 2), (1, 1), (1, 0), (0, 1), (0, 0)]}


def test_constants_of_the_source():
    s = open(os.path.join(CSRC, "conv_common.hpp")).read()
    val = lambda n: re.search(r"constexpr int %s = ([^;]+);" % n, s).group(1)
    assert int(val("kRegMaxH")) == MAXH
    assert eval(val("kRegOff"), {"kRegMaxH": MAXH}) == OFF
    assert int(eval(val("kRegW"), {"kRegMaxH": MAXH, "kRegOff": OFF})) == W
    f = open(os.path.join(CSRC, "conv_fwd_reg.hip")).read()
    assert "kRegQB = 2;" in f and "kRegGW = 32;" in f
    for name in ("conv_fwd_reg.hip", "conv_adj.hip"):
        t = open(os.path.join(CSRC, name)).read()
        for v in ("[6] = {2, 0, 1, 1, 0, 0}", "[6] = {0, 2, 1, 0, 1, 0}"):
            assert v in t


def tap_rows(K, h, NP, s0):
    """The LDS words of the tap rows as half-words; K[i][p][q] is piece i of tap (p, q)."""
    words = ((2 * (h + 1) + 1) * NP * W + 3) & ~3
    H = np.zeros(2 * words)
    CS = (h + 1) * NP * W
    for q in range(h + 1):
        for p in range(q + 1):
            for i in range(NP):
                for base, sh in ((2 * W * i, 0), (2 * W * i + 2 * CS, 1)):
                    for row, col, v in ((p, q, K[i][p][q] * (s0 if p == 0 else 1.0)),
                                        (q, p, K[i][p][q] * (s0 if q == 0 else 1.0))):
                        start = base + 2 * NP * W * row
                        for x in (OFF + col, OFF - col):
                            assert 0 <= x - sh < 2 * W
                            H[start + x - sh] = v
    return H, CS


def run_start(x, h, margin):
    """Element at which a lane's run starts, moved off the taps where it meets none."""
    x0, x1 = OFF - h - margin, OFF + h + 1
    x = np.where(x < x0 + 1, x0 + ((x ^ x0) & 1), x)
    return np.where(x > x1, x1 + ((x ^ x1) & 1), x)


def read(H, word, n):
    """n half-words from word offset `word` (per lane)."""
    i = 2 * word[:, None] + np.arange(n)
    assert i.min() >= 0 and i.max() < H.size
    return H[i]


LANES = np.arange(64)
N16, KK = LANES & 15, LANES >> 4


def mfma(a, b):
    """16 x 16 x 32: lane l = 16 kk + m holds A[m][8 kk + e] and B[8 kk + e][m]; D[j][n]."""
    m = lambda v: v.reshape(4, 16, 8).transpose(1, 0, 2).reshape(16, 32)
    return m(a) @ m(b).T


def shl(y, s):
    r = np.zeros_like(y)
    r[:, :16 - s] = y[:, s:]
    return r


def shr(y, s):
    r = np.zeros_like(y)
    r[:, s:] = y[:, :16 - s]
    return r


def forward(x, box, h, K, NP, T, SU, carry):
    """x[i]: piece i of the plane."""
    Nu, Nv = x[0].shape
    flat = [np.concatenate([p.ravel(), np.full(3, np.nan)]) for p in x]  # up to three words past the plane
    H, CS = tap_rows(K, h, NP, 1.0)
    dst = np.full((Nu, Nv), np.nan)
    r0, r1, c0, c1 = max(box[0], 0), min(box[1], Nu), max(box[2], 0), min(box[3], Nv)
    if r1 <= r0 or c1 <= c0:
        return np.zeros((Nu, Nv))
    cw0, cw1 = max(0, c0 - h), min(Nv, c1 + h)
    njt, nrc, ncc = (cw1 - cw0 + 15) // 16, -(-(r1 - r0) // (16 * T)), -(-(c1 - c0) // (GW * SU))
    NB = T + 2 * QB
    store = carry or nrc == 1
    if store:
        zr0 = min(max(r0 - 16 * QB, 0), Nu)
        zr1 = min(max(r0 + 16 * (T * nrc + QB), zr0), Nu)
        dst[:zr0], dst[zr1:] = 0.0, 0.0
        dst[zr0:zr1, :cw0], dst[zr0:zr1, min(Nv, cw0 + 16 * njt):] = 0.0, 0.0
    else:
        dst[:] = 0.0
    single = nrc == 1 and ncc == 1

    def run4(i, r, c):
        a = np.where(r < r1, r, r0) * Nv + np.where(c < c1, c, c0)
        idx = a[:, None] + np.arange(4)
        assert idx.min() >= 0 and idx.max() < flat[i].size
        ok = (r < r1)[:, None] & (c[:, None] + np.arange(4) < c1)
        return np.where(ok, flat[i][idx], 0.0)

    def load_b(R, C, t, u):
        r, c = R + 16 * t + N16, C + GW * u + 8 * KK
        return [np.concatenate([run4(i, r, c), run4(i, r, c + 4)], axis=1) for i in range(NP)]

    for jt in range(njt):
        J = cw0 + 16 * jt
        O = np.zeros((NB, 16, 16))
        for rc in range(nrc):
            R = r0 + 16 * T * rc
            if not carry:
                O[:] = 0.0
            for cc in range(ncc):
                C = c0 + GW * SU * cc
                nsu = min(SU, -(-(c1 - C) // GW))
                lo, hi = J - h - C - (GW - 1), J + 15 + h - C
                ua, ub = 0 if lo <= 0 else -(-lo // GW), min(nsu - 1, hi // GW if hi >= 0 else -1)
                if ua > ub:
                    continue
                B = [[load_b(R, C, t, u) if single or ua <= u <= ub else [np.zeros((64, 8))] * NP
                      for u in range(SU)] for t in range(T)]
                at = []
                for u in range(SU):
                    xx = run_start(C + GW * u + 8 * KK - J - N16 + OFF, h, 9)
                    assert xx.min() >= 0 and ((xx >> 1) + 3).max() < W
                    at.append(np.where(xx & 1, CS, 0) + (xx >> 1))
                for u in range(SU):
                    for i in range(NP):
                        read(H, at[u] + ((h + 1) * NP + i) * W, 8)  # (the spare row)
                for p in range(h + 1):
                    S, Q = p & 15, p >> 4
                    A = [[read(H, at[u] + (p * NP + i) * W, 8) for i in range(NP)] for u in range(SU)]
                    for t in range(T):
                        y = np.zeros((16, 16))
                        for u in sorted({0} | set(range(max(1, ua), ub + 1))):
                            for a, b in PAIRS[NP]:
                                y += mfma(A[u][a], B[t][u][b])
                        c = QB + t
                        if p == 0:
                            O[c] += y
                        elif S == 0:
                            O[c - Q] += y
                            O[c + Q] += y
                        else:
                            O[c - Q] += shl(y, S)
                            O[c - Q - 1] += shr(y, 16 - S)
                            O[c + Q] += shr(y, S)
                            O[c + Q + 1] += shl(y, 16 - S)
            for q in range(NB):
                for n in range(16):
                    row = R - 16 * QB + 16 * q + n
                    if 0 <= row < Nu:
                        w = min(16, Nv - J)
                        if store:
                            dst[row, J:J + w] = O[q, :w, n]
                        else:
                            dst[row, J:J + w] += O[q, :w, n]
            if carry:
                O = np.concatenate([O[T:], np.zeros((T, 16, 16))])
    return dst


def adjoint(x, box, h, K, NP, n, waves, grid_y):
    """x[i]: piece i of the plane.  The folded rows' pieces are the sums of the rows' (a split
    of the sum in the kernel)."""
    Nu, Nv = x[0].shape
    T = n
    H, CS = tap_rows(K, h, NP, 0.5)
    flat = [np.concatenate([p.ravel(), np.full(3, np.nan)]) for p in x]
    dst, writer = np.full((Nu, Nv), np.nan), np.full((Nu, Nv), -1)
    r0, r1, c0, c1 = max(box[0], 0), min(box[1], Nu), max(box[2], 0), min(box[3], Nv)
    if r1 <= r0 or c1 <= c0:
        return dst
    pitch = (min(Nv, 16 * n + 2 * h) + 31) // 32 * 32 + 8
    nr, nc = -(-(r1 - r0) // 16), -(-(c1 - c0) // 16)
    npi, npj = -(-nr // T), -(-nc // T)
    tr, tc = -(-nr // npi) if npi > 1 else nr, -(-nc // npj) if npj > 1 else nc
    for pp in [q for y in range(grid_y) for q in range(y, npi * npj, grid_y)]:
        I, J = r0 + 16 * tr * (pp // npj), c0 + 16 * tc * (pp % npj)
        I1, J1 = min(I + 16 * tr, r1), min(J + 16 * tc, c1)
        wc0, wc1 = max(0, J - h), min(Nv, J1 + h)
        ng = -(-(wc1 - wc0) // 32)
        assert 32 * ng <= pitch
        img = np.full((NP, 16 * T + 2 * h, pitch), np.nan)  # (what is not staged is anything)
        for r in range(16 * tr + 2 * h):
            for q in range(8 * ng):
                pr, pc = I - h + r, wc0 + 4 * q
                v = np.zeros((NP, 4))
                if 0 <= pr < Nu and pc < wc1:
                    for i in range(NP):
                        a = pr * Nv + pc
                        assert a + 4 <= flat[i].size
                        v[i] = np.where(pc + np.arange(4) < wc1, flat[i][a:a + 4], 0.0)
                img[:, r, 4 * q:4 * q + 4] = v
        side = max(I1 - I, J1 - J)
        st, sc = I1 - I <= 16 * (T - 1), J1 - J <= 16 * (T - 1)
        if T > 2 and side <= 16:
            TT, CC = 1, 1
        elif T > 3 and side <= 32:
            TT, CC = 2, 2
        else:
            TT, CC = max(T - 1, 1) if st else T, max(T - 1, 1) if sc else T
        acc = np.zeros((T, T, 16, 16))
        total = ng * (h + 1)
        for wave in range(waves):
            ua, uz = total * wave // waves, total * (wave + 1) // waves
            gq = ua // (h + 1)
            while gq * (h + 1) < uz:
                pa, pz = max(ua - gq * (h + 1), 0), min(uz - gq * (h + 1), h + 1)
                for p in range(pa, pz):
                    A = [[None] * NP for _ in range(CC)]
                    for c in range(CC):
                        for i in range(NP):
                            half = []
                            for e in range(2):
                                xx = run_start(OFF + wc0 + 32 * gq + 16 * e + 4 * KK - (J + 16 * c + N16), h, 5)
                                assert xx.min() >= 0 and ((xx >> 1) + 1).max() < W
                                half.append(read(H, np.where(xx & 1, CS, 0) + (xx >> 1) + (p * NP + i) * W, 4))
                            A[c][i] = np.concatenate(half, axis=1)
                    for t in range(TT):
                        col = 32 * gq + 4 * KK[:, None] + np.array([0, 1, 2, 3, 16, 17, 18, 19])
                        up, dn = 16 * t + N16 + h + p, 16 * t + N16 + h - p
                        assert col.max() < pitch and up.max() < img.shape[1] and dn.min() >= 0
                        fold = [img[i][up[:, None], col] + img[i][dn[:, None], col] for i in range(NP)]
                        for c in range(CC):
                            for a, b in PAIRS[NP]:
                                acc[t, c] += mfma(A[c][a], fold[b])
                gq += 1
        for t in range(T):
            for c in range(T):
                for m in range(16):
                    i = I + 16 * t + m
                    if i >= min(I + 16 * tr, Nu):
                        continue
                    j0, j1 = J + 16 * c, min(J + 16 * c + 16, J + 16 * tc, Nv)
                    if j1 > j0:
                        assert (writer[i, j0:j1] == -1).all()  # one piece writes an output
                        writer[i, j0:j1] = pp
                        dst[i, j0:j1] = acc[t, c, :j1 - j0, m]
    return dst


def direct(x, h, K, NP):
    Nu, Nv = x[0].shape
    pad = [np.pad(p, h) for p in x]
    out = np.zeros((Nu, Nv))
    for a, b in PAIRS[NP]:
        for p in range(-h, h + 1):
            for q in range(-h, h + 1):
                out += K[a][abs(p), abs(q)] * pad[b][h + p:h + p + Nu, h + q:h + q + Nv]
    return out


def _inputs(Nu, Nv, h, NP):
    rng = np.random.default_rng(Nu + 3 * Nv + 7 * h + NP)
    K = rng.uniform(0.1, 1.0, size=(NP, h + 1, h + 1))
    return [rng.normal(size=(Nu, Nv)) for _ in range(NP)], K + K.transpose(0, 2, 1)


# plane, half-width, rectangle, row blocks per chunk, column groups, carried
FORWARD = [
    (25, 23, 6, (8, 14, 3, 12), 1, 1, 0), (25, 23, 6, (8, 14, 3, 12), 1, 1, 1), (57, 51, 15, (15, 44, 14, 43), 2, 1, 0),
    (73, 71, 31, (28, 47, 20, 54), 2, 2, 0), (73, 71, 31, (20, 55, 8, 66), 3, 2, 0), (95, 90, 30, (8, 88, 0, 90), 5, 2, 0),
    (99, 71, 1, (0, 99, 3, 68), 6, 2, 1), (150, 90, 16, (5, 149, 2, 90), 4, 2, 1), (150, 90, 17, (5, 149, 2, 90), 3, 1, 0),
    (40, 120, 6, (3, 38, 1, 118), 1, 2, 1), (30, 30, 8, (12, 12, 3, 20), 2, 2, 0), (45, 40, 16, (-3, 60, -2, 50), 1, 1, 1),
    (50, 47, 16, (20, 21, 46, 47), 2, 2, 0),
]


@pytest.mark.parametrize("NP", [1, 3])
@pytest.mark.parametrize("Nu,Nv,h,box,T,SU,carry", FORWARD)
def test_forward(Nu, Nv, h, box, T, SU, carry, NP):
    x, K = _inputs(Nu, Nv, h, NP)
    got = forward(x, box, h, K, NP, T, SU, carry)
    inside = np.zeros((Nu, Nv))
    inside[max(box[0], 0):box[1], max(box[2], 0):box[3]] = 1.0
    ref = direct([p * inside for p in x], h, K, NP)
    assert np.isfinite(got).all()
    assert np.abs(got - ref).max() <= 1e-11 * max(1.0, np.abs(ref).max())


# plane, half-width, rectangle, tiles per side of a piece, wavefronts, workgroups per item
ADJOINT = [
    (25, 23, 6, (8, 14, 3, 12), 1, 4, 1), (57, 51, 15, (15, 44, 14, 43), 2, 4, 1), (57, 51, 15, (15, 61, -2, 51), 2, 4, 2),
    (73, 71, 31, (20, 65, 8, 56), 3, 8, 1), (73, 71, 31, (30, 41, 28, 44), 3, 8, 1), (73, 71, 31, (30, 62, 28, 55), 4, 8, 1),
    (100, 97, 16, (3, 92, 1, 96), 3, 4, 4), (100, 97, 16, (3, 92, 1, 96), 4, 8, 4), (90, 60, 1, (0, 90, 0, 60), 4, 4, 1),
    (60, 90, 30, (9, 50, 1, 25), 4, 8, 1), (30, 30, 8, (12, 12, 3, 20), 2, 4, 1), (120, 40, 17, (20, 110, 10, 25), 3, 8, 1),
]


@pytest.mark.parametrize("NP", [1, 3])
@pytest.mark.parametrize("Nu,Nv,h,box,n,waves,grid_y", ADJOINT)
def test_adjoint(Nu, Nv, h, box, n, waves, grid_y, NP):
    x, K = _inputs(Nu, Nv, h, NP)
    got = adjoint(x, box, h, K, NP, n, waves, grid_y)
    s = np.s_[max(box[0], 0):min(box[1], Nu), max(box[2], 0):min(box[3], Nv)]
    ref = direct(x, h, K, NP)[s]
    assert np.isfinite(got[s]).all()
    if ref.size:
        assert np.abs(got[s] - ref).max() <= 1e-11 * np.abs(ref).max()
