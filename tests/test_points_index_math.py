"""Host-side emulation of the point finder and binning of the gridding kernels
(paper_1307_5824_amd/csrc/points.h) for every tile and window width that they launch: the LDS and
bit-field budgets, the bins' footprints inside the tile, the even/odd window polynomials, and the FP32
plane, row and slab tests against every half-disk point of random views.  Runs on the CPU; no kernel
is launched."""
import math

import numpy as np
import pytest

NTH, NW, GROUP, RUN, SURV = 1024, 16, 32768, 64, 96
LDS = 160 * 1024 - 640  # 132 row starts of the disk are the kernels' own
# (lattice step, bins along axis 0, bound on P1, row pitch, bytes per cell, floats per value)
KINDS = {"ker": (4, 1, 22, 22, 8, 1), "atb": (2, 1, 14, 18, 16, 2), "atb8": (2, 1, 16, 18, 16, 2),
         "prj": (2, 1, 18, 18, 8, 2), "prjw": (2, 1, 22, 22, 8, 2)}


class Tile:
    def __init__(self, kind, W):
        if kind == "atb" and W == 8:
            kind = "atb8"
        self.S, NB0, P1MAX, self.RP, CELL, self.NV = KINDS[kind]
        self.W = W
        self.CHUNK = 32 if W == 8 else 64
        self.NJ = 8 if W == 8 else 4
        self.CJ = 2 * self.NJ
        self.B = (17 - W, self.CJ + 1 - W, 9 - W)
        self.NB = (NB0, (P1MAX - W + 1) // self.B[1], (self.RP - W + 1) // self.B[2])
        self.T = tuple(n * b for n, b in zip(self.NB, self.B))
        self.P = tuple(t + W - 1 for t in self.T)
        self.P1MAX = P1MAX
        self.PADLO = (W + 1) // 2 - 1
        self.nbins = math.prod(self.NB)
        self.S0, self.LEAD, self.SB, self.OFFV = 20, 12, self.CJ + 12, self.CJ + 8
        self.WAVE = self.LEAD + 16 * self.S0 + 16 * self.SB
        fixed = (self.P[0] * self.P[1] * self.RP * CELL + NW * self.WAVE * 4 + NW * SURV * 2 + GROUP // RUN * 2 +
                 self.nbins * 4 + 64)
        per = lambda q: q * (20 + 4 * self.NV) + (q // self.CHUNK + self.nbins) * 4  # noqa: E731
        q = 4096
        while q > 1024 and fixed + per(q) > LDS:
            q -= 256
        self.QCAP, self.lds = q, fixed + per(q)
        self.DIAG = math.isqrt(sum(t * t for t in self.T) - 1) + 1
        self.ROWS, self.CMAX = self.DIAG // self.S + 1, self.DIAG // self.S + 2


ALL = [(k, W) for k in ("ker", "atb", "prj", "prjw") for W in range(4, 9)]


@pytest.mark.parametrize("kind,W", ALL)
def test_budgets_and_footprints(kind, W):
    t = Tile(kind, W)
    assert t.lds <= LDS and all(n >= 1 for n in t.NB) and t.P[1] <= t.P1MAX and t.P[2] <= t.RP and t.nbins <= 192
    # a chunk-table entry: bin above bit 20, start in 13 bits, count in 7; the packed scan of
    # (chunks << 16) | points; at most one chunk per CHUNK points and one more per bin
    assert t.QCAP <= 8191 and t.CHUNK < 128 and t.nbins < 2048
    assert t.QCAP // t.CHUNK + t.nbins < 32768 and t.QCAP < 65536
    assert 64 * t.CMAX <= t.QCAP  # one step of a wavefront always fits an empty queue
    # a queue entry: 15 bits of view, k1 <= N/2 <= 128 in 8, k2 + 256 in 9; views collected per step
    assert GROUP <= 1 << 15 and GROUP // RUN * RUN == GROUP and SURV - RUN + RUN <= SURV
    # every bin's 16 x CJ x 8 footprint lies inside the padded tile; a start o in the bin and its W
    # weights fit the padded weight rows, and the start fits 4 bits
    for d, foot in ((0, 16), (1, t.CJ), (2, 8)):
        assert (t.NB[d] - 1) * t.B[d] + foot <= (t.P[d] if d < 2 else t.RP)
        assert t.B[d] - 1 + W <= foot and t.B[d] <= 16
    # the lanes of one quarter of an 8-byte access: two rows of 8 cells, at W <= 7 in 16 distinct slots
    for n in range(t.NJ):
        slots = {((t.NJ * e + n) * t.RP + k) % 16 for e in range(2) for k in range(8)}
        assert len(slots) == (16 if t.NJ == 4 else 8)


@pytest.mark.parametrize("W", range(4, 9))
def test_staged_points(W):
    """The wavefront's staging area: what the four lanes of a point write (axis-0 weights in 8 slots,
    axis 1 in CJ, axis 2 in 8, the value in 4) does not overlap, and the weight of footprint row i,
    read i - o0 floats after the point's first, is its window's or a zero that nothing writes."""
    t = Tile("ker", W)
    written, base = {}, t.LEAD + 16 * t.S0
    for p in range(16):
        for what, at, n in (("w0", t.LEAD + p * t.S0, 8), ("w1", base + p * t.SB, t.CJ),
                            ("w2", base + p * t.SB + t.CJ, 8), ("v", base + p * t.SB + t.OFFV, 4)):
            assert at % 4 == 0
            for k in range(n):
                assert at + k not in written and at + k < t.WAVE
                written[at + k] = (what, p, k)
    for p in range(16):
        for o in range(t.B[0]):
            for i in range(16):
                at = t.LEAD + p * t.S0 + i - o
                assert 0 <= at < t.WAVE
                k = i - o
                if 0 <= k < W:
                    assert written[at] == ("w0", p, k)
                else:  # a slot past the window's end (written as zero) or one that is never written
                    assert at not in written or (written[at][0] == "w0" and written[at][2] >= W)


@pytest.mark.parametrize("W", range(4, 9))
def test_window_polynomials_mirror(W):
    """The window is even, so cell W-1-j's polynomial is cell j's at -x: the even and odd coefficients of
    the first half of the cells give all weights to FP64 rounding."""
    beta = np.pi * np.sqrt((W / 2) ** 2 * 1.5 ** 2 - 0.8)
    D = 10
    x = np.cos(np.pi * (np.arange(D + 1) + 0.5) / (D + 1))
    coef = []
    for j in range(W):
        u = 0.5 * (x + 1) - 0.5 * W + j
        phi = np.i0(beta * np.sqrt(np.maximum(0.0, 1 - (2 * u / W) ** 2))) / np.i0(beta)
        coef.append(np.linalg.solve(np.vander(x, D + 1, increasing=True), phi))
    z = np.linspace(-1, 1, 101)
    for j in range((W + 1) // 2):
        a, b = coef[j], coef[W - 1 - j]
        even, odd = 0.5 * (a + b)[0::2], 0.5 * (a - b)[1::2]
        e, o = np.polyval(even[::-1], z * z), np.polyval(odd[::-1], z * z) * z
        assert np.abs(e + o - np.polyval(a[::-1], z)).max() < 1e-11
        assert np.abs(e - o - np.polyval(b[::-1], z)).max() < 1e-11


def test_unit_conversion_is_exact():
    """x + 1.5 2^52 in FP64, less the constant's bits, is the integer nearest to x."""
    x = np.concatenate([np.linspace(-3, 3, 25), [2.0 ** 37, -2.0 ** 37 + 3, 12345678.5, 2 ** 31 - 1]]).astype(np.float32)
    t = (x.astype(np.float64) + 6755399441055744.0).view(np.int64) - 0x4338000000000000
    assert np.array_equal(t, np.rint(x.astype(np.float64)).astype(np.int64))


@pytest.mark.parametrize("kind,W", ALL)
def test_every_point_is_found_by_its_tile(kind, W):
    """For each half-disk point: its window start's tile passes the view test in FP32, the point's row is
    one of the view's ROWS, and its k2 lies in the FP32 slab interval, less than CMAX from its start."""
    f32 = np.float32
    t = Tile(kind, W)
    N = 128
    L, s = t.S * N, t.S
    rng = np.random.default_rng(100 + W)
    k = np.arange(-N // 2, N // 2 + 1)
    k1, k2 = (a.ravel() for a in np.meshgrid(k, k, indexing="ij"))
    half = (4 * (k1 * k1 + k2 * k2) <= N * N) & ((k1 > 0) | ((k1 == 0) & (k2 > 0)))
    k1, k2 = k1[half], k2[half]
    H = np.array([0.5 * v for v in t.T], dtype=f32)
    HW = 0.5 if W % 2 else 0.0
    for v in range(16):
        q, r = np.linalg.qr(rng.standard_normal((3, 3)))
        R = q * np.sign(np.diag(r))[None, :]
        if v < 3:
            R = np.roll(np.eye(3), v, axis=0)  # slices along the axes: points on the tiles' edges
        c1, c2 = R[0], R[1]
        n = np.cross(c1, c2).astype(f32)
        tau = np.clip(s * (k2[:, None] * c2 + k1[:, None] * c1) + 0.5 * L, 0.0, L)
        start = np.floor(tau - 0.5 * W).astype(np.int64) + 1 + t.PADLO
        assert start.min() >= 0 and start.max() <= L
        tt = start // np.array(t.T)
        c = (tt * np.array(t.T) + H - HW - 0.5 * L).astype(f32)
        c1f, c2f = c1.astype(f32), c2.astype(f32)
        assert np.all(np.abs(c @ n) <= (H * np.abs(n)).sum() + f32(2e-3))
        assert np.all(c @ c1f + (H * np.abs(c1f)).sum() >= f32(-2e-3))
        cs = (c / f32(s)).astype(f32)
        uc = cs @ c1f
        uh = (H / f32(s) * np.abs(c1f)).sum() + f32(1e-3)
        first = np.ceil(uc - uh).astype(np.int64)
        assert np.all(k1 >= first) and np.all(k1 < first + t.ROWS) and np.all(k1 <= uc + uh)
        kd = np.floor(np.sqrt((N * N // 4 - k1 * k1).astype(np.float64) + 1e-9))
        lo, hi = np.where(k1 == 0, 1.0, -kd), kd.copy()
        for d in range(3):
            al = (k1.astype(f32) * c1f[d] - cs[:, d]).astype(f32)
            be = np.copysign(np.maximum(np.abs(c2f[d]), f32(1e-6)), c2f[d]).astype(f32)
            rb = (f32(1) / be).astype(f32)
            mid, half = -al * rb, (H[d] + f32(1e-2)) / f32(s) * np.abs(rb)
            lo, hi = np.maximum(lo, mid - half), np.minimum(hi, mid + half)
        klo, khi = np.ceil(lo), np.floor(hi)
        assert np.all(k2 >= klo) and np.all(k2 <= khi)
        assert (khi - klo).max() + 1 <= t.CMAX
