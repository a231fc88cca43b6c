"""Host-side emulation of the point finder and binning of the gridding kernels
(paper_1307_5824_amd/csrc/points.h) for every tile and window width that they launch: the LDS and
bit-field budgets, the bins' footprints inside the tile, the even/odd window polynomials, and the FP32
plane, row and slab tests against every half-disk point of random views.  Runs on the CPU; no kernel
is launched."""
import math

import numpy as np
import pytest

NTH, NW, RP, CHUNK, GROUP, RUN = 1024, 16, 22, 64, 32768, 64
LDS = 160 * 1024
# (name, lattice step, bins along axis 0, bound on P1, bytes per cell, bytes per value)
KINDS = {"ker": (4, 2, 22, 8, 4), "ker8": (4, 2, 16, 8, 4), "atb": (2, 1, 16, 16, 8)}


class Tile:
    def __init__(self, kind, W):
        if kind == "ker" and W == 8:
            kind = "ker8"
        self.S, NB0, P1MAX, CELL, VAL = KINDS[kind]
        self.W = W
        self.NJ = 8 if W == 8 else 4
        self.CJ = 2 * self.NJ
        self.B = (17 - W, self.CJ + 1 - W, 9 - W)
        self.NB = (NB0, (P1MAX - W + 1) // self.B[1], (RP - W + 1) // self.B[2])
        self.T = tuple(n * b for n, b in zip(self.NB, self.B))
        self.P = tuple(t + W - 1 for t in self.T)
        self.PADLO = (W + 1) // 2 - 1
        self.nbins = math.prod(self.NB)
        STR = 28 if W <= 7 else 36
        fixed = (self.P[0] * self.P[1] * RP * CELL + NW * 16 * STR * 4 + NW * 64 * 2 + GROUP // RUN * 2 +
                 self.nbins * 4 + 64)
        per = lambda q: q * (4 + VAL) + (q // CHUNK + self.nbins) * 4  # noqa: E731
        q = 4 * NTH
        while q > NTH and fixed + per(q) > LDS:
            q -= NTH
        self.QCAP, self.lds = q, fixed + per(q)
        self.DIAG = math.isqrt(sum(t * t for t in self.T) - 1) + 1
        self.ROWS, self.CMAX = self.DIAG // self.S + 1, self.DIAG // self.S + 2


ALL = [(k, W) for k in ("ker", "atb") for W in range(4, 9)]


@pytest.mark.parametrize("kind,W", ALL)
def test_budgets_and_footprints(kind, W):
    t = Tile(kind, W)
    assert t.lds <= LDS and all(n >= 1 for n in t.NB) and t.P[2] <= RP and t.nbins <= 192
    # a chunk-table entry: bin above bit 19, start in 12 bits, count in 7; the packed scan of
    # (chunks << 16) | points
    assert t.QCAP <= 4096 and CHUNK < 128 and t.nbins < 4096
    assert t.QCAP // CHUNK + t.nbins < 32768 and t.QCAP < 65536
    assert 64 * t.CMAX <= t.QCAP  # one step of a wavefront always fits an empty queue
    # a queue entry: 15 bits of view, k1 <= N/2 <= 128 in 8, k2 + 256 in 9
    assert GROUP <= 1 << 15 and 128 < 256 and 0 <= -128 + 256 + 0 and 128 + 256 < 512
    # every bin's 16 x CJ x 8 footprint lies inside the padded tile; a start o in the bin and its W
    # weights fit the padded weight rows
    for d, foot in ((0, 16), (1, t.CJ), (2, 8)):
        assert (t.NB[d] - 1) * t.B[d] + foot <= t.P[d] if d < 2 else (t.NB[d] - 1) * t.B[d] + foot <= RP
        assert t.B[d] - 1 + W <= foot
    last = ((t.P[0] - 1) * t.P[1] + t.P[1] - 1) * RP + RP - 1
    assert last < t.P[0] * t.P[1] * RP
    # the lanes of one quarter of an 8-byte access: two rows of 8 cells in 16 distinct slots
    for n in range(t.NJ):
        slots = {((t.NJ * e + n) * RP + k) % 16 for e in range(2) for k in range(8)}
        assert len(slots) == (16 if t.NJ == 4 else 8)


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
        uc = (c @ c1f) * f32(1 / s)
        uh = (H * np.abs(c1f)).sum() * f32(1 / s) + f32(1e-3)
        first = np.ceil(uc - uh).astype(np.int64)
        assert np.all(k1 >= first) and np.all(k1 < first + t.ROWS) and np.all(k1 <= uc + uh)
        kd = np.floor(np.sqrt((N * N // 4 - k1 * k1).astype(np.float64) + 1e-9))
        lo, hi = -kd, kd.copy()
        for d in range(3):
            al = (f32(s) * k1.astype(f32) * c1f[d] - c[:, d]).astype(f32)
            be = f32(s) * c2f[d]
            h = H[d] + f32(1e-2)
            if abs(be) < 1e-6:
                assert np.all(np.abs(al) <= h)
                continue
            a, b = (-h - al) / be, (h - al) / be
            lo, hi = np.maximum(lo, np.minimum(a, b)), np.minimum(hi, np.maximum(a, b))
        klo, khi = np.ceil(lo), np.floor(hi)
        klo = np.where(k1 == 0, np.maximum(klo, 1), klo)
        assert np.all(k2 >= klo) and np.all(k2 <= khi)
        assert (khi - klo).max() + 1 <= t.CMAX
