"""CPU tests of what the gridding kernels' point finder is given and of the tables it makes
(paper_1307_5824_amd/csrc/points.h, spread.hip, project.hip): the work lists, from the library's own host code,
cover every tile that can hold a point, and every view of it once; the test of a run's box of normals keeps every
run that has a point in the tile, in the kernel's FP32 at the largest grids; the queue's sort places every
point once and its chunks cover each bin.  No kernel is launched."""
import ctypes

import numpy as np
import pytest

from test_points_index_math import ALL, GROUP, NW, RUN, Tile

f32 = np.float32


def worklist(N, W, M, kind):
    """(items, tile): the library's work list as rows (tile, first view, end view, 0)."""
    from paper_1307_5824_amd import firm
    lib = ctypes.CDLL(firm.LIB_PATH)
    vec = (ctypes.c_void_p * 3)()  # std::vector<int>: begin, end, capacity; returned through a pointer
    if kind in ("ker", "atb"):
        f = lib._Z15spread_worklistiiib
        f.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_bool]
        f(vec, N, W, M, kind == "atb")
    else:
        f = lib._Z16project_worklistiiilRb
        wide = ctypes.c_bool()
        f.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_int64,
                      ctypes.POINTER(ctypes.c_bool)]
        f(vec, N, W, M, lib.firm_slice_points(N), ctypes.byref(wide))
        kind = "prjw" if wide.value else "prj"
    n = (vec[1] - vec[0]) // 4
    items = np.ctypeslib.as_array(ctypes.cast(vec[0], ctypes.POINTER(ctypes.c_int)), (n,)).reshape(-1, 4).copy()
    return items, Tile(kind, W)


@pytest.mark.parametrize("W", [4, 5, 6, 7, 8])
@pytest.mark.parametrize("kind,N,M", [("ker", 8, 1), ("ker", 16, 20001), ("ker", 64, 9973), ("ker", 128, 300), ("atb", 8, 50001),
                                      ("atb", 32, 257), ("atb", 64, 70000), ("prj", 16, 5), ("prj", 16, 20001),
                                      ("prj", 64, 513)])
def test_work_list_covers_every_tile_and_view_once(kind, N, M, W):
    items, t = worklist(N, W, M, kind)
    L = t.S * N
    nt = [L // d + 1 for d in t.T]
    # each tile's ranges follow one another from 0 to M, on whole runs
    order = np.lexsort((items[:, 1], items[:, 0]))
    it = items[order]
    first = np.r_[True, it[1:, 0] != it[:-1, 0]]
    last = np.r_[first[1:], True]
    assert np.all(it[first, 1] == 0) and np.all(it[last, 2] == M)
    assert np.all(it[1:, 1][~first[1:]] == it[:-1, 2][~last[:-1]])
    assert np.all(it[:, 1] < it[:, 2]) and np.all(it[:, 1] % RUN == 0)
    assert it[:, 0].min() >= 0 and it[:, 0].max() < nt[0] * nt[1] * nt[2]
    # every tile with a start that a point within L/2 of the centre can have, from the finest sampling of
    # positions that the tile size can miss (steps of half a cell near the sphere's surface are the extreme ones)
    rng = np.random.default_rng(N + W)
    d = rng.standard_normal((40000, 3))
    d /= np.linalg.norm(d, axis=1)[:, None]
    r = 0.5 * L * np.r_[np.ones(20000), rng.random(20000) ** (1 / 3)]
    tau = np.clip(d * r[:, None] + 0.5 * L, 0.0, L)
    start = np.floor(tau - 0.5 * W).astype(np.int64) + 1 + t.PADLO
    tile = start // np.array(t.T)
    ids = (tile[:, 0] * nt[1] + tile[:, 1]) * nt[2] + tile[:, 2]
    assert np.isin(ids, it[:, 0]).all()
    # the order: by the expected share of views that meet the tile, heavy first, to the resolution of 2,048 classes
    nr = np.zeros(nt[0] * nt[1] * nt[2])
    np.add.at(nr, items[:, 0], 1)
    ijk = np.stack(np.unravel_index(items[:, 0], nt), 1)
    rho = np.linalg.norm((ijk + 0.5) * np.array(t.T) - 0.5 * L - (0.5 if W % 2 else 0.0), axis=1)
    rt = 0.5 * np.linalg.norm(t.T)
    work = np.minimum(1.0, rt / np.maximum(rho, 1e-9)) / nr[items[:, 0]]
    if M <= 4 * RUN:  # one range a tile
        assert np.all(work[1:] <= work[:-1] + work.max() / 2048 + 1e-12)


@pytest.mark.parametrize("kind,W", [(k, W) for k, W in ALL if k != "prjw"])
def test_box_of_normals_keeps_every_run_with_a_point(kind, W):
    """N = 256, where FP32 positions are coarsest: runs of 64 views in a small cone and one of any views; for
    every point the test of its view's run, and the view's own two tests, in FP32, with the tile of its start."""
    t = Tile(kind, W)
    N = 256
    L, s = t.S * N, t.S
    rng = np.random.default_rng(W)
    H = np.array([0.5 * v for v in t.T], dtype=f32)
    off = f32((-0.5 if W % 2 else 0.0) - 0.5 * L)
    k = np.arange(-N // 2, N // 2 + 1)
    k1, k2 = (a.ravel() for a in np.meshgrid(k, k, indexing="ij"))
    half = (4 * (k1 * k1 + k2 * k2) <= N * N) & ((k1 > 0) | ((k1 == 0) & (k2 > 0)))
    k1, k2 = k1[half], k2[half]
    for cone in (0.0, 0.02, 0.2, 3.0):
        q, _ = np.linalg.qr(rng.standard_normal((3, 3)))
        R = np.empty((RUN, 3, 3))
        for v in range(RUN):
            w = q + 0.5 * cone * rng.standard_normal((3, 3))
            R[v], _ = np.linalg.qr(w)
            R[v] *= np.sign(np.linalg.det(R[v]))
        if cone == 0.0:
            R[:] = np.eye(3)
        n = np.cross(R[:, 0], R[:, 1]).astype(f32)
        ax = np.argmax(np.abs(n), axis=1)
        n *= np.where(n[np.arange(RUN), ax] < 0, -1, 1).astype(f32)[:, None]
        lo, hi = n.min(0), n.max(0)
        lim = (H * np.maximum(np.abs(lo), np.abs(hi))).sum(dtype=f32) + f32(4e-3)
        for v in range(0, RUN, 21):
            pick = rng.integers(0, k1.size, 4000)
            a, b = k1[pick], k2[pick]
            tau = np.clip(s * (b[:, None] * R[v, 1] + a[:, None] * R[v, 0]) + 0.5 * L, 0.0, L)
            start = np.floor(tau - 0.5 * W).astype(np.int64) + 1 + t.PADLO
            c = ((start // np.array(t.T)) * np.array(t.T)).astype(f32) + H + off
            p, r = c * lo, c * hi
            dmin, dmax = np.minimum(p, r).sum(1, dtype=f32), np.maximum(p, r).sum(1, dtype=f32)
            assert np.all(dmin <= lim) and np.all(dmax >= -lim)
            c1, c2 = R[v, 0].astype(f32), R[v, 1].astype(f32)
            m = np.array([c1[1] * c2[2] - c1[2] * c2[1], c1[2] * c2[0] - c1[0] * c2[2], c1[0] * c2[1] - c1[1] * c2[0]], dtype=f32)
            assert np.all(np.abs((c * m).sum(1, dtype=f32)) <= (H * np.abs(m)).sum(dtype=f32) + f32(2e-3))
            assert np.all((c * c1).sum(1, dtype=f32) + (H * np.abs(c1)).sum(dtype=f32) >= f32(-2e-3))
            # the point's row, one of ROWS from the first
            cs = c / f32(s)
            uc = (cs * c1).sum(1, dtype=f32)
            uh = (H / f32(s) * np.abs(c1)).sum(dtype=f32) + f32(1e-3)
            row = np.ceil(uc - uh).astype(np.int64)
            assert np.all((a >= row) & (a < row + t.ROWS) & (a <= uc + uh))
            # and its k2, in the three slabs' interval
            left, right = np.full(a.size, -1e9), np.full(a.size, 1e9)
            for d in range(3):
                al = (a.astype(f32) * c1[d] - cs[:, d]).astype(f32)
                rb = f32(1) / np.copysign(max(abs(c2[d]), f32(1e-6)), c2[d]).astype(f32)
                mid, wid = -al * rb, (H[d] + f32(1e-2)) / f32(s) * abs(rb)
                left, right = np.maximum(left, mid - wid), np.minimum(right, mid + wid)
            assert np.all((b >= np.ceil(left)) & (b <= np.floor(right)))
            assert (np.floor(right) - np.ceil(left)).max() + 1 <= t.CMAX


@pytest.mark.parametrize("kind,W", ALL)
def test_queue_sort_and_chunks(kind, W):
    """The sort of a queueful as the workgroup does it: each point's bin and rank in it, the packed scan of
    (chunks << 16) | points over 64 bins at a time, the chunk table's entries, the points' places."""
    t = Tile(kind, W)
    rng = np.random.default_rng(W)
    for fill in (1, 7, t.CHUNK, t.CHUNK + 1, t.QCAP // 2, t.QCAP):
        for spread in (1, 3, t.nbins):
            bins = rng.integers(0, spread, fill) * (t.nbins - 1) // max(1, spread - 1) if spread > 1 else np.full(fill, t.nbins - 1)
            drop = rng.random(fill) < 0.1  # queued, but a point of another tile
            hist, place = np.zeros(t.nbins, np.int64), np.full(fill, -1, np.int64)
            for i in range(fill):
                if not drop[i]:
                    place[i] = bins[i] << 16 | hist[bins[i]]
                    hist[bins[i]] += 1
            base, table, at0 = 0, {}, np.zeros(t.nbins, np.int64)
            for b in range(t.nbins):  # the scan's exclusive sums, in bin order
                at, ci, rest = base & 0xffff, base >> 16, hist[b]
                at0[b] = at
                base += ((hist[b] + t.CHUNK - 1) // t.CHUNK << 16) | hist[b]
                while rest > 0:
                    e = np.int32(b << 20 | at << 7 | min(rest, t.CHUNK))
                    table[ci] = (int(e) >> 20, (int(e) >> 7) & 8191, int(e) & 127)
                    rest, at, ci = rest - t.CHUNK, at + t.CHUNK, ci + 1
            assert base < 1 << 31 and sorted(table) == list(range(base >> 16))
            assert len(table) <= t.QCAP // t.CHUNK + t.nbins
            order = np.full(fill, -1, np.int64)
            for i in np.flatnonzero(place >= 0):
                order[at0[place[i] >> 16] + (place[i] & 0xffff)] = i
            kept = np.flatnonzero(place >= 0)
            assert np.array_equal(np.sort(order[:kept.size]), kept)
            seen = []
            for b, at, cnt in table.values():
                assert 1 <= cnt <= t.CHUNK and np.all(bins[order[at:at + cnt]] == b)
                seen.extend(range(at, at + cnt))
            assert sorted(seen) == list(range(kept.size))


def test_parts_of_a_run():
    """Fewer live runs than wavefronts: a run's 64 views in 2^sh parts, each view in one of them."""
    for nlive in range(0, GROUP // RUN + 1):
        sh = 0
        while (nlive << sh) < NW and sh < 4:
            sh += 1
        assert nlive == 0 or nlive << sh >= NW
        lanes = np.arange(RUN)
        units = [(u >> sh, u & ((1 << sh) - 1)) for u in range(nlive << sh)]
        assert sorted(set(r for r, _ in units)) == list(range(nlive))
        assert np.bincount((lanes << sh) >> 6, minlength=1 << sh).tolist() == [RUN >> sh] * (1 << sh)
