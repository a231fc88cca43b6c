"""GPU tests of the accuracy of the gridded sums over many views (paper_1307_5824_amd/csrc/spread.hip), where
rounding in their accumulation would show: small volumes with many views, whose tiles are split into many
view ranges and whose bins hold many points, on the slices of one volume, whose terms add up in phase near the
origin instead of averaging out.  Expected values are the oracle's direct sums in FP64.

The bounds are one and a half times the error of sums that take every point's term into 64-bit integers
by itself and round the grid once (N = 8 with 50,000 views, means of six seeds: Ker 2.25e-7 and A*b
1.40e-7 at W = 7, 1.03e-7 and 1.14e-7 at W = 8; N = 16 with 2,000 views 2.96e-7, 1.35e-7, 1.13e-7 and 1.11e-7).
With one FP32 add to the grid per range and cell, A*b had 3.5e-7 and 5.5e-7 at N = 8."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from gpu_common import ker_to_centred, rel, small_geometry  # noqa: E402
from oracle import direct  # noqa: E402
from oracle import firm as ofirm  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def firm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1307_5824_amd import firm as f
    return f


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy().astype(np.float64)


def some_of(n, N, rng):
    """At most n indices of an N^3 grid, the one nearest to its centre among them."""
    i = np.stack(np.meshgrid(*[np.arange(N)] * 3, indexing="ij"), -1).reshape(-1, 3)
    keep = rng.permutation(len(i))[:n]
    keep[0] = (N // 2) * (N * N + N + 1)
    return i[np.unique(keep)]


@pytest.mark.parametrize("N,M,W,ker_bound,atb_bound", [
    (8, 50000, 7, 3.4e-7, 2.1e-7), (8, 50000, 8, 1.6e-7, 1.7e-7),
    (16, 2000, 7, 4.5e-7, 2.1e-7), (16, 2000, 8, 1.7e-7, 1.7e-7)])
def test_sums_over_many_views(firm, N, M, W, ker_bound, atb_bound):
    print(f"accumulation N={N} M={M} W={W}", flush=True)
    R, sh, grp, table = small_geometry(N, M, 500 + N, 10, True)
    rng = np.random.default_rng(N)
    c, s = rng.uniform(-0.25 * N, 0.25 * N, (12, 3)), rng.uniform(0.05 * N, 0.15 * N, 12)
    b = direct.blob_slices(N, R, c, s, np.ones(12), grp, table, sh).astype(np.complex64)
    plan = firm.Plan(N, R, shifts=sh, ctf_group=grp, ctf_table=table, kb_width=W)
    plan.kernel_precompute()
    i = some_of(700, 2 * N - 1, rng)  # offsets -N + 1 .. N - 1
    ker = rel(host(plan.kernel_get())[tuple((i + 1).T)], direct.kernel_at(i - (N - 1), N, R, grp, table).real)
    i = some_of(700, N, rng)
    ref = direct.backproject_at(i - N // 2, b, N, R, grp, table, sh).real
    atb = rel(host(plan.backproject(torch.as_tensor(b).cuda()))[tuple(i.T)], ref)
    print(f"  Ker {ker:.2e}, A*b {atb:.2e}", flush=True)
    assert ker < ker_bound and atb < atb_bound
    plan.close()


def test_repeated_views_at_the_widest_window(firm):
    """Ker at W = 8 of 20 views repeated 300 times each: the terms of a bin are the same over and over, so the
    roundings of a long FP32 chain do not average out.  Bound: 1.53e-7, the mean error here of sums that take each point
    into the integers by itself, and a tenth of it (chains of 16 points 1.61e-7, of
    32 points 1.85e-7)."""
    N, errs = 16, []
    for seed in range(3):
        R, _, _, _ = small_geometry(N, 20, 800 + seed)
        plan = firm.Plan(N, np.tile(R, (300, 1, 1)), kb_width=8)
        plan.kernel_precompute()
        errs.append(rel(host(plan.kernel_get()), ker_to_centred(300 * ofirm.kernel_direct(N, R).real, N)))
        plan.close()
    print(f"repeated views: {errs}", flush=True)
    assert np.mean(errs) < 1.69e-7
