"""GPU tests of the gridding spreads on the matrix units (paper_1307_5824_amd/csrc/points.h, spread.hip)
where their tiling can go wrong: every window width (each has its own bins), view counts around a
run (64) and a work range (256), more points in one tile than its queue holds, and values that are
not finite.  Expected values come from the oracle's direct sums."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from gpu_common import ker_to_centred, rel, small_geometry  # noqa: E402
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


def tol(W):
    """FP32 operators (1e-5) plus the aliasing of a Kaiser-Bessel window at oversampling 2, about
    exp(-pi W sqrt(1/2)) per axis, with a factor of 20."""
    return 1e-5 + 20 * np.exp(-np.pi * W * np.sqrt(0.5))


@pytest.mark.parametrize("W", [4, 5, 6, 7, 8])
@pytest.mark.parametrize("N,M", [(8, 1), (16, 65), (16, 257)])
def test_spreads_at_every_width(firm, W, N, M):
    print(f"spread W={W} N={N} M={M}", flush=True)
    R, sh, grp, table = small_geometry(N, M, 300 + W, 3, True)
    h = ofirm.ctf_weights(N, M, grp, table)
    plan = firm.Plan(N, R, shifts=sh, ctf_group=grp, ctf_table=table, kb_width=W)
    plan.kernel_precompute()
    assert rel(host(plan.kernel_get()), ker_to_centred(ofirm.kernel_direct(N, R, h), N)) < tol(W)
    rng = np.random.default_rng(W)
    P = ofirm.slice_point_count(N)
    b = (rng.standard_normal((M, P)) + 1j * rng.standard_normal((M, P))).astype(np.complex64)
    ref = ofirm.back_project(ofirm.recentre(b, N, sh), N, R, h).real
    assert rel(host(plan.backproject(torch.as_tensor(b).cuda())), ref) < tol(W)
    plan.close()


def test_many_points_per_tile(firm):
    """N = 8 with 6,000 views: the tiles hold many queuefuls of points, in few bins."""
    N, M = 8, 6000
    R, sh, grp, table = small_geometry(N, M, 71, 2, True)
    h = ofirm.ctf_weights(N, M, grp, table)
    plan = firm.Plan(N, R, shifts=sh, ctf_group=grp, ctf_table=table)
    plan.kernel_precompute()
    assert rel(host(plan.kernel_get()), ker_to_centred(ofirm.kernel_direct(N, R, h), N)) < 1e-5
    P = ofirm.slice_point_count(N)
    rng = np.random.default_rng(5)
    b = (rng.standard_normal((M, P)) + 1j * rng.standard_normal((M, P))).astype(np.complex64)
    ref = ofirm.back_project(ofirm.recentre(b, N, sh), N, R, h).real
    assert rel(host(plan.backproject(torch.as_tensor(b).cuda())), ref) < 1e-5
    plan.close()


@pytest.mark.parametrize("W", [4, 5, 6, 7, 8])
@pytest.mark.parametrize("N,M", [(32, 3), (8, 2500)])
def test_projector_with_few_and_many_points_per_tile(firm, W, N, M):
    """The forward projector's two tile shapes: a few points per tile, and queuefuls of them."""
    print(f"project W={W} N={N} M={M}", flush=True)
    R, sh, grp, table = small_geometry(N, M, 400 + W, 3, True)
    V = np.random.default_rng(W).standard_normal((N, N, N)).astype(np.float32)
    plan = firm.Plan(N, R, shifts=sh, ctf_group=grp, ctf_table=table, kb_width=W)
    got = plan.forward_project(torch.as_tensor(V).cuda())
    torch.cuda.synchronize()
    got = got.cpu().numpy()
    some = np.unique(np.linspace(0, M - 1, 12).astype(int))  # the oracle on some of the views
    ref = ofirm.forward_project(V, R[some], ofirm.ctf_weights(N, M, grp, table)[some]) * ofirm.shift_phase(N, sh[some]).conj()
    assert rel(got[some], ref) < tol(W)
    plan.close()


def test_a_point_that_is_not_a_number_touches_no_other(firm):
    """A NaN sample drops its own point (the pair k, -k), as the integer conversion always did."""
    N, M = 16, 40
    R, sh, grp, table = small_geometry(N, M, 72, 2, True)
    P = ofirm.slice_point_count(N)
    rng = np.random.default_rng(6)
    b = (rng.standard_normal((M, P)) + 1j * rng.standard_normal((M, P))).astype(np.complex64)
    k = P // 2 + 17
    bad = b.copy()
    bad[3, k] = np.nan
    zero = b.copy()
    zero[3, k] = zero[3, P - 1 - k] = 0
    plan = firm.Plan(N, R, shifts=sh, ctf_group=grp, ctf_table=table)
    got, ref = (host(plan.backproject(torch.as_tensor(v).cuda())) for v in (bad, zero))
    assert np.isfinite(got).all() and rel(got, ref) < 1e-6
    plan.close()
