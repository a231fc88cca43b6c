"""GPU tests of the gridding's point finder (paper_1307_5824_amd/csrc/points.h) by the number of views.

Few: a gather with fewer live runs of 64 views than wavefronts (16) hands each run out in parts; counts on both
sides of a run's end and up to 16 runs, every slice against the oracle's direct sum.  Many: a workgroup walks
its views in groups of 32,768; the sums over 70,000 views (three groups) must equal those of three plans that
hold one group each, and the slices those of the same views there."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from gpu_common import rel, small_geometry  # noqa: E402
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
    return t.detach().cpu().numpy()


@pytest.mark.parametrize("W", [4, 7, 8])
@pytest.mark.parametrize("N,M", [(8, 2), (16, 5), (16, 63), (16, 65), (16, 200), (8, 1023), (8, 1025), (32, 33)])
def test_few_views(firm, N, M, W):
    """Bound: FP32 operators (1e-5) plus twenty times the window's aliasing at oversampling 2,
    exp(-pi W sqrt(1/2)) per axis."""
    print(f"few views N={N} M={M} W={W}", flush=True)
    R, sh, grp, table = small_geometry(N, M, 600 + M, 3, True)
    V = np.random.default_rng(M).standard_normal((N, N, N)).astype(np.float32)
    plan = firm.Plan(N, R, shifts=sh, ctf_group=grp, ctf_table=table, kb_width=W)
    got = host(plan.forward_project(torch.as_tensor(V).cuda()))
    ref = ofirm.forward_project(V, R, ofirm.ctf_weights(N, M, grp, table)) * ofirm.shift_phase(N, sh).conj()
    assert rel(got, ref) < 1e-5 + 20 * np.exp(-np.pi * W * np.sqrt(0.5))
    plan.close()


def test_groups_of_views(firm):
    """Against plans of one group each: 2e-6 for the sums (both carry FP32 rounding of a few 1e-7), and the same
    for the slices; sampled slices on both sides of the groups' ends too."""
    N, M, G = 16, 70000, 30000
    print(f"groups N={N} M={M}", flush=True)
    R, sh, grp, table = small_geometry(N, M, 700, 3, True)
    V = torch.as_tensor(np.random.default_rng(7).standard_normal((N, N, N)).astype(np.float32)).cuda()
    g = torch.Generator(device="cuda").manual_seed(8)
    b = torch.randn((M, ofirm.slice_point_count(N)), dtype=torch.complex64, device="cuda", generator=g)

    def run(sel):
        plan = firm.Plan(N, R[sel], shifts=sh[sel], ctf_group=grp[sel], ctf_table=table)
        plan.kernel_precompute()
        out = (host(plan.kernel_get()).astype(np.float64), host(plan.backproject(b[sel])).astype(np.float64),
               host(plan.forward_project(V)))
        plan.close()
        return out

    ker, atb, slices = run(slice(0, M))
    parts = [run(slice(a, min(M, a + G))) for a in range(0, M, G)]
    assert rel(ker, sum(p[0] for p in parts)) < 2e-6
    assert rel(atb, sum(p[1] for p in parts)) < 2e-6
    ref = np.concatenate([p[2] for p in parts])
    worst = np.max(np.linalg.norm(slices - ref, axis=1) / np.linalg.norm(ref, axis=1))
    print(f"  worst slice {worst:.2e}", flush=True)
    assert worst < 2e-6
    some = np.array([0, 29999, 30000, 32767, 32768, 65535, 65536, M - 1])
    want = ofirm.forward_project(V.cpu().numpy(), R[some], ofirm.ctf_weights(N, M, grp, table)[some])
    assert rel(slices[some], want * ofirm.shift_phase(N, sh[some]).conj()) < 1e-5
