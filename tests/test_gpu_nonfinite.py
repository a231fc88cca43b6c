"""GPU test of an infinite sample in the back-projection: the data's fixed-point unit follows the largest
component, so no other point keeps a digit beside an infinity, and the result must say so instead of looking
like a volume.  The next call on the same plan is not touched by it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from gpu_common import rel, small_geometry  # noqa: E402
from oracle import firm as ofirm  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M", [(16, 40), (16, 600), (64, 3)])
@pytest.mark.parametrize("bad", [np.inf, -np.inf])
def test_an_infinite_sample_leaves_no_finite_voxel(N, M, bad):
    """40 and 3 views add up in the FP32 grid, 600 in the integer one."""
    from paper_1307_5824_amd import firm
    print(f"infinite sample N={N} M={M} {bad}", flush=True)
    R, sh, grp, table = small_geometry(N, M, 73, 2, True)
    P = ofirm.slice_point_count(N)
    rng = np.random.default_rng(6)
    b = (rng.standard_normal((M, P)) + 1j * rng.standard_normal((M, P))).astype(np.complex64)
    plan = firm.Plan(N, R, shifts=sh, ctf_group=grp, ctf_table=table)
    clean = plan.backproject(torch.as_tensor(b).cuda()).cpu().numpy()
    # a point whose CTF is not zero
    q = np.add(*(k.astype(np.int64) ** 2 for k in ofirm.disk_points(N)))
    k = P // 2 + 1 + int(np.argmax(np.abs(table[grp[1], q[P // 2 + 1:]])))
    broken = b.copy()
    broken[1, k] = bad
    got = plan.backproject(torch.as_tensor(broken).cuda()).cpu().numpy()
    assert not np.isfinite(got).any()
    again = plan.backproject(torch.as_tensor(b).cuda()).cpu().numpy()
    assert np.isfinite(again).all() and rel(again, clean) < 1e-6
    plan.close()
