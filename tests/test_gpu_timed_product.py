"""GPU test of firm_apply_AtA_timed at every size of the product, among them those whose outer passes share a
launch (N <= 32): it is the product that firm_apply_AtA runs, so its result is the same bits and its durations
fit into the wall time of as many calls."""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from gpu_common import even_random_kernel, ker_to_centred, small_geometry  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [8, 16, 32, 64])
def test_timed_product_is_the_product(N):
    from paper_1307_5824_amd import firm
    rng = np.random.default_rng(N)
    R, _, _, _ = small_geometry(N, 2, N)
    plan = firm.Plan(N, R)
    plan.kernel_set(torch.as_tensor(ker_to_centred(even_random_kernel(N, rng), N)).float().cuda())
    x = torch.as_tensor(rng.standard_normal((N,) * 3)).float().cuda()
    y0, y1 = plan.apply_AtA(x, 0.3), torch.empty_like(x)
    reps = 20
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ms = plan.apply_AtA_timed(x, 0.3, reps, y1)
    wall = (time.perf_counter() - t0) * 1e3 / reps
    print(f"timed product N={N}: {np.round(np.array(ms) * 1e3, 2)} us, wall {wall * 1e3:.1f} us", flush=True)
    assert torch.equal(y0, y1)
    assert len(ms) == 5 and all(v > 0 for v in ms) and sum(ms) <= wall
    if N <= 32:  # two passes of one launch
        assert ms[0] == ms[1] and ms[3] == ms[4]
