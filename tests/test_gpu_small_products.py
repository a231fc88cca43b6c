"""GPU test of the product's slab kernels (paper_1307_5824_amd/csrc/fft.hip, k_apply_slab): the sizes
N <= 32 that they take and the first one that they do not, against the circulant product in FP64."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lam", [0.0, 0.3])
@pytest.mark.parametrize("N", [8, 16, 32, 64])
def test_product_against_fp64_circulant(N, lam):
    """The FP32 product's two 3D transforms have 6 log2(2N) butterfly levels, each of relative error
    about 2^-24 (FP32 rounding of sums, products and twiddles), growing as the square root: at most
    42 levels, 6.5 x 2^-24 = 3.9e-7; the spectrum itself comes from one such transform.  Twice that."""
    from paper_1307_5824_amd import firm

    rng = np.random.default_rng(N)
    half = rng.standard_normal((2 * N,) * 3)
    half[0] = half[:, 0] = half[:, :, 0] = 0.0
    K = half.copy()
    K[1:, 1:, 1:] += half[1:, 1:, 1:][::-1, ::-1, ::-1]  # even about its centre (N, N, N)
    K = K.astype(np.float32)
    x = rng.standard_normal((N,) * 3).astype(np.float32)
    plan = firm.Plan(N, np.eye(3)[None], lambda_relative=0)
    plan.kernel_set(torch.from_numpy(K).cuda())
    lam_abs = lam * float(np.abs(K).max())
    y = plan.apply_AtA(torch.from_numpy(x).cuda(), lam_abs).cpu().numpy()
    S = np.fft.rfftn(np.fft.ifftshift(K.astype(np.float64)))
    want = np.fft.irfftn(S * np.fft.rfftn(x.astype(np.float64), s=(2 * N,) * 3), s=(2 * N,) * 3)[:N, :N, :N]
    want = want + lam_abs * x
    err = np.linalg.norm(y - want) / np.linalg.norm(want)
    print(f"N={N} lam={lam}: {err:.2e}", flush=True)
    assert err < 8e-7
