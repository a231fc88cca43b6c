"""GPU tests of the images' transforms (paper_1307_5824_amd/csrc/images.hip) at the sizes where their tiling
can go wrong: every size of the one-kernel form, with more than one workgroup of images and a last one that is
not full (64, 32, 8, 2 and 1 images a workgroup at N = 8 ... 128), and the gather of N = 256 with an image's rows
over one workgroup and over many.  Expected values come from the oracle's centred DFT."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from gpu_common import rel  # noqa: E402
from oracle import blobs as oblobs  # noqa: E402
from oracle import firm as ofirm  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M", [(8, 131), (16, 33), (32, 9), (32, 17), (64, 3), (128, 1), (128, 3), (256, 1), (256, 7),
                                 (256, 2500)])
def test_every_image_size_against_the_dft(N, M):
    """White-noise images, at the tolerance of two FP32 transforms of length N (1e-5); of many images the
    first, the last and some between."""
    from paper_1307_5824_amd import firm
    print(f"images N={N} M={M}", flush=True)
    img = torch.randn((M, N, N), device="cuda", generator=torch.Generator(device="cuda").manual_seed(N + M))
    plan = firm.Plan(N, np.broadcast_to(np.eye(3), (M, 3, 3)))
    b = plan.images_to_slices(img)
    torch.cuda.synchronize()
    k1, k2 = ofirm.disk_points(N)
    pick = np.arange(k1.size)
    if N >= 128:  # some of the points, the disk's edge among them
        edge = np.flatnonzero((np.abs(k1) >= N // 2 - 1) | (np.abs(k2) >= N // 2 - 1))
        pick = np.unique(np.concatenate([edge, np.random.default_rng(N).integers(0, k1.size, 60)]))
    for m in range(M) if M <= 131 else (0, 1, M // 2, M - 1):
        got = b[m].cpu().numpy().astype(np.complex128)[pick]
        ref = oblobs.centred_dft2(img[m].cpu().numpy().astype(np.float64), k1[pick], k2[pick])
        assert rel(got, ref) < 1e-5, m
    plan.close()
