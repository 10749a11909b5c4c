"""Image rebuild where one form hands over to the next: pixel by pixel up to 40 pixels a patch, rows of
patches with one value a lane up to 64, two up to 128, four up to 256, and pixel by pixel beyond.  Bars as in
the other rebuild tests (the sums have up to 256 terms of s products: 1e-12 FP64, 1e-5 FP32)."""
import numpy as np
import pytest
import torch

from oracle import denoise as oden
from paper_2007_03800_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,bar", [(torch.float64, 1e-12), (torch.float32, 1e-5)], ids=["fp64", "fp32"])
@pytest.mark.parametrize("m1,m2", [(1, 1), (5, 8), (41, 1), (7, 6), (2, 32), (13, 5), (8, 16), (3, 43), (16, 16), (1, 64)])
def test_rebuild_of_patch_sizes(m1, m2, dtype, bar, rng):
    H, W, n1, n2 = m1 + 22, m2 + 37, min(m1 + 3, 64), min(m2 + 1, 64)
    s = min(6, m1 * m2)
    d1, d2 = (rng.standard_normal(k).astype(np.float32).astype(np.float64) for k in ((m1, n1), (m2, n2)))
    N = (H - m1 + 1) * (W - m2 + 1)
    supp = rng.integers(0, n1 * n2, (N, s)).astype(np.int32)
    supp[rng.random((N, s)) < 0.4] = -1
    coef = rng.standard_normal((N, s)).astype(np.float32).astype(np.float64)
    pr = api.Problem(torch.zeros((N, m2, m1), dtype=dtype, device="cuda"), torch.as_tensor(d1.T.copy(), device="cuda"),
                     torch.as_tensor(d2.T.copy(), device="cuda"), s, supp=torch.as_tensor(supp, device="cuda"),
                     coef=torch.as_tensor(coef, dtype=dtype, device="cuda"))
    g = api.patches_to_image(pr, H, W).double().cpu().numpy()
    ref = oden.image_from_codes(supp, coef, d1, d2, H, W)
    assert np.abs(g - ref).max() <= bar * np.abs(ref).max()
