"""Coefficients held to what the arithmetic allows, signal by signal: with k the condition number of the
signal's own support Gram matrix and u the unit roundoff, |x - x_oracle| <= sqrt(s m1 m2) u k |x| (s
correlations, each a sum of m1 m2 products whose roundings add like a random walk, amplified by the
solve).  An FP32 form of the method on the CPU stays below a tenth of that."""
import numpy as np
import pytest
import torch

import oracle
from paper_2007_03800_amd import api
from tests.conftest import planted, rand_dicts
from tests.gpu_helpers import compare_codes, kron_cols
from tests.test_gpu_kernel_edges import ANY_SHAPE, ids

pytestmark = pytest.mark.gpu


def within_rounding(supp_g, coef_g, supp_o, coef_o, d1, d2, u):
    K, M = kron_cols(d1, d2), d1.shape[0] * d2.shape[0]
    seen = 0
    for sg, cg, so, co in zip(supp_g, coef_g, supp_o, coef_o):
        a = so[so >= 0]
        if len(a) == 0 or not np.array_equal(sg, so):
            continue
        kappa = np.linalg.cond(K[:, a].T @ K[:, a])
        assert np.linalg.norm(cg - co) <= np.sqrt(len(so) * M) * u * kappa * np.linalg.norm(co), (a, kappa)
        seen += 1
    return seen


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32, torch.bfloat16], ids=["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("shape", ANY_SHAPE, ids=ids)
def test_any_shape_coefficients(shape, dtype, rng):
    m1, m2, n1, n2, s = shape
    d1, d2 = rand_dicts(rng, m1, m2, n1, n2)
    Y, _ = planted(rng, 70, d1, d2, s, noise=0.05)
    Y = torch.as_tensor(Y).to(dtype).double().numpy()
    pr = api.Problem.from_math(Y, d1, d2, s, dtype=dtype)
    api.sparse_code(pr, kernel=1)
    torch.cuda.synchronize()
    so, co, _ = oracle.omp(Y, d1, d2, s, p=8)
    u = 2.0 ** -53 if dtype == torch.float64 else 2.0 ** -24
    assert within_rounding(pr.supp.cpu().numpy(), pr.coef.cpu().double().numpy(), so, co, d1, d2, u) >= 67


@pytest.mark.parametrize("pivot", [1e-3, 1.0], ids=["fp32", "fp64"])
@pytest.mark.parametrize("shape", [(12, 12, 24, 24, 12), (8, 8, 16, 16, 8), (12, 12, 20, 20, 10)], ids=ids)
def test_mixed_coefficients(shape, pivot, rng):
    """Mixed precision with the pivots in FP32 where they may be, and all through the FP64 loop; near-ties
    at the band within which candidates are re-scored (2^-6), as in the other mixed tests."""
    m1, m2, n1, n2, s = shape
    N = 611  # a last group of three
    d1, d2 = rand_dicts(rng, m1, m2, n1, n2)
    Y, _ = planted(rng, N, d1, d2, s, noise=0.03)
    Y[4] = 0.0
    Y[9] = 3.0 * np.outer(d1[:, 2], d2[:, 5])
    Y = torch.as_tensor(Y).to(torch.bfloat16).double().numpy()
    pr = api.Problem.from_math(Y, d1, d2, s, dtype=torch.bfloat16)
    api.sparse_code(pr, mixed=True, pivot_fp64=pivot)
    torch.cuda.synchronize()
    so, co, ro = oracle.omp(Y, d1, d2, s, p=8)
    sg, cg = pr.supp.cpu().numpy(), pr.coef.cpu().double().numpy()
    agree, ties, bad, err = compare_codes(Y, d1, d2, sg, cg, so, co, 2.0 ** -6)
    assert agree >= 0.97 * N and bad == 0 and err <= 1e-4, (agree, ties, bad, err)
    assert within_rounding(sg, cg, so, co, d1, d2, 2.0 ** -24) >= 0.97 * N - 1
    ok = np.all(sg == so, axis=1)
    np.testing.assert_allclose(pr.res2.cpu().double().numpy()[ok], ro[ok], rtol=2e-3, atol=1e-6)
