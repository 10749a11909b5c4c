"""Signals that fewer than s atoms represent exactly, atom (0, 0) among them: after the last of these
atoms every correlation is exactly zero, and the any-shape kernel stops the signal there, beside
ordinary signals in the same wave.  tests/test_group_search.py shows on the CPU that the search ends.

All inputs are dyadic and the dictionaries exactly orthonormal, so supports and coefficients of these
signals are the oracle's exactly, in every precision; the ordinary signals are held to the bars of the
other parity tests (near-ties 1e-9 FP64, 1e-4 FP32 and BF16; coefficients 1e-10 and 1e-4: the dictionaries
are orthonormal, so nothing amplifies rounding)."""
import numpy as np
import pytest
import torch

import oracle
from oracle import tensor as ot
from paper_2007_03800_amd import api
from tests.gpu_helpers import compare_codes, kron_all
from tests.test_group_search import exact_signals, hadamard

pytestmark = pytest.mark.gpu
DTYPES = pytest.mark.parametrize("dtype", [torch.float64, torch.float32, torch.bfloat16], ids=["fp64", "fp32", "bf16"])


def batch(kind, m, dtype):
    """Exact signals at every place of a four-signal wave, ordinary ones between: (dictionary, Y, exact)."""
    d, E = exact_signals(kind, m)
    rng = np.random.default_rng(11)
    Y = rng.standard_normal((67, m, m))
    Y = torch.as_tensor(Y).to(dtype).double().numpy()
    exact = np.zeros(len(Y), bool)
    for k, at in enumerate(rng.permutation(60)[:4 * len(E)]):
        Y[at], exact[at] = E[k % len(E)], True
    Y[60:], exact[60:] = E[:7], True  # a wave of exact signals only and a last one that is not full
    return d, Y, exact


def check(pr, Y, d, s, exact, dtype):
    so, co, ro = oracle.omp(Y, d, d, s)
    sg, cg = pr.supp.cpu().numpy(), pr.coef.cpu().double().numpy()
    np.testing.assert_array_equal(sg[exact], so[exact])
    np.testing.assert_array_equal(cg[exact], co[exact])
    np.testing.assert_array_equal(pr.res2.cpu().double().numpy()[exact], ro[exact])
    band, tol = (1e-9, 1e-10) if dtype == torch.float64 else (1e-4, 1e-4)
    agree, ties, bad, err = compare_codes(Y, d, d, sg, cg, so, co, band)
    assert bad == 0 and ties <= 1 and err <= tol, (agree, ties, bad, err)
    return so


# 16 lanes a signal (blocks of 1, 2 and 4 rows in use), then 64 (supports beyond 16 atoms, wide dictionaries)
@DTYPES
@pytest.mark.parametrize("kind,m,s", [("identity", 4, 3), ("hadamard", 4, 3), ("identity", 9, 6), ("hadamard", 16, 8),
                                      ("identity", 8, 17), ("hadamard", 16, 20), ("identity", 30, 4)])
def test_exact_signals_stop(kind, m, s, dtype):
    d, Y, exact = batch(kind, m, dtype)
    pr = api.Problem.from_math(Y, d, d, s, dtype=dtype)
    st = api.new_stats()
    api.sparse_code(pr, kernel=1, stats=st)
    torch.cuda.synchronize()
    so = check(pr, Y, d, s, exact, dtype)
    assert st.early_stops == int((so[:, -1] < 0).sum())


@pytest.mark.parametrize("kind", ["identity", "hadamard"])
def test_exact_signals_every_call(kind):
    """The default path of FP64, the sums call and one learning iteration."""
    d, Y, exact = batch(kind, 4, torch.float64)
    s = 3
    pr = api.Problem.from_math(Y, d, d, s, dtype=torch.float64)
    api.sparse_code(pr)
    torch.cuda.synchronize()
    check(pr, Y, d, s, exact, torch.float64)
    A, B, r = api.split_sums(api.sparse_code_sums(pr, 1), 1, pr)
    so, co, ro = oracle.omp(Y, d, d, s)
    Ao, Bo = oracle.tmod_sums(1, Y, d, d, so, co)
    assert np.abs(A - Ao).max() <= 1e-10 * np.abs(Ao).max() and np.abs(B - Bo).max() <= 1e-10 * np.abs(Bo).max()
    assert abs(r - ro.sum()) <= 1e-10 * ro.sum()
    ref = oracle.learn(Y, d, d, s, 1)
    trace = api.learn(pr, 1)[0]
    np.testing.assert_allclose(trace, ref["rmse"], rtol=1e-8)
    assert np.abs(pr.d1() - ref["D1"]).max() <= 1e-8 and np.abs(pr.d2() - ref["D2"]).max() <= 1e-8


# three modes in FP64: Kronecker factors on the 16-lane, the 8 x 8 and the 4 x 16 lane grids
@pytest.mark.parametrize("kind,ms,s", [("identity", (4, 4, 4), 3), ("hadamard", (4, 4, 4), 3), ("identity", (8, 8, 8), 3),
                                       ("identity", (3, 5, 4), 17)])
def test_exact_tensors_stop(kind, ms, s):
    T = [np.eye(m) if kind == "identity" else hadamard(m) for m in ms]
    rng = np.random.default_rng(5)
    X = np.zeros((41, *ms))
    for k in range(0, 41, 2):  # up to two atoms, atom 0 in most of them; ordinary tensors between
        X[k].flat[rng.integers(0, X[k].size)] = 8.0 * (k % 4)
        X[k, 0, 0, 0] = -8.0 * (k % 3)
    Y = np.einsum("ai,bj,cl,kijl->kabc", *T, X)
    Y[1::2] = rng.standard_normal(Y[1::2].shape)
    pr = api.TensorProblem.from_math(Y, T, s, dtype=torch.float64)
    api.tensor_sparse_code(pr)
    torch.cuda.synchronize()
    so, co, _ = ot.tensor_omp(Y, T, s)
    sg, cg = pr.supp.cpu().numpy(), pr.coef.cpu().numpy()
    np.testing.assert_array_equal(sg[::2], so[::2])
    np.testing.assert_array_equal(cg[::2], co[::2])
    agree, ties, bad, err = compare_codes(Y, None, None, sg, cg, so, co, 1e-9, K=kron_all(T))
    assert bad == 0 and ties <= 1 and err <= 1e-10


# ---- atoms that hold NaN (the first of each dictionary): never chosen, and the residuals of signals with
# fewer than s atoms, or none, stay those of a dictionary with zeros in their place
@DTYPES
@pytest.mark.parametrize("m,s", [(4, 3), (9, 6), (8, 17)])
def test_nan_atoms_leave_residuals_alone(m, s, dtype):
    d, Y, _ = batch("identity", m, dtype)
    z1, z2 = d.copy(), d.copy()
    z1[:, 0], z2[:, 0] = 0.0, 0.0
    n1, n2 = d.copy(), d.copy()
    n1[0, 0], n2[1, 0] = np.nan, np.nan
    pr = api.Problem.from_math(Y, n1, n2, s, dtype=dtype)
    api.sparse_code(pr, kernel=1)
    torch.cuda.synchronize()
    so, co, ro = oracle.omp(Y, z1, z2, s)
    np.testing.assert_array_equal(pr.supp.cpu().numpy(), so)
    np.testing.assert_array_equal(pr.coef.cpu().double().numpy(), co)
    np.testing.assert_allclose(pr.res2.cpu().double().numpy(), ro, rtol=1e-12 if dtype == torch.float64 else 1e-5)
    assert (so[:, -1] < 0).any() and (so[:, 0] < 0).any()
