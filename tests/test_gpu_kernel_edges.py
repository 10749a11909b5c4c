"""Kernels at the sizes where a tile, a lane grid, a chunk or a launch rule begins or ends, each
against the oracle, or exactly against the same work done another way.

Bars as in the other parity tests: FP64 supports identical except classified near-ties (1e-9),
coefficients and dictionaries 1e-10; FP32 near-ties at 1e-4; any-shape coefficients
10 u kappa / COEF_FLOOR (u the unit roundoff, kappa the largest condition number of a support's Gram
matrix, 10 about the square root of the sums' length), at least 1e-10 and 1e-4; BF16 network within 2e-2 of the largest logit and 5e-2 (relative norm) of each gradient block.  Where two routes do the
same arithmetic the results must be equal bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from oracle import denoise as oden
from oracle import mlp
from oracle import tensor as ot
from paper_2007_03800_amd import api, synth
from tests.conftest import planted, rand_dicts
from tests.gpu_helpers import COEF_FLOOR, compare_codes, kron_all, kron_cols
from tests.test_gpu_learned import weights
from tests.test_gpu_tensor import planted as planted_tensor
from tests.test_gpu_tensor import unit_cols

pytestmark = pytest.mark.gpu
DEV = "cuda"
ids = lambda x: "x".join(map(str, x)) if isinstance(x, tuple) else str(x)  # noqa: E731


# ---- any-shape coding: blocks of the 4 x 4 and 8 x 8 lane grids (full, one over, one short), supports
# of 8, 9, 16, 17 and 32 (unrolled lengths), a narrow dictionary against a wide one

ANY_SHAPE = [(8, 8, 8, 8, 8), (8, 8, 9, 8, 9), (10, 10, 16, 16, 16), (10, 10, 17, 24, 16), (10, 12, 24, 24, 17),
             (7, 9, 25, 8, 5), (3, 40, 4, 64, 16), (16, 8, 64, 33, 20), (8, 24, 33, 64, 32)]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32, torch.bfloat16], ids=["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("shape", ANY_SHAPE, ids=ids)
def test_any_shape_coding(shape, dtype, rng):
    m1, m2, n1, n2, s = shape
    N = 70  # whole groups of four signals per wave and a rest of two
    d1, d2 = rand_dicts(rng, m1, m2, n1, n2)
    Y, _ = planted(rng, N, d1, d2, s, noise=0.05)
    Y = torch.as_tensor(Y).to(dtype).double().numpy()  # the values the kernel reads
    pr = api.Problem.from_math(Y, d1, d2, s, dtype=dtype)
    api.sparse_code(pr, kernel=1)
    torch.cuda.synchronize()
    so, co, ro = oracle.omp(Y, d1, d2, s, p=8)
    K = kron_cols(d1, d2)
    kappa = max(np.linalg.cond(K[:, a].T @ K[:, a]) for a in (r[r >= 0] for r in so))
    band, tol = (1e-9, max(1e-10, 10 * 2.0 ** -53 * kappa / COEF_FLOOR)) if dtype == torch.float64 else \
        (1e-4, max(1e-4, 10 * 2.0 ** -24 * kappa / COEF_FLOOR))
    sg, cg, rg = pr.supp.cpu().numpy(), pr.coef.cpu().double().numpy(), pr.res2.cpu().double().numpy()
    agree, ties, bad, err = compare_codes(Y, d1, d2, sg, cg, so, co, band)
    assert bad == 0 and ties <= 3 and err <= tol, (agree, ties, bad, err, tol)
    ok = np.all(sg == so, axis=1)
    yy = np.sum(Y ** 2, axis=(1, 2))
    assert np.max(np.abs(rg[ok] - ro[ok]) / yy[ok]) <= (1e-12 if dtype == torch.float64 else 1e-5)


# ---- n-dimensional FP64 problems: splits onto the 4 x 16 grid's edges and the other grids, and the
# update sums of every mode (one and two 16-row tiles)

@pytest.mark.parametrize("ms,ns,s", [((6, 6, 2), (12, 16, 6), 4), ((4, 4, 4), (16, 8, 8), 4),
                                     ((3, 4, 6), (13, 5, 13), 4), ((2, 9, 2, 2), (3, 17, 4, 2), 3)], ids=ids)
def test_tensor_splits_and_sums(ms, ns, s, rng):
    T = [unit_cols(rng, m, n) for m, n in zip(ms, ns)]
    Y = planted_tensor(rng, 67, T, s, 0.05)
    pr = api.TensorProblem.from_math(Y, T, s, dtype=torch.float64)
    api.tensor_sparse_code(pr)
    torch.cuda.synchronize()
    sg, cg = pr.supp.cpu().numpy(), pr.coef.cpu().numpy()
    so, co, _ = ot.tensor_omp(Y, T, s)
    agree, ties, bad, err = compare_codes(Y, None, None, sg, cg, so, co, 1e-9, K=kron_all(T))
    assert bad == 0 and ties <= 1 and err <= 1e-10
    for mode in range(1, len(ms) + 1):
        q = api.TensorProblem.from_math(Y, T, s, dtype=torch.float64)
        q.supp.copy_(pr.supp)
        q.coef.copy_(pr.coef)
        api.tensor_update(q, mode)
        Dn, _, _ = ot.tensor_update(mode, Y, T, sg, cg)
        for g, o in zip(q.dicts(), Dn):
            assert np.abs(g - o).max() <= 1e-10 * np.abs(o).max()


# ---- the network: one fused kernel up to 512 hidden units (one to four column tiles a wave), layer by
# layer above; 64-signal tiles with a remainder

@pytest.mark.parametrize("H,N", [(64, 1), (128, 63), (192, 65), (448, 64), (512, 129), (576, 129)])
def test_bf16_logits(H, N, rng):
    p = weights(rng, H)
    Y = rng.standard_normal((N, 8, 8))
    net = api.Proposer(8, 8, 16, 16, hidden=H)
    net.set_params(p)
    Yd = torch.from_numpy(np.ascontiguousarray(Y.transpose(0, 2, 1))).float().cuda()
    z = net.logits(Yd).cpu().numpy()
    zref, _ = mlp.forward(p.astype(np.float64), mlp.inputs(Y), 64, H, 256)
    assert np.max(np.abs(z - zref)) <= 2e-2 * np.max(np.abs(zref))


# ---- training gradients: 64 x 64 tiles with the weight gradients split over the batch (one split, a
# last split that is shorter), and above 8192 rows the large-tile kernel

@pytest.mark.parametrize("B,H", [(64, 64), (192, 320), (576, 128), (8256, 64)])
def test_bf16_gradient(B, H, rng):
    p = weights(rng, H)
    Y = rng.standard_normal((B, 8, 8))
    supp = np.argsort(rng.random((B, 256)), axis=1)[:, :8].astype(np.int32)
    net = api.Proposer(8, 8, 16, 16, hidden=H)
    net.set_params(p)
    Yd = torch.from_numpy(np.ascontiguousarray(Y.transpose(0, 2, 1))).float().cuda()
    loss, g = net.gradient(Yd, torch.from_numpy(supp).cuda(), 8)
    lref, gref = mlp.loss_and_grad(p.astype(np.float64), mlp.inputs(Y), mlp.labels(supp, 256), 64, H, 256)
    assert abs(loss - lref) <= 1e-2 * abs(lref)
    off, _ = mlp.layout(64, H, 256)
    for b in range(6):
        gb, rb = g[off[b]:off[b + 1]], gref[off[b]:off[b + 1]]
        assert np.linalg.norm(gb - rb) <= 5e-2 * np.linalg.norm(rb), b


# ---- proposals: the factor has one row per lane; both support lengths that have a fallback kernel, and a
# last wave with one signal

@pytest.mark.parametrize("s", [6, 8])
def test_proposal_least_squares(s, rng):
    p = weights(rng, 64)
    d1, d2 = rand_dicts(rng, 8, 8, 16, 16)
    Y, _ = planted(rng, 65, d1, d2, s, noise=0.05)
    net = api.Proposer(8, 8, 16, 16, hidden=64, fp32_check=True)
    net.set_params(p)
    pr = api.Problem.from_math(Y, d1, d2, s, dtype=torch.float32)
    acc = torch.zeros(65, dtype=torch.int32, device=DEV)
    api.learned_sparse_code(net, pr, tau=1e30, accept=acc)
    torch.cuda.synchronize()
    z = net.logits(pr.Y).cpu().numpy()
    sg = pr.supp.cpu().numpy()
    ok = acc.cpu().numpy() == 1  # (a support whose atoms are dependent is not accepted)
    assert ok.mean() >= 0.9
    np.testing.assert_array_equal(sg[ok], mlp.top_s(z, s)[ok])
    cref, rref = mlp.least_squares_on_support(Y, d1, d2, sg)
    assert np.max(np.abs(pr.coef.cpu().double().numpy() - cref)[ok]) <= 1e-3 * np.max(np.abs(cref))
    np.testing.assert_allclose(pr.res2.cpu().double().numpy()[ok], rref[ok], rtol=1e-2, atol=1e-5)


def test_rejected_signals_listed_over_many_blocks():
    """More than 1024 blocks of signals: the list of rejected ones (a scan of the blocks' counts) sends
    exactly those to 2D-OMP, so every signal has either the all-accepted or the all-rejected result."""
    N = 1024 * 256 + 77
    torch.manual_seed(5)
    w = synth.WORKLOADS["fp32_8x8_n16_s8"]
    d1, d2 = synth.true_dictionaries(w)
    Y = torch.randn(N, 8, 8, device=DEV)  # ABI layout
    D1, D2 = (torch.as_tensor(d.T.copy(), device=DEV) for d in (d1, d2))
    net = api.Proposer(8, 8, 16, 16, hidden=64)
    got, acc = [], torch.empty(N, dtype=torch.int32, device=DEV)
    pr = api.Problem(Y, D1, D2, 8)
    api.learned_sparse_code(net, pr, tau=1e30)
    torch.cuda.synchronize()
    tau = float((pr.res2 / (Y * Y).sum((1, 2))).double().median())
    for t in (1e30, 0.0, tau):
        q = api.Problem(Y, D1, D2, 8)
        api.learned_sparse_code(net, q, tau=t, accept=acc)
        torch.cuda.synchronize()
        got.append((q.supp, q.coef, q.res2))
    yes = acc == 1
    assert 0.4 <= yes.double().mean().item() <= 0.6
    for all_in, all_out, mixed in zip(*got):
        want = torch.where(yes.view(-1, *([1] * (mixed.dim() - 1))), all_in, all_out)
        assert torch.equal(mixed, want)


# ---- image rebuild: rows of patches (one value a lane up to 64 pixels, four up to 256) against the
# pixel-by-pixel kernel beyond; images of one patch, one row or column of patches, several column tiles

@pytest.mark.parametrize("dtype,bar", [(torch.float64, 1e-12), (torch.float32, 1e-5)], ids=["fp64", "fp32"])
@pytest.mark.parametrize("H,W,m1,m2", [(8, 8, 8, 8), (8, 300, 8, 8), (150, 9, 8, 8), (33, 70, 13, 5),
                                       (16, 16, 16, 16), (18, 140, 16, 16), (40, 35, 17, 16)])
def test_rebuild_edges(H, W, m1, m2, dtype, bar, rng):
    n1, n2, s = m1 + 2, m2 + 1, 5
    d1, d2 = rng.standard_normal((m1, n1)), rng.standard_normal((m2, n2))
    N = (H - m1 + 1) * (W - m2 + 1)
    supp = rng.integers(0, n1 * n2, (N, s)).astype(np.int32)
    supp[rng.random((N, s)) < 0.3] = -1
    coef = rng.standard_normal((N, s)).astype(np.float32).astype(np.float64)
    pr = api.Problem(torch.zeros((N, m2, m1), dtype=dtype, device=DEV), torch.as_tensor(d1.T.copy(), device=DEV),
                     torch.as_tensor(d2.T.copy(), device=DEV), s, supp=torch.as_tensor(supp, device=DEV),
                     coef=torch.as_tensor(coef, dtype=dtype, device=DEV))
    g = api.patches_to_image(pr, H, W).double().cpu().numpy()
    if dtype == torch.float32:
        d1, d2 = d1.astype(np.float32).astype(np.float64), d2.astype(np.float32).astype(np.float64)
    ref = oden.image_from_codes(supp, coef, d1, d2, H, W)
    assert np.abs(g - ref).max() <= bar * np.abs(ref).max()


# ---- one launch prepares up to eight dictionaries of a call

def test_more_problems_than_one_preparation_launch(rng):
    shapes = [(8, 8, 16, 16, 4), (1, 5, 1, 3, 1), (64, 2, 64, 3, 4), (3, 4, 5, 6, 2), (12, 12, 20, 20, 6), (2, 2, 2, 2, 1)]
    data = [(rng.standard_normal((9, m1, m2)), *rand_dicts(rng, m1, m2, n1, n2), s) for m1, m2, n1, n2, s in shapes]
    one = [api.Problem.from_math(*d, dtype=torch.float64) for d in data]
    api.sparse_code(one)
    for d, together in zip(data, one):
        alone = api.Problem.from_math(*d, dtype=torch.float64)
        api.sparse_code(alone)
        torch.cuda.synchronize()
        assert torch.equal(together.supp, alone.supp) and torch.equal(together.coef, alone.coef)
        so, co, _ = oracle.omp(*d)
        assert compare_codes(d[0], d[1], d[2], alone.supp.cpu().numpy(), alone.coef.cpu().numpy(), so, co, 1e-9)[2] == 0


# ---- residual sums: fewer signals than one workgroup, a rest, several workgroups

@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("N", [1, 255, 1025, 70001])
def test_rmse_of_a_coding_sweep(N, dtype, rng):
    d1, d2 = rand_dicts(rng, 4, 4, 6, 6)
    pr = api.Problem.from_math(rng.standard_normal((N, 4, 4)), d1, d2, 3, dtype=dtype)
    for _ in range(2):  # the counters are left as they were found
        trace = api.learn(pr, 0)[0]
        want = np.sqrt(pr.res2.double().sum().item() / (N * 16))
        assert trace.shape == (1,) and abs(trace[0] - want) <= 1e-12 * want


# ---- long supports, one wave per signal: each wave codes several signals of different lengths, and the
# factor keeps nothing of the one before

def test_long_supports_of_one_wave(rng):
    w = synth.WORKLOADS["fp32_8x8_n16_s8"]
    d1, d2 = synth.true_dictionaries(w)
    N = 40_000
    Y = synth.signals(w, 0, N)
    Y[::7] *= 0.02     # below the threshold at once
    Y[3::7] = rng.standard_normal(Y[3::7].shape)  # up to the cap
    err2 = (1.15 * w.sigma() * 8) ** 2
    whole = api.Problem.from_math(Y, d1, d2, 32, dtype=torch.float32)
    api.sparse_code(whole, err2=err2)
    torch.cuda.synchronize()
    nnz = (whole.supp >= 0).sum(1)
    assert nnz.min() == 0 and nnz.max() == 32
    for k0 in range(0, N, 4096):
        part = api.Problem.from_math(Y[k0:k0 + 4096], d1, d2, 32, dtype=torch.float32)
        api.sparse_code(part, err2=err2)
        torch.cuda.synchronize()
        for f in ("supp", "coef", "res2"):
            assert torch.equal(getattr(whole, f)[k0:k0 + 4096], getattr(part, f)), (k0, f)


# ---- orthonormal codes: equal magnitudes (smaller atom first), zeros chosen after every nonzero entry

def test_ortho_exact_ties(rng):
    Y = rng.integers(-2, 3, (333, 8, 8)).astype(np.float64)
    Y[5] = 0.0
    Y[6] = -1.0
    Y[7, :, :] = 0.0
    Y[7, 3, 2] = -7.0
    eye = np.eye(8)
    pr = api.Problem.from_math(Y, eye, eye, 8, dtype=torch.float32)
    api.sparse_code(pr, method=1)
    torch.cuda.synchronize()
    so, co, _ = oracle.ortho_code(Y, eye, eye, 8)
    np.testing.assert_array_equal(pr.supp.cpu().numpy(), so)
    np.testing.assert_array_equal(pr.coef.cpu().double().numpy(), co)


# ---- mixed precision: every pivot through the FP64 loop, and signals that stop early or are zero

@pytest.mark.parametrize("shape", [(12, 12, 24, 24, 12), (8, 8, 16, 16, 8), (12, 12, 20, 20, 10)], ids=ids)
def test_mixed_fp64_pivots(shape, rng):
    m1, m2, n1, n2, s = shape
    d1, d2 = rand_dicts(rng, m1, m2, n1, n2)
    Y, _ = planted(rng, 131, d1, d2, s, noise=0.03)
    Y[4] = 0.0
    Y[9] = 3.0 * np.outer(d1[:, 2], d2[:, 5])
    Y = torch.as_tensor(Y).to(torch.bfloat16).double().numpy()
    pr = [api.Problem.from_math(Y, d1, d2, s, dtype=torch.bfloat16) for _ in range(2)]
    st = api.new_stats()
    api.sparse_code(pr[0], mixed=True, pivot_fp64=1.0, stats=st)
    api.sparse_code(pr[1], mixed=True)
    torch.cuda.synchronize()
    so, co, _ = oracle.omp(Y, d1, d2, s, p=8)
    for p in pr:
        sg, cg = p.supp.cpu().numpy(), p.coef.cpu().double().numpy()
        assert np.all(sg[4] == -1) and np.all(cg[4] == 0) and sg[9, 0] == 2 + n1 * 5
        agree, ties, bad, err = compare_codes(Y, d1, d2, sg, cg, so, co, 1e-4)
        print(shape, agree, ties, bad, err)
    rows = int((pr[0].supp >= 0).sum()) - 130
    assert st.fp64_pivots >= 0.95 * rows
    # the two pivots differ by FP32 rounding alone: supports part only at near-ties
    a, b = pr[0].supp.cpu().numpy(), pr[1].supp.cpu().numpy()
    assert np.all(a == b, axis=1).mean() >= 0.97


# ---- problems of one learning call on streams of their own: more of them than streams, an empty one,
# and two that write the same dictionary (in order, as without streams)

@pytest.mark.parametrize("shared", [False, True])
def test_learn_side_by_side_equals_in_order(shared, rng):
    data = []
    for q in range(11):
        m1, m2 = 4 + q % 3, 5
        d1, d2 = rand_dicts(rng, m1, m2, m1 + 2, 7)
        data.append((planted(rng, 0 if q == 4 else 150 + 40 * q, d1, d2, 3, noise=0.05)[0], d1, d2, 3))
    outs = []
    for use_graph in (0, 1):
        probs = [api.Problem.from_math(*d, dtype=torch.float64) for d in data]
        if shared:
            probs[3].D1 = probs[0].D1  # both are 4 x 6
        traces = api.learn(probs, 3, use_graph=use_graph)
        torch.cuda.synchronize()
        outs.append((traces, [(p.d1(), p.d2(), p.supp.cpu().numpy(), p.coef.cpu().numpy()) for p in probs]))
    np.testing.assert_array_equal(outs[0][0], outs[1][0])
    for a, b in zip(outs[0][1], outs[1][1]):
        for u, v in zip(a, b):
            np.testing.assert_array_equal(u, v)


# ---- Procrustes updates: sizes around the eight-lane form and the largest, B from well conditioned
# (Newton's iteration) to beyond what it takes (Jacobi rotations).  B differs by rounding, 1e-15 n of its
# norm, which moves the polar factor by up to the condition number times that: ten times as much is allowed

@pytest.mark.parametrize("power", [0, 3, 8])
@pytest.mark.parametrize("m1,m2", [(1, 2), (7, 8), (9, 16), (17, 15), (31, 8), (8, 32)])
def test_procrustes_sizes(m1, m2, power, rng):
    N, s = 400, min(3, m1 * m2)
    d1, d2 = (np.linalg.qr(rng.standard_normal((m, m)))[0] for m in (m1, m2))
    t1, t2 = (np.linalg.qr(rng.standard_normal((m, m)))[0] for m in (m1, m2))
    supp = np.argsort(rng.random((N, m1 * m2)), axis=1)[:, :s].astype(np.int32)
    i, j = supp % m1, supp // m1
    # energies of the atoms spread over 10^-power on each side, so B's singular values are too
    coef = rng.choice([-1.0, 1.0], (N, s)) * 10.0 ** (-power / 2 * (i / max(1, m1 - 1) + j / max(1, m2 - 1)))
    X = oracle.densify(supp, coef, m1, m2)
    Y = np.einsum("pi,kij,qj->kpq", t1, X, t2)
    for side in (1, 2):
        pr = api.Problem.from_math(Y, d1, d2, s, dtype=torch.float64)
        pr.supp.copy_(torch.from_numpy(supp))
        pr.coef.copy_(torch.from_numpy(coef))
        api.tmod_update(pr, sides=side, method=1)
        torch.cuda.synchronize()
        e = oracle.procrustes_update(side, Y, d1, d2, supp, coef)[side - 1]
        B = sum(y @ d2 @ x.T if side == 1 else y.T @ d1 @ x for y, x in zip(Y, X))
        g, kappa = (pr.d1(), pr.d2())[side - 1], np.linalg.cond(B)
        print(m1, m2, side, "cond %.1e, diff %.1e" % (kappa, np.abs(g - e).max()))
        assert np.abs(g - e).max() <= 1e-14 * len(B) * kappa
        np.testing.assert_allclose(g.T @ g, np.eye(len(B)), atol=1e-12)
