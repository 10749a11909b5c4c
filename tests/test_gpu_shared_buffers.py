"""Problems of one call that share memory: the results are those of the problems one after the other,
bit for bit (the same kernels on the same values)."""
import numpy as np
import pytest
import torch

from paper_2007_03800_amd import api
from tests.conftest import planted, rand_dicts

pytestmark = pytest.mark.gpu


def results(probs):
    torch.cuda.synchronize()
    return [t.cpu().numpy() for p in probs for t in (p.D1, p.D2, p.supp, p.coef, p.res2)]


def equal(a, b):
    for u, v in zip(a, b):
        np.testing.assert_array_equal(u, v)


# ---- an update of several problems: each one sees the dictionaries as the problems before it left them

@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("sides", [1, 2, 3])
@pytest.mark.parametrize("share", ["D1", "D2", "both", "part"])
def test_update_of_problems_that_share_a_dictionary(share, sides, dtype, rng):
    m1, m2, n1, n2, s = 5, 4, 7, 6, 3
    dicts = [rand_dicts(rng, m1, m2, n1, n2) for _ in range(3)]
    data = [planted(rng, 200 + 30 * q, *dicts[q], s, noise=0.1)[0] for q in range(3)]

    def problems():
        out = [api.Problem.from_math(Y, *d, s, dtype=dtype) for Y, d in zip(data, dicts)]
        api.sparse_code(out)  # codes at each problem's own dictionaries
        if share == "part":   # problem 1's D2 begins one atom into problem 0's
            whole = torch.cat([out[0].D2, out[0].D2[:1]])
            out[0].D2, out[1].D2 = whole[:n2], whole[1:]
        for q in (1, 2):
            if share in ("D1", "both"):
                out[q].D1 = out[0].D1
            if share in ("D2", "both"):
                out[q].D2 = out[0].D2
        return out

    together, alone = problems(), problems()
    api.tmod_update(together, sides=sides)
    for p in alone:
        api.tmod_update(p, sides=sides)
    equal(results(together), results(alone))


# ---- learning side by side: problems of which one writes what another reads or writes run in order, also
# where their buffers begin at different addresses

@pytest.mark.parametrize("K", [1, 3])
@pytest.mark.parametrize("share", ["dictionaries", "codes and signals", "residuals and signals"])
def test_learning_with_overlapping_buffers(share, K, rng):
    m1, m2, n1, n2, s = 4, 5, 6, 7, 3
    data = []
    for q in range(5):
        d1, d2 = rand_dicts(rng, m1, m2, n1, n2)
        data.append((planted(rng, 120 + 40 * q, d1, d2, s, noise=0.05)[0], d1, d2, s))
    outs = []
    for use_graph in (0, 1):
        probs = [api.Problem.from_math(*d, dtype=torch.float64) for d in data]
        a, b = probs[0], probs[3]
        if share == "dictionaries":  # one atom further in the same buffer
            whole = torch.cat([a.D1, a.D1[:1]])
            a.D1, b.D1 = whole[:n1], whole[1:]
        else:  # the first signals of problem 0 are what problem 3 writes, shifted by one element
            Y = torch.cat([a.Y.flatten(), a.Y.flatten()[:8]])
            if share == "codes and signals":
                b.coef = Y[1:1 + b.N * s].view(b.N, s)
            else:
                b.res2 = Y[1:1 + b.N]
            a.Y = Y[:a.Y.numel()].view(a.Y.shape)
        traces = api.learn(probs, K, use_graph=use_graph)
        outs.append([traces] + results(probs))
    equal(*outs)


# ---- more problems than internal streams, on the caller's own stream: results as in order on the default one,
# and complete for work queued on the caller's stream afterwards

def test_learning_side_by_side_on_a_stream(rng):
    data = []
    for q in range(7):
        d1, d2 = rand_dicts(rng, 8, 8, 16, 16)
        data.append((planted(rng, 300 + 500 * (q % 3), d1, d2, 8, noise=0.05)[0], d1, d2, 8))
    outs = []
    for use_graph, stream in ((0, torch.cuda.current_stream()), (1, torch.cuda.Stream())):
        probs = [api.Problem.from_math(*d, dtype=torch.float32) for d in data]
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            traces = [api.learn(probs, 3, use_graph=use_graph) for _ in range(2)]
            copies = [p.coef.clone() for p in probs]
        outs.append(traces + results(probs) + [c.cpu().numpy() for c in copies])
    equal(*outs)


# ---- n modes that share a dictionary buffer: in FP64 every mode works with its own copy, made at the start of the
# call and renewed by its own updates, so codes and trace are those of modes with buffers of their own

@pytest.mark.parametrize("ms,ns,shared", [((4, 4, 4), (6, 6, 6), (0, 2)), ((4, 4, 4), (6, 6, 6), (1, 2)),
                                          ((4, 4, 3), (6, 6, 5), (0, 1)), ((3, 4, 4, 2), (4, 5, 5, 3), (1, 2))])
def test_tensor_modes_that_share_a_dictionary(ms, ns, shared, rng):
    T = [rng.standard_normal((m, n)) for m, n in zip(ms, ns)]
    T = [d / np.linalg.norm(d, axis=0) for d in T]
    T[shared[1]] = T[shared[0]]
    Y = rng.standard_normal((400, *ms))
    outs = []
    for same in (False, True):
        pr = api.TensorProblem.from_math(Y, T, 4, dtype=torch.float64)
        if same:
            pr.Ds[shared[1]] = pr.Ds[shared[0]]
        trace = api.tensor_learn(pr, 2)
        torch.cuda.synchronize()
        outs.append([trace] + [t.cpu().numpy() for t in (pr.supp, pr.coef, pr.res2)])
    equal(*outs)
