"""The any-shape kernel's greedy search (omp_group.h), modelled lane by lane on the CPU.

Signals with an exact representation of fewer than s atoms leave every correlation exactly zero; the
search has to end there, in at most two passes a step, and the codes have to be the oracle's.  The model
keeps the kernel's lane grids, blocks, scan order, merge and repeat rule; the arithmetic is numpy's, exact
for these inputs."""
import numpy as np
import pytest

import oracle

# (lanes over rows, lanes over columns, rows and columns of a lane's block): 16 lanes and 64 lanes a signal
GRIDS = [(4, 4, 2, 2), (4, 4, 4, 4), (4, 4, 3, 4), (8, 8, 2, 2), (8, 8, 4, 2), (4, 16, 3, 2)]


def hadamard(n):
    h = np.ones((1, 1))
    while len(h) < n:
        h = np.block([[h, h], [h, -h]])
    return h / np.sqrt(n)  # n = 4, 16: exact


class Signal:
    """One signal's lanes: the correlations' blocks (NaN beyond the dictionary) and its atoms so far."""

    def __init__(self, y, d1, d2, grid):
        self.grid, self.n = grid, (d1.shape[1], d2.shape[1])
        self.c = d1.T @ y @ d2
        self.masked = np.zeros(self.n, bool)
        self.atoms, self.active = [], True

    def best(self):
        """(value, code j << 8 | i) of the largest magnitude: within a lane the first of equal values in
        column order, starting from value 0 at the block's first element; lanes merge to the smaller code."""
        lr, lc, ri, cj = self.grid
        found = []
        for sc in range(lc):
            for sr in range(lr):
                bs, be = 0.0, (0, 0)
                for j in range(cj):
                    for i in range(ri):
                        a, b = sr * ri + i, sc * cj + j
                        inside = a < self.n[0] and b < self.n[1] and not self.masked[a, b]
                        v = self.c[a, b] if inside else np.nan
                        if abs(v) > abs(bs):
                            bs, be = v, (i, j)
                found.append((-abs(bs), (sc * cj + be[1]) << 8 | (sr * ri + be[0]), bs))
        _, code, bs = min(found)
        return bs, code


def search(signals, thr):
    """One step's picks of the signals of a wave and the passes it took.  A signal whose pick is one of
    its atoms has its support masked and searches again; a pick that is not above the stopping threshold
    never counts as a repeat (the signal stops on it)."""
    passes = 0
    while True:
        passes += 1
        assert passes <= 2, "the search does not end"
        picks = [s.best() for s in signals]
        again = [s.active and abs(bs) > t and code in s.atoms for s, (bs, code), t in zip(signals, picks, thr)]
        if not any(again):
            return picks, passes
        for s, rep in zip(signals, again):
            if rep:
                for code in s.atoms:
                    s.masked[code & 255, code >> 8] = True


def held(signal, l, t):
    """The code whose Gram entry lane l of a signal reads while atom t is appended, in every signal of the
    wave: the lane's own atom, atom 0 in a lane that holds none."""
    code = signal.atoms[l] if l < len(signal.atoms) else -1
    return code if l < t and code >= 0 else 0


def code_wave(Y, d1, d2, s, grid, stop_rel=1e-14):
    """Codes of the signals that share a wave (at most 64 / lanes per signal of them)."""
    n1 = d1.shape[1]
    g1, g2 = d1.T @ d1, d2.T @ d2
    sig = [Signal(y, d1, d2, grid) for y in Y]
    thr = [stop_rel * np.linalg.norm(y) for y in Y]
    for t in range(s):
        picks, _ = search(sig, thr)
        for x, (_, code) in zip(sig, picks):  # every signal's lanes read the tables while one goes on
            for c in [code] + [held(x, l, t) for l in range(grid[0] * grid[1])]:
                assert 0 <= (c & 255) < n1 and 0 <= c >> 8 < d2.shape[1], "a table read out of range"
        for x, y, (bs, code), th in zip(sig, Y, picks, thr):
            x.active = x.active and abs(bs) > th
            if not x.active:
                continue
            x.atoms.append(code)
            i, j = np.array([a & 255 for a in x.atoms]), np.array([a >> 8 for a in x.atoms])
            gram = g1[np.ix_(i, i)] * g2[np.ix_(j, j)]
            x.x = np.linalg.solve(gram, (d1.T @ y @ d2)[i, j])
            x.c = d1.T @ (y - d1[:, i] @ np.diag(x.x) @ d2[:, j].T) @ d2
        if not any(x.active for x in sig):
            break
    supp, coef = np.full((len(Y), s), -1), np.zeros((len(Y), s))
    for k, x in enumerate(sig):
        if x.atoms:
            supp[k, :len(x.atoms)] = [(a & 255) + n1 * (a >> 8) for a in x.atoms]
            coef[k, :len(x.atoms)] = x.x
    return supp, coef


def exact_signals(kind, m):
    """(dictionary, signals): one atom, atom 0 first or last, zero and flat signals, dense ones."""
    d = np.eye(m) if kind == "identity" else hadamard(m)
    X = np.zeros((9, m, m))
    X[0, 0, 0] = 4.0                             # atom 0 alone
    X[1, m - 1, m - 2] = -4.0                    # another atom alone
    X[2, m - 1, m - 2], X[2, 0, 0] = 8.0, 4.0    # atom 0 second
    X[3, 0, 0], X[3, 1, 0] = 8.0, 8.0            # a tie with atom 0
    X[5, :2, :2] = 4.0 * np.arange(1, 5).reshape(2, 2)
    X[6] = np.round(8 * np.random.default_rng(3).standard_normal((m, m))) * 4.0
    X[7, 0, 0], X[7, 0, 1] = -4.0, 2.0
    Y = d @ X @ d.T
    Y[8] = 3.0  # flat
    return d, Y


@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "%dx%d_%dx%d" % g)
@pytest.mark.parametrize("kind", ["identity", "hadamard"])
@pytest.mark.parametrize("s", [2, 3, 5])
def test_search_ends_on_exact_signals(kind, s, grid):
    d, Y = exact_signals(kind, 4)
    ns = 64 // (grid[0] * grid[1])
    so, co, _ = oracle.omp(Y, d, d, s)
    for order in (np.arange(len(Y)), np.random.default_rng(1).permutation(len(Y))):
        for k0 in range(0, len(Y), ns):
            k = order[k0:k0 + ns]
            supp, coef = code_wave(Y[k], d, d, s, grid)
            np.testing.assert_array_equal(supp, so[k])
            np.testing.assert_array_equal(coef, co[k])


@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "%dx%d_%dx%d" % g)
def test_search_ends_on_random_sparse_signals(grid):
    """Sums of up to four pixels of random integer values in random places, s = 6: every step of every
    signal ends in two passes, whether the stopping threshold is relative or zero."""
    rng = np.random.default_rng(7)
    d, Y = np.eye(5), np.zeros((60, 5, 5))
    for y in Y:
        for _ in range(rng.integers(0, 5)):
            y[tuple(rng.integers(0, 5, 2) * rng.integers(0, 2, 2))] = rng.integers(-3, 4)
    ns = 64 // (grid[0] * grid[1])
    for stop_rel in (1e-14, 0.0):
        so, co, _ = oracle.omp(Y, d, d, 6, stop_rel=stop_rel)
        for k0 in range(0, len(Y), ns):
            supp, coef = code_wave(Y[k0:k0 + ns], d, d, 6, grid, stop_rel)
            np.testing.assert_array_equal(supp, so[k0:k0 + ns])
            np.testing.assert_array_equal(coef, co[k0:k0 + ns])
