"""The workloads this library is timed on: what a program that uses it calls, from the smallest
call to the largest, through paper_2007_03800_amd.api.

    listed()              the named cases
    draw(rng)             one more case of the same ranges
    prepare(case, seed)   the device buffers, dictionaries and networks such a program holds
    run(state)            one pass; returns every output
    work(case)            bytes and flops one pass cannot do without
    exact(case, seed)     the same outputs from plain torch in 64 bits

Kinds: "code" (2D-OMP of a set of signals), "learn" (Algorithm 1 on one problem), "uneven"
(Algorithm 1 on a batch of problems of different shapes in one call), "ortho" (Remark 1's
orthonormal variant of Algorithm 1), "tensor" (Remark 3, signals of two to four modes), "denoise"
(Sec. IV: overlapping patches, error-driven 2D-OMP, overlap average), "proposal" (learned support
proposal with 2D-OMP fallback) and "gradient" (the proposal network's training gradient).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2007_03800_amd import api

DTYPES = {"float32": torch.float32, "float64": torch.float64, "bfloat16": torch.bfloat16}

# the four problems of the uneven batch: signals m1 x m2, atoms n1 x n2, s atoms per signal and
# the signals at scale 1
UNEVEN = ((8, 8, 16, 16, 6, 200_000), (12, 12, 20, 20, 10, 100_000), (16, 16, 32, 32, 16, 50_000),
          (32, 24, 48, 36, 20, 20_000))

# the FP32 kernel that api.autotune settles on for each shape it can choose for (lanes, lanes, waves
# or signals per wave, kind), pinned here so that a run does not depend on the tuner's timing
TUNED = {(8, 8, 16, 16, 8): (1, 4, 2, 1), (8, 8, 16, 16, 6): (1, 4, 3, 1), (8, 8, 12, 12, 4): (1, 4, 4, 1),
         (12, 12, 20, 20, 10): (4, 10, 4, 2), (12, 12, 24, 24, 12): (8, 8, 4, 2), (16, 16, 32, 32, 16): (8, 8, 1, 2)}


def listed():
    return [
        # a service that codes a handful of patches per request: launches and latency
        dict(name="code_few", kind="code", dtype="float32", m1=8, m2=8, n1=16, n2=16, s=8, N=64),
        # the benchmarked problem: 100,000 8x8 patches, 256 atoms, 20 iterations
        dict(name="learn_patches", kind="learn", dtype="float32", m1=8, m2=8, n1=16, n2=16, s=8, N=100_000, K=20),
        # the default precision at the reference-parity size: a small problem learned in FP64
        dict(name="learn_fp64", kind="learn", dtype="float64", m1=8, m2=8, n1=12, n2=12, s=4, N=2_000, K=10),
        # the benchmarked shape coded in FP64
        dict(name="code_fp64", kind="code", dtype="float64", m1=8, m2=8, n1=16, n2=16, s=8, N=100_000),
        # patch and dictionary sizes nobody tuned for
        dict(name="code_ragged", kind="code", dtype="float32", m1=9, m2=7, n1=13, n2=11, s=6, N=20_011),
        # several dictionary problems of different patch sizes, learning resumed in one call
        dict(name="learn_uneven", kind="uneven", scale=1.0, K=1),
        # the largest run: a million BF16 patches, correlations on the BF16 matrix cores
        dict(name="learn_mixed", kind="learn", dtype="mixed", m1=12, m2=12, n1=24, n2=24, s=12, N=1_000_000, K=2),
        # one 512 x 512 image denoised with an overcomplete dictionary
        dict(name="denoise_512", kind="denoise", dtype="float32", H=512, W=512, n=16, sigma=20.0),
        # orthonormal dictionaries at the paper's timing size (8x8 patches, s = 8)
        dict(name="learn_ortho", kind="ortho", dtype="float32", m=8, s=8, N=128_000, K=4),
        # multispectral patches (8 x 8 pixels, 4 bands) in the tensor interface's default precision
        dict(name="learn_tensor", kind="tensor", dtype="float64", modes="8x8x4", atoms="12x12x6", s=8, N=20_000, K=1),
        # proposal network in front of 2D-OMP over a large set of patches
        dict(name="proposal_1m", kind="proposal", n=16, s=8, hidden=512, N=1_000_000),
        # one training gradient of the proposal network at the default batch
        dict(name="gradient_1024", kind="gradient", n=16, s=8, hidden=512, N=1_024),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["code", "code", "code", "learn", "learn", "uneven", "denoise", "ortho", "tensor", "tensor",
                       "proposal", "gradient"])
    if kind in ("code", "learn"):
        # half the shapes are ones the library has its own kernels for, half are arbitrary
        if rng.random() < 0.5:
            m1, m2, n1, n2, s = rng.choice([(8, 8, 16, 16, 8), (8, 8, 16, 16, 6), (8, 8, 12, 12, 4),
                                            (12, 12, 20, 20, 10), (12, 12, 24, 24, 12), (16, 16, 32, 32, 16)])
        else:
            m1, m2 = rng.randint(4, 16), rng.randint(4, 16)
            n1, n2 = m1 + rng.randint(0, 8), m2 + rng.randint(0, 8)
            s = rng.randint(2, 12)
        most = 100_000 if n1 * n2 * s <= 2_500 else 30_000
        if kind == "code":
            return dict(kind="code", dtype=rng.choice(["float32", "float64", "bfloat16"]), m1=m1, m2=m2, n1=n1, n2=n2,
                        s=s, N=_log(rng, 16, most))
        dtype = rng.choice(["float32", "float64", "mixed"])
        if dtype == "mixed":
            m1, m2, n1, n2, s = rng.choice([(8, 8, 16, 16, 8), (12, 12, 20, 20, 10), (12, 12, 24, 24, 12)])
            most = 500_000
        return dict(kind="learn", dtype=dtype, m1=m1, m2=m2, n1=n1, n2=n2, s=s, N=_log(rng, 1_000, most),
                    K=rng.randint(1, 8) if most < 500_000 else rng.randint(1, 3))
    if kind == "uneven":
        return dict(kind="uneven", scale=round(math.exp(rng.uniform(math.log(0.02), 0.0)), 4), K=1)
    if kind == "denoise":
        return dict(kind="denoise", dtype=rng.choice(["float32", "float32", "float64"]), H=rng.randint(64, 512),
                    W=rng.randint(64, 512), n=rng.choice([8, 16]), sigma=float(rng.choice([10, 20, 30])))
    if kind == "ortho":
        m = rng.choice([6, 8, 8, 12, 16])
        return dict(kind="ortho", dtype=rng.choice(["float32", "float64"]), m=m, s=rng.randint(3, 8),
                    N=_log(rng, 1_000, 128_000 if m <= 8 else 20_000), K=rng.randint(1, 6))
    if kind == "tensor":
        modes, atoms = rng.choice([("8x8x4", "12x12x6"), ("6x5x4", "9x7x5"), ("7x5x3", "10x8x4"), ("9x8", "13x12"),
                                   ("4x4x3x2", "6x5x4x3"), ("8x6x5", "10x9x7")])
        return dict(kind="tensor", dtype=rng.choice(["float32", "float64"]), modes=modes, atoms=atoms,
                    s=rng.randint(3, 8), N=_log(rng, 1_000, 20_000), K=1)
    if kind == "proposal":
        return dict(kind="proposal", n=16, s=rng.choice([6, 8]), hidden=rng.choice([256, 512]),
                    N=_log(rng, 64, 1_000_000))
    return dict(kind="gradient", n=16, s=rng.choice([6, 8]), hidden=rng.choice([256, 512]),
                N=64 * _log(rng, 1, 64))


# ------------------------------------------------------------------ inputs

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)


def _unit(g, m, n):
    """(n, m) tensor, atom i = row i: i.i.d. N(0, 1) entries scaled to unit norm."""
    d = torch.randn(n, m, generator=g, device="cuda", dtype=torch.float64)
    return (d / d.norm(dim=1, keepdim=True)).contiguous()


def _orthonormal(g, m):
    return torch.linalg.qr(torch.randn(m, m, generator=g, device="cuda", dtype=torch.float64).cpu())[0].cuda().contiguous()


def _signals(g, Ds, s, N, dtype, snr_db=30.0):
    """Planted signals (N, m_n, ..., m_1): s atoms each, uniform with N(0, 1) coefficients, plus white noise."""
    ns, ms = [D.shape[0] for D in Ds], [D.shape[1] for D in Ds]
    A, M = math.prod(ns), math.prod(ms)
    sigma = math.sqrt(s / M * 10.0 ** (-snr_db / 10.0))
    out = torch.empty((N, M), device="cuda", dtype=dtype)
    for k0 in range(0, N, 100_000):
        n = min(100_000, N - k0)
        atom = torch.randint(0, A, (n, s), generator=g, device="cuda")
        coef = torch.randn(n, s, generator=g, device="cuda", dtype=torch.float32)
        y = sigma * torch.randn(n, M, generator=g, device="cuda", dtype=torch.float32)
        for t in range(s):
            a, f = atom[:, t], coef[:, t:t + 1]
            for D in Ds:  # first mode fastest: later modes are the outer factor
                f = (D.float()[a % D.shape[0]][:, None, :] * f[:, :, None]).reshape(n, -1) if D is Ds[0] else \
                    (D.float()[a % D.shape[0]][:, :, None] * f[:, None, :]).reshape(n, -1)
                a = a // D.shape[0]
            y += f
        out[k0:k0 + n] = y.to(dtype)
    return out.reshape([N] + ms[::-1])


def _problem(g, m1, m2, n1, n2, s, N, dtype, off):
    """Planted signals and the dictionaries a call starts from: the planting ones (off = 0), ones
    near them (learning resumed, or begun from similar images; off = relative distance)."""
    true = _unit(g, m1, n1), _unit(g, m2, n2)
    Y = _signals(g, true, s, N, dtype)
    other = _unit(g, m1, n1), _unit(g, m2, n2)
    near = [D + off * E for D, E in zip(true, other)]
    return Y, tuple((D / D.norm(dim=1, keepdim=True)).contiguous() for D in near)


def _sizes(text):
    return [int(v) for v in text.split("x")]


def _image(g, H, W):
    """Grey levels in [0, 255]: a smooth background, rectangles, discs and a band of fine stripes."""
    y = torch.arange(H, device="cuda", dtype=torch.float64)[:, None].expand(H, W) / 512
    x = torch.arange(W, device="cuda", dtype=torch.float64)[None, :].expand(H, W) / 512
    u = torch.rand(400, generator=g, device="cuda", dtype=torch.float64).tolist()
    img = torch.full((H, W), 110.0, device="cuda", dtype=torch.float64)
    for k in range(3):
        img += 50 * (u[k] - 0.5) * torch.cos(2 * math.pi * ((1 + 3 * u[3 + k]) * y + (1 + 3 * u[6 + k]) * x + u[9 + k]))
    for k in range(24):
        a, b, h, w, v = u[20 + 5 * k:25 + 5 * k]
        img = torch.where((y >= a * 0.9) & (y < a * 0.9 + 0.02 + h / 4) & (x >= b * 0.9) & (x < b * 0.9 + 0.02 + w / 4),
                          30 + 200 * v, img)
    for k in range(12):
        a, b, r, v = u[150 + 4 * k:154 + 4 * k]
        img = torch.where((y - a) ** 2 + (x - b) ** 2 <= (0.01 + 0.08 * r) ** 2, 20 + 215 * v, img)
    band = (y > 0.70) & (y < 0.78)
    img = img + torch.where(band, 30 * torch.sign(torch.sin(2 * math.pi * 512 * x / 6)), 0.0)
    return img.clamp(0, 255)


def _dct(m, n):
    """(n, m): sampled cosines of unit norm (n = m: the orthonormal DCT-II basis)."""
    d = torch.cos(math.pi * (torch.arange(m, dtype=torch.float64)[None, :] + 0.5)
                  * torch.arange(n, dtype=torch.float64)[:, None] / n)
    return (d / d.norm(dim=1, keepdim=True)).cuda().contiguous()


def _params(g, M, hidden, A):
    """Flat FP32 weights of a proposal network: [W1, b1, W2, b2, W3, b3], fan-in scaled."""
    parts = []
    for rows, fan in ((hidden, M), (hidden, hidden), (A, hidden)):
        parts += [torch.randn(rows * fan, generator=g, device="cuda") * math.sqrt(2.0 / fan),
                  0.05 * torch.randn(rows, generator=g, device="cuda")]
    return torch.cat(parts).cpu().numpy()


def _inputs(case, seed):
    """Everything of a case that is made from the seed, as plain tensors (exact() starts from these too)."""
    g, kind = _gen(seed), case["kind"]
    if kind in ("code", "learn"):
        dtype = torch.bfloat16 if case["dtype"] == "mixed" else DTYPES[case["dtype"]]
        return _problem(g, case["m1"], case["m2"], case["n1"], case["n2"], case["s"], case["N"], dtype,
                        0.3 if kind == "learn" else 0.0)
    if kind == "uneven":
        return [_problem(g, *sh[:5], max(500, int(sh[5] * case["scale"])), torch.float32, 0.1) for sh in UNEVEN]
    if kind == "ortho":
        m = case["m"]
        Y = _signals(g, (_orthonormal(g, m), _orthonormal(g, m)), case["s"], case["N"], DTYPES[case["dtype"]])
        return Y, (_orthonormal(g, m), _orthonormal(g, m))
    if kind == "tensor":
        ms, ns = _sizes(case["modes"]), _sizes(case["atoms"])
        Y = _signals(g, [_unit(g, m, n) for m, n in zip(ms, ns)], case["s"], case["N"], DTYPES[case["dtype"]])
        return Y, [_unit(g, m, n) for m, n in zip(ms, ns)]
    if kind == "denoise":
        img = _image(g, case["H"], case["W"])
        noisy = img + case["sigma"] * torch.randn(img.shape, generator=g, device="cuda", dtype=torch.float64)
        return noisy.to(DTYPES[case["dtype"]]).contiguous(), (_dct(8, case["n"]), _dct(8, case["n"]))
    # proposal, gradient
    n, s = case["n"], case["s"]
    D = _unit(g, 8, n), _unit(g, 8, n)
    Y = _signals(g, D, s, case["N"], torch.float32)
    supp = torch.rand(case["N"] if kind == "gradient" else 1, n * n, generator=g, device="cuda").topk(s, dim=1)[1]
    return Y, D, _params(g, 64, case["hidden"], n * n), supp.to(torch.int32).contiguous()


def _tuned(*shapes):
    for sh in shapes:
        if sh in TUNED:
            api.set_kernel_variant(*sh, TUNED[sh])


def prepare(case, seed):
    kind, x = case["kind"], _inputs(case, seed)
    st = {"case": case}
    if kind in ("code", "learn"):
        _tuned(tuple(case[v] for v in ("m1", "m2", "n1", "n2", "s")))
    elif kind == "uneven":
        _tuned(*(sh[:5] for sh in UNEVEN))
    elif kind == "proposal":
        _tuned((8, 8, case["n"], case["n"], case["s"]))
    if kind in ("code", "learn", "ortho"):
        Y, first = x
        st["first"] = first
        st["pr"] = api.Problem(Y, first[0].clone(), first[1].clone(), case["s"])
    elif kind == "uneven":
        st["first"] = [first for _, first in x]
        st["pr"] = [api.Problem(Y, first[0].clone(), first[1].clone(), sh[4]) for (Y, first), sh in zip(x, UNEVEN)]
    elif kind == "tensor":
        Y, first = x
        st["first"] = first
        st["pr"] = api.TensorProblem(Y, [D.clone() for D in first], case["s"])
    elif kind == "denoise":
        st["noisy"], st["D"] = x
    else:
        Y, D, params, supp = x
        st["net"] = api.Proposer(8, 8, case["n"], case["n"], hidden=case["hidden"], seed=int(seed) % 1000)
        st["net"].set_params(params)
        if kind == "proposal":
            st["pr"] = api.Problem(Y, D[0], D[1], case["s"])
            st["accept"] = torch.empty(case["N"], dtype=torch.int32, device="cuda")
        else:
            st["Y"], st["supp"] = Y, supp
    return st


# ------------------------------------------------------------------ one pass

def _codes(pr):
    return {"supp": pr.supp, "coef": pr.coef, "res2": pr.res2}


def _learn(prs, firsts, **opts):
    for pr, first in zip(prs, firsts):  # every pass starts from the same dictionaries
        pr.D1.copy_(first[0])
        pr.D2.copy_(first[1])
    trace = api.learn(prs, opts.pop("K"), **opts)
    return {"trace": trace, "problems": [dict(_codes(pr), D1=pr.D1, D2=pr.D2) for pr in prs]}


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "code":
        return _codes(api.sparse_code(st["pr"])[0])
    if kind == "learn":
        return _learn([st["pr"]], [st["first"]], K=case["K"], mixed=case["dtype"] == "mixed")
    if kind == "uneven":
        return _learn(st["pr"], st["first"], K=case["K"])
    if kind == "ortho":
        return _learn([st["pr"]], [st["first"]], K=case["K"], method=1)
    if kind == "tensor":
        pr = st["pr"]
        for D, first in zip(pr.Ds, st["first"]):
            D.copy_(first)
        return dict(_codes(pr), trace=api.tensor_learn(pr, case["K"]), Ds=list(pr.Ds))
    if kind == "denoise":
        image, pr = api.denoise(st["noisy"], st["D"][0], st["D"][1], case["sigma"])
        return dict(_codes(pr), image=image)
    if kind == "proposal":
        # tau keeps part of the proposals; the rest take the 2D-OMP fallback
        pr = api.learned_sparse_code(st["net"], st["pr"], 0.8, accept=st["accept"])[0]
        return dict(_codes(pr), accept=st["accept"])
    loss, grad = st["net"].gradient(st["Y"], st["supp"], case["s"])
    return {"loss": loss, "grad": grad}


# ------------------------------------------------------------------ what a pass cannot do without

def _omp_work(ms, ns, s, N, elem_y, elem_c):
    """(bytes, flops) of one sweep: the first correlation by mode products, the Gram-form refreshes."""
    A, M, f, pre = math.prod(ns), math.prod(ms), 0.0, 1
    for d in range(len(ms)):
        f += 2.0 * pre * ns[d] * math.prod(ms[d:])
        pre *= ns[d]
    return N * (M * elem_y + s * (4 + elem_c) + elem_c), N * (f + s * (s + 1.0) * A)


def _update_flops(ms, s, N):
    return N * (2.0 * s * math.prod(ms) + 2.0 * s * s)


def work(case):
    kind = case["kind"]
    ec = 8 if case.get("dtype") == "float64" else 4
    ey = 2 if case.get("dtype") in ("bfloat16", "mixed") else ec
    if kind == "code":
        b, f = _omp_work((case["m1"], case["m2"]), (case["n1"], case["n2"]), case["s"], case["N"], ey, ec)
        return {"bytes": b, "flops": f}
    if kind == "learn":
        ms = case["m1"], case["m2"]
        b, f = _omp_work(ms, (case["n1"], case["n2"]), case["s"], case["N"], ey, ec)
        return {"bytes": b, "flops": (2 * case["K"] + 1) * f + 2 * case["K"] * _update_flops(ms, case["s"], case["N"])}
    if kind == "uneven":
        tb = tf = 0.0
        for m1, m2, n1, n2, s, n in UNEVEN:
            N = max(500, int(n * case["scale"]))
            b, f = _omp_work((m1, m2), (n1, n2), s, N, 4, 4)
            tb += b
            tf += (2 * case["K"] + 1) * f + 2 * case["K"] * _update_flops((m1, m2), s, N)
        return {"bytes": tb, "flops": tf}
    if kind == "ortho":
        m, s, N = case["m"], case["s"], case["N"]
        return {"bytes": N * (m * m * ec + s * (4 + ec) + ec),
                "flops": N * ((2 * case["K"] + 1) * 4.0 * m ** 3 + 2 * case["K"] * 2.0 * s * m)}
    if kind == "tensor":
        ms, ns = _sizes(case["modes"]), _sizes(case["atoms"])
        b, f = _omp_work(ms, ns, case["s"], case["N"], ec, ec)
        K, nm = case["K"], len(ms)
        return {"bytes": b, "flops": (nm * K + 1) * f + nm * K * _update_flops(ms, case["s"], case["N"])}
    if kind == "denoise":
        N = (case["H"] - 7) * (case["W"] - 7)
        # patches are a view of the image; the codes (cap 32) are results
        return {"bytes": 2.0 * case["H"] * case["W"] * ec + N * (32 * (4 + ec) + ec),
                "flops": N * 2.0 * (64 * case["n"] + 8 * case["n"] ** 2)}
    n, s, h, N = case["n"], case["s"], case["hidden"], case["N"]
    net = 64 * h + h * h + h * n * n
    if kind == "proposal":
        b, f = _omp_work((8, 8), (n, n), s, N, 4, 4)
        return {"bytes": b + 4.0 * N, "flops": f + 2.0 * net * N}
    return {"bytes": N * (256.0 + 4 * s) + 8.0 * (net + 2 * h + n * n), "flops": 2.0 * N * (3 * net - 64 * h)}


# ------------------------------------------------------------------ 64-bit results

def _kron(Ds):
    """(A, M): row a is atom a on the flattened signal (first mode fastest)."""
    K = Ds[0]
    for D in Ds[1:]:
        K = torch.einsum("ip,aq->iapq", D, K).reshape(D.shape[0] * K.shape[0], D.shape[1] * K.shape[1])
    return K


def _omp(Y, Ds, s, err2=0.0):
    """Textbook OMP on the explicit Kronecker dictionary, by Gram-Schmidt on the chosen atoms."""
    K = _kron(Ds)
    A, M = K.shape
    N = Y.shape[0]
    supp = torch.full((N, s), -1, dtype=torch.int64, device="cuda")
    coef = torch.zeros((N, s), dtype=torch.float64, device="cuda")
    res2 = torch.zeros(N, dtype=torch.float64, device="cuda")
    step = max(1, min(N, int(3e8) // max(s * M, 2 * A)))
    for k0 in range(0, N, step):
        y = Y[k0:k0 + step].reshape(-1, M).double()
        n = y.shape[0]
        r = y.clone()
        norm = y.norm(dim=1)
        Q = torch.zeros((n, s, M), dtype=torch.float64, device="cuda")
        R = torch.zeros((n, s, s), dtype=torch.float64, device="cuda")
        z = torch.zeros((n, s), dtype=torch.float64, device="cuda")
        sup = torch.full((n, s), -1, dtype=torch.int64, device="cuda")
        live = torch.arange(n, device="cuda")
        for t in range(s):
            rl = r[live]
            if err2 > 0:
                live = live[(rl * rl).sum(1) > err2]
                rl = r[live]
            c = (rl @ K.T).abs()
            if t:
                c.scatter_(1, sup[live, :t], -1.0)
            best, a = c.max(1)
            keep = best > 1e-14 * norm[live]
            live, a = live[keep], a[keep]
            if live.numel() == 0:
                break
            q = K[a]
            h = torch.zeros((live.numel(), s), dtype=torch.float64, device="cuda")
            for _ in range(2 if t else 0):  # twice is enough
                p = torch.matmul(Q[live, :t], q[:, :, None])[:, :, 0]
                q = q - torch.matmul(p[:, None, :], Q[live, :t])[:, 0]
                h[:, :t] += p
            nq = q.norm(dim=1)
            q = q / nq[:, None]
            h[:, t] = nq
            R[live, :, t] = h
            Q[live, t] = q
            zt = (q * r[live]).sum(1)
            z[live, t] = zt
            r[live] -= zt[:, None] * q
            sup[live, t] = a
        x = torch.zeros_like(z)
        for t in range(s - 1, -1, -1):
            v = z[:, t] - (R[:, t, t + 1:] * x[:, t + 1:]).sum(1)
            x[:, t] = torch.where(sup[:, t] >= 0, v / torch.where(R[:, t, t] > 0, R[:, t, t], 1.0), 0.0)
        supp[k0:k0 + step], coef[k0:k0 + step], res2[k0:k0 + step] = sup, x, (r * r).sum(1)
    return supp, coef, res2


def _factors(Y, Ds, supp, coef, d):
    """Sums A = sum W W^T and B = sum Y_(d) W^T of the update of mode d."""
    ns, ms = [D.shape[0] for D in Ds], [D.shape[1] for D in Ds]
    nd, md, rest = ns[d], ms[d], math.prod(ms) // ms[d]
    A = torch.zeros((nd, nd), dtype=torch.float64, device="cuda")
    B = torch.zeros((md, nd), dtype=torch.float64, device="cuda")
    N, s = supp.shape
    step = max(1, min(N, int(2e8) // (rest * (s + nd + md))))
    for k0 in range(0, N, step):
        sp = supp[k0:k0 + step]
        n = sp.shape[0]
        cf = torch.where(sp >= 0, coef[k0:k0 + step], 0.0)
        a = sp.clamp(min=0)
        f, own = cf[:, :, None], None
        for e, D in enumerate(Ds):
            i = a % ns[e]
            a = a // ns[e]
            if e == d:
                own = i
            else:
                f = (D[i][:, :, :, None] * f[:, :, None, :]).reshape(n, s, -1)
        W = torch.zeros((n, nd, rest), dtype=torch.float64, device="cuda")
        W.scatter_add_(1, own[:, :, None].expand(n, s, rest), f)
        y = Y[k0:k0 + step].double()  # (n, m_n, ..., m_1)
        y = y.movedim(len(ms) - d, 1).reshape(n, md, rest)
        W, y = W.transpose(0, 1).reshape(nd, -1), y.transpose(0, 1).reshape(md, -1)
        A += W @ W.T
        B += y @ W.T
    return A, B


def _update(Y, Ds, supp, coef, d):
    A, B = _factors(Y, Ds, supp, coef, d)
    used = torch.nonzero(torch.diagonal(A) > 0)[:, 0].cpu()
    A, B = A.cpu(), B.cpu()
    new = Ds[d].cpu().clone()
    X = torch.linalg.solve(A[used][:, used], B[:, used].T)
    new[used] = X / X.norm(dim=1, keepdim=True)
    return new.cuda()


def _polar(Y, Ds, supp, coef, d):
    U, _, V = torch.linalg.svd(_factors(Y, Ds, supp, coef, d)[1].cpu())
    return (U @ V).T.contiguous().cuda()


def _threshold(Y, Ds, s):
    """Codes for orthonormal dictionaries: the s largest correlations."""
    c = Y.reshape(Y.shape[0], -1).double() @ _kron(Ds).T
    supp = c.abs().topk(s, dim=1)[1]
    coef = c.gather(1, supp)
    return supp, coef, ((Y.double() ** 2).flatten(1).sum(1) - (coef ** 2).sum(1)).clamp(min=0)


def _iterate(Y, Ds, s, K, code, update):
    Ds, trace = list(Ds), []
    for _ in range(K):
        for d in range(len(Ds)):
            supp, coef, res2 = code(Y, Ds, s)
            if d == 0:
                trace.append(math.sqrt(float(res2.sum()) / Y.numel()))
            Ds[d] = update(Y, Ds, supp, coef, d)
    _, coef, res2 = code(Y, Ds, s)
    trace.append(math.sqrt(float(res2.sum()) / Y.numel()))
    return trace, Ds, {"supp": None, "coef": coef, "res2": res2}


def exact(case, seed):
    kind = case["kind"]
    if kind == "proposal":
        return None  # which atoms a BF16 network proposes has no 64-bit counterpart
    x = _inputs(case, seed)
    if kind == "code":
        _, coef, res2 = _omp(x[0], x[1], case["s"])
        return {"supp": None, "coef": coef, "res2": res2}
    if kind in ("learn", "uneven", "ortho"):
        many = x if kind == "uneven" else [x]
        size = [sh[4] for sh in UNEVEN] if kind == "uneven" else [case["s"]]
        how = (_threshold, _polar) if kind == "ortho" else (_omp, _update)
        if sum(Y.shape[0] * D[0].shape[0] * D[1].shape[0] * s for (Y, D), s in zip(many, size)) * case["K"] > 2e10:
            return None  # too long
        got = [_iterate(Y, D, s, case["K"], *how) for (Y, D), s in zip(many, size)]
        return {"trace": np.array([t for t, _, _ in got]),
                "problems": [dict(c, D1=D[0], D2=D[1]) for _, D, c in got]}
    if kind == "tensor":
        trace, Ds, codes = _iterate(x[0], x[1], case["s"], case["K"], _omp, _update)
        return dict(codes, trace=np.array(trace), Ds=Ds)
    if kind == "denoise":
        noisy, D = x[0].double(), x[1]
        H, W = noisy.shape
        R, C = H - 7, W - 7
        Y = noisy.unfold(0, 8, 1).unfold(1, 8, 1).reshape(R * C, 8, 8).transpose(1, 2)  # (N, m2, m1)
        supp, coef, res2 = _omp(Y.contiguous(), D, 32, err2=(1.15 * case["sigma"]) ** 2 * 64)
        est = torch.zeros((R * C, 64), dtype=torch.float64, device="cuda")
        K = _kron(D)
        for t in range(32):
            on = torch.nonzero(supp[:, t] >= 0)[:, 0]
            est[on] += coef[on, t:t + 1] * K[supp[on, t]]
        image, cover = torch.zeros_like(noisy), torch.zeros_like(noisy)
        est = est.reshape(R, C, 8, 8)  # (r, c, j, i)
        for i in range(8):
            for j in range(8):
                image[i:i + R, j:j + C] += est[:, :, j, i]
                cover[i:i + R, j:j + C] += 1
        return {"supp": None, "coef": coef, "res2": res2, "image": image / cover}
    Y, D, params, supp = x
    h, A = case["hidden"], case["n"] ** 2
    p = torch.from_numpy(params).cuda().double().requires_grad_()
    w1, b1, w2, b2, w3, b3 = p.split([64 * h, h, h * h, h, A * h, A])
    v = Y.reshape(case["N"], 64).double()
    v = v / v.norm(dim=1, keepdim=True)
    v = torch.nn.functional.gelu(v @ w1.reshape(h, 64).T + b1)
    v = torch.nn.functional.gelu(v @ w2.reshape(h, h).T + b2)
    z = v @ w3.reshape(A, h).T + b3
    label = torch.zeros_like(z).scatter_(1, supp.long(), 1.0)
    loss = torch.nn.functional.binary_cross_entropy_with_logits(z, label)
    loss.backward()
    return {"loss": float(loss.detach()), "grad": p.grad}
