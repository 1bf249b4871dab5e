"""Measured cases of the band bidiagonalization library, through its Python entry points.

Kinds of case (key "kind"):

  band     one reduction of an m x n matrix to band form with a plan the program keeps.  The reduction works in
           place, so a pass starts from a fresh copy of the input.
  call     the same through the one-line call ``band(A, nb, plan=plan)``, which copies, allocates and checks the
           status as an interactive user's program does.
  batch    many uneven matrices in one launch, tile size and tree chosen per size class by the library's tuner.
  train    forward and backward of loss = sum(W * B) over the band through ``band_autograd``.
  apply    the explicit thin Q and P of a finished reduction, from its reflector records.
  ge2val   singular values of a matrix in one call (band reduction, band to bidiagonal, bisection).
  bandval  singular values of a band matrix (band to bidiagonal, bisection).

Everything is FP64, the library's data type.  "gaussian" inputs have iid N(0,1) entries; "graded" ones are
U diag(s) V^T with s geometric from 1 to "smin" and dense orthogonal U and V.
"""
import math
import random

import numpy as np
import torch

import paper_1611_06892_amd as bb


def listed():
    return [
        # The smallest call: a few tiles, where launches and hand-offs count.
        dict(name="call_192x128_nb32", kind="call", m=192, n=128, nb=32, tree="greedy", variant="bidiag",
             input="gaussian"),
        # The small square of the tests and the paper's validation sizes: 8 x 8 tiles along the flat tree.
        dict(name="call_512_nb64_flatts", kind="call", m=512, n=512, nb=64, tree="flatts", variant="bidiag",
             input="gaussian"),
        # An ordinary rectangular matrix whose sizes are no multiples of the tile.
        dict(name="band_3001x1777_nb128", kind="band", m=3001, n=1777, nb=128, tree="auto", variant="rbidiag",
             input="gaussian"),
        # More columns than rows: reduced as its transpose, in its own storage.
        dict(name="band_1500x4100_nb128", kind="band", m=1500, n=4100, nb=128, tree="greedy", variant="bidiag",
             input="gaussian"),
        # The tall matrix of the benchmark (a least-squares or PCA shape), graded spectrum.
        dict(name="band_tall_32768x2048", kind="band", m=32768, n=2048, nb=128, tree="greedy",
             variant="rbidiag", input="graded", smin=1e-8),
        # The benchmark's headline: the large square, condition number 1e6.
        dict(name="band_square_16384_nb256", kind="band", m=16384, n=16384, nb=256, tree="auto",
             variant="bidiag", input="graded", smin=1e-6),
        # The benchmark's batch: thousands of uneven matrices in one launch.
        dict(name="batch_4096", kind="batch", count=4096, mlo=64, mhi=1024, nlo=32, shapes=5),
        # A step of a program that learns through the band form (the benchmark's differentiated workload).
        dict(name="train_8192x1024_nb128", kind="train", m=8192, n=1024, nb=128, tree="greedy",
             variant="rbidiag"),
        # Explicit Q and P of a ragged tall reduction.
        dict(name="apply_6000x1500_nb128", kind="apply", m=6000, n=1500, nb=128, tree="greedy",
             variant="rbidiag"),
        # Singular values of an ordinary tall matrix, one call.
        dict(name="ge2val_3000x2000_nb64", kind="ge2val", m=3000, n=2000, nb=64, tree="auto",
             variant="rbidiag", input="graded", smin=1e-6),
        # ... and of a large square one with the wide band that suits the band reduction.
        dict(name="ge2val_8192_nb256", kind="ge2val", m=8192, n=8192, nb=256, tree="auto", variant="bidiag",
             input="graded", smin=1e-6),
        # The two steps after the band alone, at the benchmark's size.
        dict(name="bandval_16384_nb128", kind="bandval", n=16384, nb=128),
    ]


def _log_size(rng, lo, hi):
    """A size between lo and hi, even over its logarithm, of any residue."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["band", "band", "band", "call", "batch", "train", "apply", "ge2val", "bandval"])
    tree, variant = rng.choice(["greedy", "auto", "auto", "flatts"]), rng.choice(["bidiag", "rbidiag"])
    if kind == "call":
        n = _log_size(rng, 40, 700)
        return dict(kind=kind, m=_log_size(rng, n, 3 * n), n=n, nb=rng.choice([32, 64]), tree=tree, variant=variant,
                    input="gaussian")
    if kind == "band":
        nb = rng.choice([64, 128, 128, 256])
        n = _log_size(rng, 2 * nb, 40 * nb)
        m = _log_size(rng, n, min(12 * n, 32768))
        if rng.random() < 0.25:
            m, n = n, m
        data = rng.choice([dict(input="gaussian"), dict(input="graded", smin=1e-6)])
        return dict(kind=kind, m=m, n=n, nb=nb, tree=tree, variant=variant, **data)
    if kind == "batch":
        mhi = _log_size(rng, 128, 1024)
        return dict(kind=kind, count=_log_size(rng, 8, 2048), mlo=64, mhi=mhi, nlo=32, shapes=rng.randrange(1 << 20))
    if kind in ("train", "apply"):
        n = _log_size(rng, 100, 2000)
        return dict(kind=kind, m=_log_size(rng, 2 * n, 12 * n), n=n, nb=rng.choice([64, 128]), tree=tree,
                    variant=variant)
    if kind == "ge2val":
        n = _log_size(rng, 200, 5000)
        return dict(kind=kind, m=_log_size(rng, n, 4 * n), n=n, nb=rng.choice([32, 64, 128, 256]), tree=tree,
                    variant=variant, input="graded", smin=rng.choice([1e-3, 1e-6, 1e-8]))
    return dict(kind=kind, n=_log_size(rng, 100, 9000), nb=rng.choice([16, 32, 64, 100, 128, 256]))


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _gaussian(m, n, gen):
    return torch.randn(m, n, generator=gen, device="cuda", dtype=torch.float64)


def _mix_rows(X, gen):
    """An orthogonal map of X's rows: random signs, then the orthonormal cosine transform (DCT-II)."""
    n = X.shape[0]
    sign = torch.randint(0, 2, (n, 1), generator=gen, device="cuda", dtype=torch.float64) * 2 - 1
    X = X * sign
    F = torch.fft.fft(torch.cat([X[::2], X[1::2].flip(0)]), dim=0)
    w = torch.polar(torch.full((n, 1), math.sqrt(2.0 / n), device="cuda", dtype=torch.float64),
                    -math.pi * torch.arange(n, device="cuda", dtype=torch.float64).view(n, 1) / (2 * n))
    w[0] *= math.sqrt(0.5)
    return (F * w).real


def _sigmas(n, smin):
    return torch.logspace(0.0, math.log10(smin), n, device="cuda", dtype=torch.float64)


def _graded(m, n, smin, gen):
    k = min(m, n)
    A = torch.zeros(m, n, device="cuda", dtype=torch.float64)
    A.diagonal().copy_(_sigmas(k, smin))
    for _ in range(2):
        A = _mix_rows(A, gen)
        A = _mix_rows(A.t(), gen).t()
    return A


def _matrix(case, seed):
    gen = _generator(seed)
    if case.get("input") == "graded":
        return _graded(case["m"], case["n"], case["smin"], gen)
    return _gaussian(case["m"], case["n"], gen)


def _column_major(A):
    """Storage of A by columns: a contiguous (n, m) tensor."""
    return A.t().contiguous()


def _shapes(case):
    """The batch's shapes: m, then n <= m, uniform."""
    r = np.random.default_rng(case["shapes"])
    out = []
    for _ in range(case["count"]):
        m = int(r.integers(case["mlo"], case["mhi"] + 1))
        out.append((m, int(r.integers(case["nlo"], m + 1))))
    return out


def _band_storage(n, nb, seed):
    """Column-major storage of an n x n upper band with N(0,1) entries and a dominant diagonal growing to
    sqrt(n), the scale at which a reduction leaves it."""
    gen = _generator(seed)
    S = torch.zeros(n, n, device="cuda", dtype=torch.float64)     # S[j, i] = B(i, j)
    for k in range(min(nb, n - 1) + 1):
        S.diagonal(-k).copy_(torch.randn(n - k, generator=gen, device="cuda", dtype=torch.float64))
    i = torch.arange(1, n + 1, device="cuda", dtype=torch.float64)
    S.diagonal().copy_(torch.sqrt(i) + 0.1 * S.diagonal())
    return S


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind == "call":
        st["A"] = _matrix(case, seed)
        st["plan"] = bb.Plan(case["m"], case["n"], case["nb"], case["tree"], case["variant"])
    elif kind == "band":
        st["S0"] = _column_major(_matrix(case, seed))
        st["S"] = torch.empty_like(st["S0"])
        st["plan"] = bb.Plan(case["m"], case["n"], case["nb"], case["tree"], case["variant"])
        st["vt"], st["ws"] = st["plan"].alloc()
    elif kind == "batch":
        shapes = _shapes(case)
        sizes = np.array([m * n for m, n in shapes], dtype=np.int64)
        offs = np.concatenate([[0], np.cumsum(sizes)])
        gen = _generator(seed)
        st["buf0"] = torch.randn(int(offs[-1]), generator=gen, device="cuda", dtype=torch.float64)
        st["buf"] = torch.empty_like(st["buf0"])
        st["ptrs"] = torch.from_numpy(st["buf"].data_ptr() + 8 * offs[:-1]).cuda()
        st["ldas"] = torch.tensor([m for m, _ in shapes], dtype=torch.int64).cuda()
        st["plan"] = bb.BatchPlan(shapes)
        st["vt"], st["ws"] = st["plan"].alloc()
    elif kind == "train":
        n, nb = case["n"], case["nb"]
        gen = _generator(seed)
        st["A"] = _gaussian(case["m"], n, gen).requires_grad_(True)
        W = _gaussian(n, n, gen)
        st["W"] = torch.triu(W) - torch.triu(W, nb + 1)
    elif kind == "apply":
        m, n, nb = case["m"], case["n"], case["nb"]
        S = _column_major(_gaussian(m, n, _generator(seed)))
        plan = bb.Plan(m, n, nb, case["tree"], case["variant"])
        vt, ws = plan.alloc()
        plan.execute(S, m, vt, ws)
        st.update(plan=plan, vt=vt, Q=torch.empty(n, m, device="cuda", dtype=torch.float64),
                  P=torch.empty(n, n, device="cuda", dtype=torch.float64))
        size = max(plan.apply_workspace(side, False, n) for side in (0, 1))
        st["ws"] = torch.empty(size, device="cuda", dtype=torch.uint8)
    elif kind == "ge2val":
        st["A"] = _matrix(case, seed)
    else:
        st["S"] = _band_storage(case["n"], case["nb"], seed)
        st["ws"] = torch.empty(bb.bnd2bd_workspace(case["n"], case["nb"]), device="cuda", dtype=torch.uint8)
    return st


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "call":
        B, _, _ = bb.band(state["A"], case["nb"], plan=state["plan"])
        return B
    if kind == "band":
        S = state["S"]
        S.copy_(state["S0"])
        state["plan"].execute(S, case["m"], state["vt"], state["ws"])
        return S.t()
    if kind == "batch":
        state["buf"].copy_(state["buf0"])
        state["plan"].execute(state["ptrs"], state["ldas"], state["vt"], state["ws"])
        return state["buf"]
    if kind == "train":
        A = state["A"]
        A.grad = None
        B = bb.band_autograd(A, case["nb"], case["tree"], case["variant"])
        (B[:case["n"]] * state["W"]).sum().backward()
        return {"B": B.detach(), "grad": A.grad}
    if kind == "apply":
        Q, P, n = state["Q"], state["P"], case["n"]
        Q.zero_().diagonal().fill_(1.0)
        P.zero_().diagonal().fill_(1.0)
        state["plan"].apply_q(Q, case["m"], n, state["vt"], ws=state["ws"])
        state["plan"].apply_p(P, n, n, state["vt"], ws=state["ws"])
        return {"Q": Q.t(), "P": P.t()}
    if kind == "ge2val":
        return bb.ge2val_oneshot(state["A"], case["nb"], case["tree"], case["variant"])
    d, e = bb.bnd2bd(state["S"], case["n"], case["n"], case["nb"], ws=state["ws"])
    return bb.bd2val(d, e)


def _band_flops(m, n, variant):
    m, n = max(m, n), min(m, n)
    direct = 4.0 * n * n * (m - n / 3.0)
    return direct if variant == "bidiag" else 2.0 * n * n * (m + n)


def work(case):
    """Bytes: inputs once, outputs once.  Flops: the reductions' published counts, 8 n^2 nb for the chase of a
    band (two reflectors per nb columns of each of n sweeps) and 4 n^2 a bit for the bisection's counts."""
    kind = case["kind"]
    if kind == "batch":
        shapes = _shapes(case)
        flops = 0.0
        for m, n in shapes:
            flops += min(_band_flops(m, n, "bidiag"), _band_flops(m, n, "rbidiag"))
        return {"bytes": 16.0 * sum(m * n for m, n in shapes), "flops": flops}
    n, nb = case["n"], case["nb"]
    if kind == "bandval":
        return {"bytes": 8.0 * (n * (nb + 1) + n), "flops": 8.0 * n * n * nb + 4.0 * 52 * n * n}
    m, variant = case["m"], case["variant"] if "variant" in case else "bidiag"
    if kind in ("band", "call"):
        return {"bytes": 16.0 * m * n, "flops": _band_flops(m, n, variant)}
    if kind == "train":
        return {"bytes": 8.0 * (3 * m * n + n * (nb + 1)),
                "flops": _band_flops(m, n, variant) + 4.0 * n * n * (m - n / 2.0) + 2.0 * n ** 3}
    if kind == "apply":
        return {"bytes": 8.0 * (2 * m * n + 2 * n * n), "flops": 4.0 * n * n * (m - n / 2.0) + 2.0 * n ** 3}
    k = min(m, n)
    return {"bytes": 8.0 * (m * n + k), "flops": _band_flops(m, n, variant) + 8.0 * k * k * nb + 4.0 * 52 * k * k}


def _eliminations(tree, u):
    """The step's eliminations (row, pivot) and whether each row is triangularized first, for the flat tree of
    square tiles and the binomial tree."""
    if tree == "flatts":
        return [(i, 0) for i in range(1, u)], False
    out, s = [], 1
    while s < u:
        out += [(i, i - s) for i in range(s, u, 2 * s)]
        s *= 2
    return out, True


def _tile_step(M, rows, cols, tree):
    """QR of the tile rows `rows` on the tile column `cols`, applied to everything right of it (M in place)."""
    def factor(idx):
        Q, _ = torch.linalg.qr(M[idx][:, cols[0]:cols[1]], mode="complete")
        M[idx, cols[0]:] = Q.t() @ M[idx, cols[0]:]
    elim, each = _eliminations(tree, len(rows))
    for r in (rows if each else rows[:1]):
        factor(torch.arange(*r))
    for i, p in elim:
        top = torch.arange(*rows[p])[: cols[1] - cols[0]]
        # the triangle's zeros stay zero: only its own rows and those of the eliminated tile take part
        below = torch.arange(*rows[i])
        factor(torch.cat([top, below]))
    return M


def _exact_band(A, nb, tree):
    """The band form by whole tile factorizations (LAPACK's QR of each tile or stacked pair), BiDiag order."""
    M = A.clone()
    m, n = M.shape
    tiles = lambda size, lo: [(a, min(a + nb, size)) for a in range(lo, size, nb)]  # noqa: E731
    for k in range(0, n, nb):
        _tile_step(M, tiles(m, k), (k, min(k + nb, n)), tree)
        if k + nb < n:
            Mt = M.t().contiguous()
            _tile_step(Mt, tiles(n, k + nb), (k, min(k + nb, m)), tree)
            M = Mt.t().contiguous()
    i, j = torch.arange(m).view(-1, 1), torch.arange(n).view(1, -1)
    M[(j < i) | (j - i > nb)] = 0.0
    return M


def exact(case, seed):
    kind = case["kind"]
    if kind == "ge2val":
        if case["input"] == "graded":
            return _sigmas(min(case["m"], case["n"]), case["smin"])
        return None
    if kind == "bandval":
        if case["n"] > 2000:
            return None
        return torch.linalg.svdvals(_band_storage(case["n"], case["nb"], seed).cpu())
    if kind in ("band", "call"):
        # The signs of B follow the tree; the flat and binomial steps are rebuilt here for the smaller sizes.
        m, n, nb = case["m"], case["n"], case["nb"]
        if m < n or m > 1100 or case["variant"] != "bidiag" or case["tree"] not in ("flatts", "greedy"):
            return None
        return _exact_band(_matrix(case, seed).cpu(), nb, case["tree"])
    return None
