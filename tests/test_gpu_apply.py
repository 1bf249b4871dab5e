"""GPU tests of bb_apply_q / bb_apply_p: the orthogonal factors of a finished
reduction, formed from its V/T records (B = Q^T A P, Sections 3.4 and 3.5).

Pins that do not involve the GPU path's own arithmetic:
  * Q^T Q = I and P^T P = I, and P = diag(I_nb, P~) exactly (no LQ reflector
    touches the first tile column);
  * A = Q B P^T with the GPU's B;
  * Q diag(s) and P diag(t), with (s, t) the sign vectors that normalize B,
    are unique (block Golub-Kahan argument) and equal the oracle's;
  * Q^T (Q y) = y and the four products agree: Q^T A = B P^T.
Tolerance 50 n eps ||.||_F throughout (FP64).
"""
import numpy as np
import pytest

import oracle
import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


@pytest.fixture(scope="module")
def bb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1611_06892_amd as m
    m.lib()
    return m


def colmajor(X):
    """Column-major device storage S (S.t() is X)."""
    return torch.as_tensor(np.asarray(X, dtype=np.float64)).cuda().t().contiguous()


def reduce(bb, A, nb, tree, variant):
    m, n = A.shape
    plan = bb.Plan(m, n, nb, tree, variant, watchdog_s=10.0)
    S = colmajor(A)
    vt, ws = plan.alloc()
    plan.execute(S, m, vt, ws)
    assert bb.poll_error(ws) == 0
    return plan, S.t(), vt


def form(bb, plan, vt, side, rows, ncols, transpose=False):
    """Q[:, :ncols] (side 0) or P[:, :ncols] (side 1) on the device."""
    E = torch.eye(rows, ncols, dtype=torch.float64, device="cuda")
    S = E.t().contiguous()
    ws = (plan.apply_q if side == 0 else plan.apply_p)(S, rows, ncols, vt, transpose=transpose)
    assert bb.poll_error(ws) == 0
    return S.t()


CASES = [
    (512, 512, 64, "flatts", "bidiag"),     # the small square workload
    (700, 300, 64, "greedy", "rbidiag"),
    (1000, 700, 128, "auto", "bidiag"),
    (333, 129, 32, "flattt", "rbidiag"),    # ragged
    (640, 64, 64, "greedy", "bidiag"),      # one tile column: Q only, P = I
    (300, 200, 32, "greedy", "qronly"),     # QR only: P = I
]


@pytest.mark.parametrize("m,n,nb,tree,variant", CASES)
def test_factors_are_orthogonal_and_reconstruct(bb, m, n, nb, tree, variant):
    print("case", m, n, nb, tree, variant, flush=True)
    A = workloads.gaussian(m, n, seed=77 + m + n)
    plan, B, vt = reduce(bb, A, nb, tree, variant)
    Q = form(bb, plan, vt, 0, m, n)
    P = form(bb, plan, vt, 1, n, n)
    torch.cuda.synchronize()
    Ad = torch.as_tensor(A).cuda()
    I = torch.eye(n, dtype=torch.float64, device="cuda")
    tol = 50 * n * EPS
    assert float(torch.linalg.norm(Q.t() @ Q - I)) <= tol
    assert float(torch.linalg.norm(P.t() @ P - I)) <= tol
    k = min(nb, n)
    assert torch.equal(P[:k, :], I[:k, :]) and torch.equal(P[:, :k], I[:, :k])
    if variant == "qronly":
        assert torch.equal(P, I)
    res = float(torch.linalg.norm(Ad - Q @ B[:n] @ P.t()) / torch.linalg.norm(Ad))
    assert res <= tol, res


@pytest.mark.parametrize("m,n,nb,tree,variant", CASES[:4])
def test_factors_match_oracle_after_sign_normalization(bb, m, n, nb, tree, variant):
    print("case", m, n, nb, tree, variant, flush=True)
    A = workloads.gaussian(m, n, seed=177 + m + n)
    plan, B, vt = reduce(bb, A, nb, tree, variant)
    Qg = form(bb, plan, vt, 0, m, n).cpu().numpy()
    Pg = form(bb, plan, vt, 1, n, n).cpu().numpy()
    Bg = B.cpu().numpy()
    Bo, refl = oracle.band_reduce(A, nb)
    Qo, Po = oracle.form_q(refl), oracle.form_p(refl)
    sg, tg = oracle.sign_vectors(Bg, nb)
    so, to = oracle.sign_vectors(Bo, nb)
    # Gaussian inputs: every block has full rank, so the normalized factors are
    # unique; 50 n eps bounds the backward error, the block conditioning of a
    # Gaussian of this size stays well below 1e3.
    tol = 1e3 * 50 * n * EPS
    dq = np.linalg.norm(Qg * sg[None, :] - Qo * so[None, :])
    dp = np.linalg.norm(Pg * tg[None, :] - Po * to[None, :])
    print("dQ", dq, "dP", dp, flush=True)
    assert dq <= tol * np.sqrt(n) and dp <= tol * np.sqrt(n)


@pytest.mark.parametrize("m,n,nb,tree,variant", CASES[:4])
def test_transposed_application_and_round_trip(bb, m, n, nb, tree, variant):
    print("case", m, n, nb, tree, variant, flush=True)
    A = workloads.gaussian(m, n, seed=277 + m + n)
    plan, B, vt = reduce(bb, A, nb, tree, variant)
    # Q^T A = B P^T: apply Q^T to a copy of A, P to B^T.
    SA = colmajor(A)
    ws = plan.apply_q(SA, m, n, vt, transpose=True)
    assert bb.poll_error(ws) == 0
    # B^T (n x m) column-major is B (m x n) row-major.
    C = B.contiguous()
    ws = plan.apply_p(C, n, m, vt, transpose=False)    # P B^T, in place
    assert bb.poll_error(ws) == 0
    lhs = SA.t()                                       # Q^T A (m x n)
    rhs = C                                            # (P B^T)^T = B P^T, m x n
    nA = float(np.linalg.norm(A))
    assert float(torch.linalg.norm(lhs - rhs)) <= 50 * n * EPS * nA
    # round trip with a ragged column count
    y = workloads.gaussian(m, 37, seed=5)
    Sy = colmajor(y)
    plan.apply_q(Sy, m, 37, vt, transpose=False)
    plan.apply_q(Sy, m, 37, vt, transpose=True)
    torch.cuda.synchronize()
    assert float(torch.linalg.norm(Sy.t().cpu() - torch.as_tensor(y))) <= 50 * n * EPS * np.linalg.norm(y)


def test_full_size_probe_vectors(bb):
    """32768 x 2048 graded, nb = 128, R-BiDiag Greedy: ||A x - Q (B (P^T x))||
    for 8 seeded x, relative to ||A||_F ||x||."""
    cfg = workloads.CONFIGS["tall_graded"]
    m, n, nb = cfg["m"], cfg["n"], cfg["nb"]
    print("case tall_graded probes", flush=True)
    Ad, s = workloads.graded_device(m, n, *cfg["seeds"], cfg["smin"])
    plan = bb.Plan(m, n, nb, "greedy", "rbidiag", watchdog_s=20.0)
    S = Ad.t().contiguous()
    vt, ws = plan.alloc()
    plan.execute(S, m, vt, ws)
    assert bb.poll_error(ws) == 0
    B = S.t()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(11)
    X = torch.randn(n, 8, generator=gen, device="cuda", dtype=torch.float64)
    Y = X.t().contiguous()                   # X column-major (n x 8)
    plan.apply_p(Y, n, 8, vt, transpose=True)          # P^T X
    Z = B[:n] @ Y.t()                                   # B P^T X  (n x 8)
    W = torch.zeros(m, 8, dtype=torch.float64, device="cuda")
    W[:n] = Z
    SW = W.t().contiguous()
    ws2 = plan.apply_q(SW, m, 8, vt, transpose=False)  # Q B P^T X
    assert bb.poll_error(ws2) == 0
    err = torch.linalg.norm(Ad @ X - SW.t(), dim=0) / (torch.linalg.norm(Ad) * torch.linalg.norm(X, dim=0))
    print("probe residuals", err.cpu().numpy(), flush=True)
    assert float(err.max()) <= 50 * n * EPS


@pytest.mark.parametrize("m,n,nb", [(1024, 256, 128), (900, 300, 128), (1024, 512, 256)])
@pytest.mark.parametrize("transpose", [False, True])
def test_strips_of_64_and_128_columns_give_the_same_bits(bb, m, n, nb, transpose):
    """Applied to a few columns, Q and P are chains of 64-column strips; to
    24000 columns, the strips are 128 wide.  Every 16-column slice is the same
    arithmetic, so the columns agree bit by bit, also those of a last tile that
    ends inside a strip."""
    print("case strips", m, n, nb, transpose, flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    S = torch.randn(n, m, generator=g, device="cuda", dtype=torch.float64)
    plan = bb.Plan(m, n, nb, "greedy", "bidiag")
    vt, ws = plan.alloc()
    plan.execute(S, m, vt, ws)
    for rows, run in ((m, plan.apply_q), (n, plan.apply_p)):
        C = torch.randn(24000, rows, generator=g, device="cuda", dtype=torch.float64)
        few = C[-331:].clone()
        run(C, rows, 24000, vt, transpose=transpose)
        # the last 331 columns start inside a tile of the wide C
        run(few, rows, 331, vt, transpose=transpose)
        assert torch.equal(C[-331:], few)
