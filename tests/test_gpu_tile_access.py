"""GPU tests of the tile kernels' two ways to a tile in memory: 16-byte accesses
through a buffer descriptor for contiguous columns (for nb <= 128 at any base and
any leading dimension below the descriptor's limit, in updates of ragged tiles
too; for nb = 256 whole, 16-byte aligned tiles), element accesses for everything
else (LQ steps).  The arithmetic does not depend on the way, so a
matrix reduced at any leading dimension and base gives the same bits, records
included, and never touches the padding between columns."""
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


def reduce_at(bb, A, plan, lda, offset):
    """The reduction of A stored with leading dimension lda, `offset` doubles
    past an aligned base; the padding holds 7.0 and must keep it."""
    m, n = A.shape
    buf = torch.full((offset + n * lda + 1,), 7.0, dtype=torch.float64, device="cuda")
    S = buf[offset:offset + n * lda].view(n, lda)
    S[:, :m] = torch.from_numpy(np.ascontiguousarray(A.T)).cuda()
    vt, ws = plan.alloc()
    print("reduce", m, n, plan.nb, lda, offset, flush=True)
    plan.execute(S, lda, vt, ws)
    assert bb.poll_error(ws) == 0
    assert bool((S[:, m:] == 7.0).all())
    return S[:, :m].t().cpu().numpy(), vt.cpu()


# one, two and (nb = 256) the two rounds of column tiles; whole and ragged
@pytest.mark.parametrize("m,n,nb,tree", [
    (96, 64, 32, "flatts"), (97, 61, 32, "greedy"), (192, 128, 64, "auto"), (256, 256, 128, "flatts"),
    (383, 255, 128, "greedy"), (512, 256, 256, "flatts"), (770, 513, 256, "greedy"),
])
def test_same_bits_at_any_leading_dimension_and_base(bb, m, n, nb, tree):
    A = workloads.gaussian(m, n, seed=m + n)
    plan = bb.Plan(m, n, nb, tree, "bidiag")
    even = m + m % 2 + 2
    B0, vt0 = reduce_at(bb, A, plan, even, 0)
    for lda, offset in [(even + 1, 0), (even, 1), (even + 1, 1)]:
        B, vt = reduce_at(bb, A, plan, lda, offset)
        assert np.array_equal(B, B0), (lda, offset)
        assert torch.equal(vt, vt0), (lda, offset)
    assert oracle.band_violation(B0, nb) == 0.0
    Bo, _ = oracle.band_reduce(A, nb)
    d = np.linalg.norm(oracle.sign_normalize(B0, nb) - oracle.sign_normalize(Bo, nb))
    assert d <= 50 * n * EPS * np.linalg.norm(A), d


@pytest.mark.parametrize("nb", [32, 64, 128, 256])
def test_zero_columns_and_scaled_columns(bb, nb):
    """Columns that are zero, or zero below the diagonal, take the identity
    reflector; columns 1e150 and 1e-150 times the others stay finite."""
    m, n = 2 * nb + 5, nb + 3
    A = workloads.gaussian(m, n, seed=nb)
    A[:, 3] = 0.0
    A[:, nb - 1] = 0.0
    A[:, nb + 1] *= 1e150
    A[:, 7] *= 1e-150
    plan = bb.Plan(m, n, nb, "greedy", "bidiag")
    B, _ = reduce_at(bb, A, plan, m, 0)
    assert np.isfinite(B).all()
    assert oracle.band_violation(B, nb) == 0.0
    assert abs(np.linalg.norm(B) / np.linalg.norm(A) - 1) <= 50 * n * EPS


@pytest.mark.parametrize("nb", [32, 64, 128])
@pytest.mark.parametrize("rest", [1, 3, 4, 15, 16, 17])
def test_last_tiles_of_any_height_and_width(bb, nb, rest):
    """Last row and column tiles that end inside a lane's four rows, at and one
    past a row tile: the band form against the oracle's, rows below the matrix
    untouched, tall and (transposed) wide."""
    m, n = 2 * nb + rest, nb + rest
    for rows, cols in ((m, n), (n, m)):
        A = workloads.gaussian(rows, cols, seed=10 * nb + rest)
        plan = bb.Plan(rows, cols, nb, "flatts", "bidiag")
        B, _ = reduce_at(bb, A, plan, rows + 3, 1)
        Bt, At = (B, A) if rows >= cols else (B.T, A.T)
        Bo, _ = oracle.band_reduce(np.ascontiguousarray(At), nb)
        d = np.linalg.norm(oracle.sign_normalize(np.ascontiguousarray(Bt), nb) - oracle.sign_normalize(Bo, nb))
        assert d <= 50 * n * EPS * np.linalg.norm(A), d


@pytest.mark.parametrize("nb", [32, 64, 128])
def test_same_bits_on_both_sides_of_the_buffer_limit(bb, nb):
    """Contiguous columns go through buffer accesses while lda nb < 2^27 and by
    element beyond: one below, at and one above, whole and ragged tiles."""
    m, n = 2 * nb + 3, nb + 5
    A = workloads.gaussian(m, n, seed=nb + 1)
    plan = bb.Plan(m, n, nb, "flatts", "bidiag")
    B0, vt0 = reduce_at(bb, A, plan, m, 0)
    limit = (1 << 27) // nb
    for lda in (limit - 1, limit, limit + 1):
        B, vt = reduce_at(bb, A, plan, lda, 0)
        assert np.array_equal(B, B0), lda
        assert torch.equal(vt, vt0), lda
