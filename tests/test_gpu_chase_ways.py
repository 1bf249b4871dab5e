"""The two ways of the band to bidiagonal chase (bb_bnd2bd): the band held in
registers where all its blocks find room, the sweeps over the band in memory
elsewhere or where a caller asks for them (bb_bnd2bd_group with a group).

* both give the same bits, at the edges of blocks, lanes and groups, and match
  the oracle;
* beside work that leaves too few compute units the call takes the second way
  and still gives the bits it gives alone.

Control word 2 of the workspace tells the way: 1 held, 2 the blocks did not
find room in time, 0 not tried.
"""
import ctypes

import numpy as np
import pytest

import oracle
import workloads
from oracle import ge2val as og

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps
HELD, GIVEN_UP, BY_SWEEPS = 1, 2, 0


@pytest.fixture(scope="module")
def bb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1611_06892_amd as m
    m.lib()
    return m


def square_band(n, nb, seed):
    """The n x n band the oracle's reduction leaves of a N(0,1) matrix, and its column-major storage."""
    A = np.ascontiguousarray(oracle.band_reduce(workloads.gaussian(n, n, seed), nb)[0][:n, :n])
    return A, torch.from_numpy(np.ascontiguousarray(A.T)).cuda()


def workspace(bb, n, nb):
    return torch.empty(bb.bnd2bd_workspace(n, nb), dtype=torch.uint8, device="cuda")


def way(ws):
    return int(ws[8:12].view(torch.int32)[0])


def check_against_oracle(A, n, nb, d, e):
    do, eo = og.bnd2bd(A, nb)
    tol = 50 * n * EPS * np.linalg.norm(og.upper_band(A, n, nb))
    assert np.max(np.abs(np.abs(d.cpu().numpy()) - np.abs(do))) <= tol
    assert np.max(np.abs(np.abs(e.cpu().numpy()) - np.abs(eo))) <= tol


@pytest.mark.parametrize("n,nb", [(3, 2), (3, 64), (9, 3), (65, 64), (67, 33), (130, 128), (194, 97), (260, 129),
                                  (273, 255), (389, 193), (514, 256), (400, 16), (1000, 96), (777, 32), (1201, 64),
                                  (1537, 2)])
def test_both_ways_give_the_same_bits(bb, n, nb):
    """Instances of 32, 64, 128 and 256 slots, one to four workgroups a block,
    bandwidths one below, at and one above a slot count or a member's rows, last
    blocks of one row and more."""
    print("case chase ways", n, nb, flush=True)
    A, S = square_band(n, nb, 8100 + n + nb)
    ws = workspace(bb, n, nb)
    held = bb.bnd2bd(S, n, n, nb, ws=ws, watchdog_s=20.0)
    assert way(ws) == HELD
    for group in (1, 16):
        d, e = bb.bnd2bd(S, n, n, nb, ws=ws, watchdog_s=20.0, group=group)
        assert way(ws) == BY_SWEEPS
        assert torch.equal(d, held[0]) and torch.equal(e, held[1])
    check_against_oracle(A, n, nb, *held)


@pytest.mark.parametrize("n,nb", [(1541, 2), (1000, 1), (2, 8)])
def test_sizes_that_are_never_held(bb, n, nb):
    """One block more than there is room for; nothing to chase."""
    print("case chase never held", n, nb, flush=True)
    A, S = square_band(n, nb, 8200 + n + nb)
    ws = workspace(bb, n, nb)
    d, e = bb.bnd2bd(S, n, n, nb, ws=ws, watchdog_s=20.0)
    assert way(ws) == BY_SWEEPS
    check_against_oracle(A, n, nb, d, e)


def random_band(n, nb, seed):
    """Column-major storage of an upper band of N(0,1) entries with sqrt(1 .. n) on the diagonal."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    S = torch.zeros(n, n, dtype=torch.float64, device="cuda")
    for k in range(1, nb + 1):
        S.diagonal(-k).copy_(torch.randn(n - k, generator=gen, dtype=torch.float64, device="cuda"))
    S.diagonal().copy_(torch.arange(1, n + 1, dtype=torch.float64, device="cuda").sqrt())
    return S


@pytest.mark.parametrize("n,nb", [(3000, 32), (4000, 64), (4000, 128), (2000, 256)])
def test_the_bits_do_not_depend_on_what_else_runs(bb, n, nb):
    """Beside a chase that takes 247 compute units with a workgroup each for
    about 0.1 s, and frees one of them every half millisecond, the 94, 63 (three
    and two a unit) and 32 workgroups of these bands do not find room in time."""
    print("case chase beside", n, nb, flush=True)
    big, bnb = 16000, 65
    Z, S = random_band(big, bnb, 8300), random_band(n, nb, 8301)
    wsz, ws = workspace(bb, big, bnb), workspace(bb, n, nb)
    alone = bb.bnd2bd(S, n, n, nb, ws=ws, watchdog_s=20.0)
    assert way(ws) == HELD
    # two streams may share a hardware queue and run one after the other: other pairs then
    for _ in range(4):
        one, two = torch.cuda.Stream(), torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.stream(one):
            bb.bnd2bd(Z, big, big, bnb, ws=wsz, watchdog_s=20.0, check=False)
        with torch.cuda.stream(two):
            d, e = bb.bnd2bd(S, n, n, nb, ws=ws, watchdog_s=20.0)
        torch.cuda.synchronize()
        assert bb.poll_error(wsz) == 0 and way(wsz) == HELD
        assert torch.equal(d, alone[0]) and torch.equal(e, alone[1])
        if way(ws) == GIVEN_UP:
            break
    assert way(ws) == GIVEN_UP


@pytest.mark.parametrize("n,nb", [(70, 16), (200, 64), (300, 128), (600, 256)])
@pytest.mark.parametrize("group", [0, 1])
def test_a_bidiagonal_passes_as_it_is(bb, n, nb, group):
    """Every reflector is the identity, which changes nothing: the entries come
    out bit by bit, and infinities, NaN and the largest numbers stay where they
    are."""
    print("case chase of a bidiagonal", n, nb, group, flush=True)
    rng = np.random.default_rng(8400 + n)
    d, e = rng.standard_normal(n), rng.standard_normal(n - 1)
    d[[3, n // 2]] = np.inf, -1e308
    e[[0, 5, n - 2]] = -np.inf, np.nan, 1e-308
    S = torch.from_numpy(np.ascontiguousarray((np.diag(d) + np.diag(e, 1)).T)).cuda()
    dg, eg = bb.bnd2bd(S, n, n, nb, watchdog_s=20.0, group=group)
    assert np.array_equal(dg.cpu().numpy(), d)
    assert np.array_equal(eg.cpu().numpy(), e, equal_nan=True)


@pytest.mark.parametrize("n,nb", [(768 * 17 + 1, 17), (512 * 33 + 1, 33), (256 * 65 + 1, 65), (85 * 129 + 1, 129),
                                  (64 * 193 + 1, 193)])
def test_the_largest_bands_are_held(bb, n, nb):
    """As many blocks as every instance has room for on the whole chip: three, two
    and one workgroup a compute unit, groups of three and of four."""
    print("case chase largest held", n, nb, flush=True)
    S = random_band(n, nb, 8500 + nb)
    ws = workspace(bb, n, nb)
    held = bb.bnd2bd(S, n, n, nb, ws=ws, watchdog_s=20.0)
    assert way(ws) == HELD
    swept = bb.bnd2bd(S, n, n, nb, ws=ws, watchdog_s=20.0, group=1)
    assert way(ws) == BY_SWEEPS
    assert torch.equal(held[0], swept[0]) and torch.equal(held[1], swept[1])


@pytest.mark.parametrize("n,nb", [(300, 64), (600, 256), (1541, 2)])
def test_a_call_takes_three_launches_at_most(bb, n, nb):
    """Beside work that fills the chip every launch waits for room of its own, so
    a small chase costs as many such waits as it has launches."""
    S = random_band(n, nb, 8600)
    ws = workspace(bb, n, nb)
    bb.bnd2bd(S, n, n, nb, ws=ws)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        bb.bnd2bd(S, n, n, nb, ws=ws, check=False)
    with open("/proc/self/maps") as maps:
        hip = ctypes.CDLL(next(line.split()[-1] for line in maps if "libamdhip64" in line))
    count = ctypes.c_size_t()
    assert hip.hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(count)) == 0
    assert count.value <= 3


@pytest.mark.parametrize("n,nb", [(1000, 1), (1000, 64), (1000, 128), (900, 256)])
@pytest.mark.parametrize("group", [0, 1])
def test_outputs_may_lie_in_the_input(bb, n, nb, group):
    """B is read before d and e are written, so they may take its place: d over
    the band of two columns, e over that of the first ones."""
    S = random_band(n, nb, 8700)
    want = bb.bnd2bd(S, n, n, nb, watchdog_s=20.0, group=group)
    ws = workspace(bb, n, nb)
    base = S.data_ptr()
    d, e = base + 8 * (n * (n // 2) + n // 2 - 20), base
    rc = bb.lib().bb_bnd2bd_group(base, n, n, nb, d, e, ws.data_ptr(), ws.numel(), 20.0, group,
                                  torch.cuda.current_stream().cuda_stream)
    assert rc == 0 and bb.poll_error(ws) == 0
    flat = S.view(-1)
    at = n * (n // 2) + n // 2 - 20
    assert torch.equal(flat[at:at + n], want[0]) and torch.equal(flat[:n - 1], want[1])
