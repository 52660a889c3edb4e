"""What follows when a resident launch is refused or gives up waiting (forced from the host by
excmg_resident_control: a wait of one look, a launch not made; every kernel ends normally).

The launch-per-sweep form takes over with the same arithmetic, so results are compared for
equality."""
import numpy as np
import pytest

import oracle as O
from manufactured import config_problem, make_arrays

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ex():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1901_05118_amd as ex
    ex.load()
    yield ex


@pytest.fixture(autouse=True)
def as_before(ex):
    ex.finalize()          # (a context, or batch, that gave up does not try again)
    ex.resident_control()
    yield
    ex.resident_control()
    ex.finalize()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


# 16^3: workgroups on one XCD (the first exchange finds out where they are); 128^3: the iterate
# of the run in memory
@pytest.mark.parametrize("N,levels,bc", [(16, 3, 1), (40, 4, 2), (96, 6, 1), (128, 6, 2)])
def test_expired_run_goes_on_by_sweeps(ex, N, levels, bc):
    print(f"give up N={N} bc={bc}", flush=True)
    ex.setup(N, levels, bc)
    rng = np.random.default_rng(N)
    b, x0 = rng.standard_normal((2, (N - 1) ** 3))
    its = 6
    xr, itr, rrr, rcr = O.bicg(N, bc, b, x0, 0.0, maxit=its)
    ex.resident_control(expire=0)
    for _ in range(2):
        x = dev(x0)
        rc, it, rr = ex.bicg(levels - 1, dev(b), x, 0.0, its)
        assert (rc, it, rr) == (ex.ENOCONV, its, rrr)
        np.testing.assert_array_equal(x.cpu().numpy(), xr)
        # given up once, and not tried again in this context
        assert ex.resident_counts() == (1, 1)


def _mixed(ex, N, levels, bc, **kw):
    arr = make_arrays(config_problem(2), N, bc)
    f, g1, g2 = dev(arr.f), dev(arr.g1), dev(arr.g2)
    u = torch.empty_like(f)
    rc, st = ex.solve_ex(N, levels, bc, f, g1, g2, 1e-7, u, precision=ex.MIXED,
                         fp32_min_unknowns=1, **kw)
    assert rc == ex.OK, ex.last_error()
    return u.cpu().numpy(), [(s["iterations"], s["runs"]) for s in st.levels()]


def test_refused_launches_of_fresh_and_resumed_runs(ex):
    """FP32 vectors with residual replacements: launch 0 is fresh, the next ones of its level
    resumed; the sweeps go on from the state that the launches before left."""
    N, levels, bc = 40, 4, 1
    ex.resident_control(refuse=0)
    u, its = _mixed(ex, N, levels, bc)
    assert ex.resident_counts() == (1, 1)
    ex.finalize()
    ex.resident_control()
    resident = _mixed(ex, N, levels, bc)
    made, gave_up = ex.resident_counts()
    assert gave_up == 0 and made > 3
    runs = [resident] + [None] * 4
    for k in range(1, 5):
        ex.finalize()
        ex.resident_control(refuse=min(k, made - 1))
        runs[k] = _mixed(ex, N, levels, bc)
        assert ex.resident_counts()[1] == 1
    for v, n in runs:
        assert n == its
        np.testing.assert_array_equal(v, u)


@pytest.mark.parametrize("turn", [1, 4, 5])
@pytest.mark.parametrize("N,levels,bc", [(8, 3, 1), (16, 3, 1), (40, 4, 2), (96, 6, 1), (128, 6, 2)])
def test_halted_run_goes_on(ex, N, levels, bc, turn):
    """A run halted after every `turn` iterations: even and odd ones (which pair of buffers holds
    the directions), the last launch not a whole one."""
    print(f"halted N={N} bc={bc} turn={turn}", flush=True)
    ex.setup(N, levels, bc)
    rng = np.random.default_rng(N)
    b, x0 = rng.standard_normal((2, (N - 1) ** 3))
    its = 11 if N < 128 else 6
    xr, itr, rrr, rcr = O.bicg(N, bc, b, x0, 0.0, maxit=its)
    ex.resident_control(turn=turn)
    x = dev(x0)
    rc, it, rr = ex.bicg(levels - 1, dev(b), x, 0.0, its)
    assert (rc, it, rr) == (ex.ENOCONV, its, rrr)
    np.testing.assert_array_equal(x.cpu().numpy(), xr)
    assert ex.resident_counts() == (-(-its // turn), 0)


@pytest.mark.parametrize("turn", [4, 5])
@pytest.mark.parametrize("N,levels", [(64, 5), (512, 6)])
def test_halted_plane_run_goes_on(ex, N, levels, turn):
    ex.setup_2d(N, levels, 1)
    rng = np.random.default_rng(N)
    b, x0 = rng.standard_normal((2, (N - 1) ** 2))
    xr, itr, rrr, rcr = O.bicg_2d(N, 1, b, x0, 0.0, maxit=11)
    ex.resident_control(turn=turn)
    x = dev(x0)
    assert ex.bicg(levels - 1, dev(b), x, 0.0, 11) == (ex.ENOCONV, 11, rrr)
    np.testing.assert_array_equal(x.cpu().numpy(), xr)
    assert ex.resident_counts() == (3, 0)


def test_a_long_run_lets_others_in(ex):
    """A launch holds the chip, so a long run takes several (20 ms of iterations each, some 4000 on
    this plane)."""
    N, levels = 256, 7
    ex.setup_2d(N, levels, 1)
    b = dev(np.random.default_rng(1).standard_normal((N - 1) ** 2))
    x = torch.zeros_like(b)
    rc, it, rr = ex.bicg(levels - 1, b, x, 1e-200, 20000)
    made, gave_up = ex.resident_counts()
    print(f"{it} iterations in {made} launches", flush=True)
    assert rc == ex.ENOCONV and it == 20000
    assert gave_up == 0 and 3 <= made <= 10


# `wait` 0: given up at the first exchange that a workgroup has to wait for; longer ones: later,
# and perhaps not by all workgroups.  turn 1 ends most launches in their last exchange.
@pytest.mark.parametrize("turn", [1, 4, 5])
@pytest.mark.parametrize("wait", [0, 120, 250])
@pytest.mark.parametrize("N,levels,bc", [(16, 3, 2), (48, 5, 1), (112, 5, 2)])
def test_run_that_gives_up_on_the_way(ex, N, levels, bc, turn, wait):
    print(f"give up on the way N={N} turn={turn} wait={wait}", flush=True)
    ex.setup(N, levels, bc)
    rng = np.random.default_rng(N)
    b, x0 = rng.standard_normal((2, (N - 1) ** 3))
    its = 11
    xr, itr, rrr, rcr = O.bicg(N, bc, b, x0, 0.0, maxit=its)
    for launch in (1, 2) if turn < 5 else (1,):
        ex.finalize()
        ex.setup(N, levels, bc)
        ex.resident_control(turn=turn, expire=launch, wait=wait)
        x = dev(x0)
        rc, it, rr = ex.bicg(levels - 1, dev(b), x, 0.0, its)
        assert (rc, it, rr) == (ex.ENOCONV, its, rrr)
        np.testing.assert_array_equal(x.cpu().numpy(), xr)
        if wait == 0:
            assert ex.resident_counts() == (launch + 1, 1)


@pytest.mark.parametrize("turn", [0, 7, 8])
def test_mixed_run_that_gives_up(ex, turn):
    """FP32 vectors: fresh, resumed and halted runs that give up equal the sweeps."""
    N, levels, bc = 40, 4, 1
    ex.resident_control(refuse=0)
    u, its = _mixed(ex, N, levels, bc)
    for launch in (None, 0, 1, 2, 3, 5, 8):
        print(f"mixed: launch {launch} gives up", flush=True)
        ex.finalize()
        ex.resident_control(turn=turn, **({} if launch is None else dict(expire=launch)))
        v, n = _mixed(ex, N, levels, bc)
        made, gave_up = ex.resident_counts()
        assert gave_up == (launch is not None and launch < made)
        assert n == its
        np.testing.assert_array_equal(v, u)


def test_mixed_plane_halted(ex):
    from manufactured.twod import family_2d, make_arrays_2d
    N, levels, bc = 96, 5, 1
    arr = make_arrays_2d(family_2d(5), N, bc)
    f, g1, g2 = dev(arr.f), dev(arr.g1), dev(arr.g2)
    got = []
    for control in (dict(refuse=0), dict(turn=8), dict(turn=9, expire=7)):
        ex.finalize()
        ex.resident_control(**control)
        u = torch.empty_like(f)
        rc, st = ex.solve_ex_2d(N, levels, bc, f, g1, g2, 1e-9, u, precision=ex.MIXED,
                                fp32_min_unknowns=1)
        assert rc == ex.OK, ex.last_error()
        got.append((u.cpu().numpy(), [(s["iterations"], s["runs"]) for s in st.levels()]))
    for v, n in got[1:]:
        assert n == got[0][1]
        np.testing.assert_array_equal(v, got[0][0])


def test_run_with_a_shadow_residual(ex):
    """A given shadow residual (r*_0 alone: M = I, no dual iterate) runs resident, halted or not."""
    N, levels, bc = 40, 4, 1
    rng = np.random.default_rng(5)
    b, x0, s = rng.standard_normal((3, (N - 1) ** 3))
    got = []
    for control in (dict(refuse=0), {}, dict(turn=4), dict(turn=4, expire=1)):
        ex.finalize()
        ex.setup(N, levels, bc)
        ex.resident_control(**control)
        x = dev(x0)
        rc, it, rr = ex.bicg_ex(levels - 1, dev(b), x, 0.0, 11, shadow=dev(s))
        assert (rc, it) == (ex.ENOCONV, 11)
        assert ex.resident_counts()[0] > 0
        got.append((rr, x.cpu().numpy()))
    for rr, x in got[1:]:
        assert rr == got[0][0]
        np.testing.assert_array_equal(x, got[0][1])


def test_resumed_run_with_nothing_to_do(ex):
    """inner_tol 2: every replaced residual is below its threshold at once, so a resumed run stops
    before its first iteration and leaves the iterate alone."""
    N, levels, bc = 40, 4, 1
    arr = make_arrays(config_problem(2), N, bc)
    f, g1, g2 = dev(arr.f), dev(arr.g1), dev(arr.g2)
    got = []
    for control in ({}, dict(refuse=0)):
        ex.finalize()
        ex.resident_control(**control)
        u = torch.empty_like(f)
        rc, st = ex.solve_ex(N, levels, bc, f, g1, g2, 1e-7, u, precision=ex.MIXED,
                             fp32_min_unknowns=1, inner_tol=2.0, max_outer=8)
        assert rc == ex.ENOCONV
        got.append(([(s["iterations"], s["runs"]) for s in st.levels()], u.cpu().numpy()))
    assert got[0][0] == got[1][0]
    np.testing.assert_array_equal(got[0][1], got[1][1])


def test_exchange_numbers_wrap(ex):
    N, levels, bc = 40, 4, 1
    rng = np.random.default_rng(7)
    b, x0 = rng.standard_normal((2, (N - 1) ** 3))
    xr, itr, rrr, rcr = O.bicg(N, bc, b, x0, 0.0, maxit=12)
    ex.resident_control(number=2 ** 32 - 50)
    ex.setup(N, levels, bc)
    for _ in range(5):
        x = dev(x0)
        assert ex.bicg(levels - 1, dev(b), x, 0.0, 12) == (ex.ENOCONV, 12, rrr)
        np.testing.assert_array_equal(x.cpu().numpy(), xr)
    assert ex.resident_counts() == (5, 0)


def _batch(ex, sizes, tol=1e-7, persistent=False, **kw):
    probs = []
    for j, (N, nl) in enumerate(sizes):
        arr = make_arrays(config_problem(2), N, 1 + j % 2)
        f = dev(arr.f)
        probs.append(dict(n_finest=N, n_levels=nl, bc_kind=1 + j % 2, f=f, g1=dev(arr.g1),
                          g2=dev(arr.g2), u_out=torch.empty_like(f)))
    rc, stats = ex.solve_batch(probs, tol, persistent=persistent, **kw)
    assert rc == ex.OK, ex.last_error()
    return ([p["u_out"].cpu().numpy() for p in probs],
            [[(s["iterations"], s["runs"], s["status"]) for s in st.levels()] for st in stats],
            [st.levels()[-1] for st in stats])


def _options(ex, case):
    return {"fp64": {}, "mixed": dict(precision=ex.MIXED, fp32_min_unknowns=1 << 16),
            "fp32": dict(precision=ex.MIXED, fp32_min_unknowns=1)}[case]


SIZES = [(32, 4), (48, 5), (64, 5), (40, 4)]


@pytest.mark.parametrize("case", ["fp64", "mixed", "fp32"])
def test_batch_hands_halted_runs_to_the_steps(ex, case):
    """From the refused launch on every system is advanced by steps, those that were halted
    too."""
    want = _batch(ex, SIZES, persistent=True, **_options(ex, case))
    for k in (1, 2, 4):
        print(f"batch {case}: launch {k} refused", flush=True)
        ex.finalize()
        ex.resident_control(refuse=k)
        got = _batch(ex, SIZES, **_options(ex, case))
        assert ex.resident_counts() == (k + 1, 1)
        assert got[1] == want[1]
        for a, b in zip(got[0], want[0]):
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("case", ["fp64", "fp32"])
@pytest.mark.parametrize("launch", [0, 2])
def test_batch_run_that_expires_leaves_the_others(ex, case, launch):
    """The waits of one run expire: its level starts again from the iterate it has, and meets
    its tolerance; the others' runs go on by steps bit for bit."""
    late = 2
    want = _batch(ex, SIZES, persistent=True, **_options(ex, case))
    ex.resident_control(expire=launch, problem=late)
    got = _batch(ex, SIZES, **_options(ex, case))
    assert ex.resident_counts() == (launch + 1, 1)
    for j, (N, nl) in enumerate(SIZES):
        if j != late:
            assert got[1][j] == want[1][j]
            np.testing.assert_array_equal(got[0][j], want[0][j])
            continue
        arr = make_arrays(config_problem(2), N, 1 + j % 2)
        b = O.rhs(N, 1 + j % 2, arr.f, arr.g1, arr.g2)
        r = O.residual(N, 1 + j % 2, b, O.interior(got[0][j].reshape((N + 1,) * 3)))
        assert np.sqrt(O.dot(r, r) / O.dot(b, b)) <= 1e-7
        assert got[2][j]["status"] == ex.OK


def test_batch_exchange_numbers_wrap(ex):
    want = _batch(ex, SIZES, persistent=True)
    ex.resident_control(number=2 ** 32 - 101000)
    got = _batch(ex, SIZES)
    assert ex.resident_counts()[1] == 0
    assert got[1] == want[1]
    for a, b in zip(got[0], want[0]):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("case", ["fp64", "fp32"])
def test_batch_runs_halted_by_their_turn(ex, case):
    want = _batch(ex, SIZES, persistent=True, **_options(ex, case))
    ex.resident_control(turn=50)
    got = _batch(ex, SIZES, **_options(ex, case))
    longest = max(sum(n for n, _, _ in its) for its in got[1])
    made, gave_up = ex.resident_counts()
    assert made >= longest / 50 and gave_up == 0
    assert got[1] == want[1]
    for a, b in zip(got[0], want[0]):
        np.testing.assert_array_equal(a, b)


def test_batch_that_gave_up(ex):
    """The iterations of the run that gave up count, and no later batch waits again."""
    N, nl = 64, 5
    arr = make_arrays(config_problem(2), N, 1)
    f, g1, g2 = dev(arr.f), dev(arr.g1), dev(arr.g2)
    prob = dict(n_finest=N, n_levels=nl, bc_kind=1, f=f, g1=g1, g2=g2, u_out=torch.empty_like(f))

    def level2():
        rc, stats = ex.solve_batch([prob], 1e-12, max_iters=60, max_runs=1)
        assert rc == ex.ENOCONV
        return stats[0].levels()[2]["iterations"]

    ex.resident_control(turn=20, expire=1)
    assert level2() == 20 + 60            # 20 resident, then a fresh run by steps
    assert ex.resident_counts() == (2, 1)
    assert level2() == 60
    assert ex.resident_counts() == (2, 1)
    ex.finalize()
    assert level2() == 60
    assert ex.resident_counts()[0] > 2
