"""Forms of the sweeps that grids up to 128^3 take only where their runs are not resident: the
phase steps of a batch (resident launches refused), in both precisions and side by side, and the
stored form with its deferred update."""
import numpy as np
import pytest

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
    ex.finalize()


@pytest.fixture(autouse=True)
def as_before(ex):
    ex.finalize()
    ex.resident_control()
    yield
    ex.resident_control()
    ex.set_timing(False)
    ex.finalize()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def _problems(sizes):
    probs = []
    for j, (N, nl) in enumerate(sizes):
        arr = make_arrays(config_problem(2 + j % 3), N, 1 + j % 2)
        f = dev(arr.f)
        probs.append(dict(n_finest=N, n_levels=nl, bc_kind=1 + j % 2, f=f, g1=dev(arr.g1),
                          g2=dev(arr.g2)))
    return probs


def _solve(ex, probs, tol, persistent=False, **kw):
    for p in probs:
        p["u_out"] = torch.full_like(p["f"], float("nan"))
    rc, stats = ex.solve_batch(probs, tol, persistent=persistent, **kw)
    assert rc == ex.OK, ex.last_error()
    return ([[(s["iterations"], s["runs"]) for s in st.levels()] for st in stats],
            [p["u_out"].cpu().numpy() for p in probs])


def _same(a, b):
    assert a[0] == b[0]
    for x, y in zip(a[1], b[1]):
        np.testing.assert_array_equal(x, y)


# FP32 levels from 2^16 unknowns: 48^3 and 64^3 finest levels beside FP64 systems
@pytest.mark.parametrize("case", ["fp64", "reliable", "restart", "all fp32"])
def test_phase_steps_equal_persistent_steps(ex, case):
    options = {"fp64": {}, "reliable": dict(precision=ex.MIXED, fp32_min_unknowns=1 << 16),
               "restart": dict(precision=ex.MIXED, fp32_min_unknowns=1 << 16, refine=ex.RESTART),
               "all fp32": dict(precision=ex.MIXED, fp32_min_unknowns=1)}[case]
    probs = _problems([(32, 4), (48, 5), (64, 5), (40, 4)])
    want = _solve(ex, probs, 1e-8, persistent=True, **options)
    ex.resident_control(refuse=0)
    got = _solve(ex, probs, 1e-8, **options)
    assert ex.resident_counts() == (1, 1)
    if case in ("reliable", "all fp32"):
        assert any(levels[-1][1] > 1 for levels in got[0])       # residuals were replaced
    _same(got, want)


def test_large_steps_of_both_precisions_beside_resident_runs(ex):
    """The finest 160^3 level in FP64 and 192^3 in FP32, on two streams, and smaller systems
    resident in between."""
    probs = _problems([(160, 6), (192, 7), (64, 5), (96, 6)])
    options = dict(precision=ex.MIXED, fp32_min_unknowns=1 << 22)
    want = _solve(ex, probs, 1e-7, persistent=True, **options)
    got = _solve(ex, probs, 1e-7, **options)
    made, gave_up = ex.resident_counts()
    assert made > 0 and gave_up == 0
    assert got[0][1][-1][1] > 1                                   # 192^3: residuals were replaced
    _same(got, want)


def test_tuned_phase_steps_keep_results(ex):
    """The shapes that the batch tuner records change no result of the steps (FP64 and FP32)."""
    probs = _problems([(32, 4), (48, 5), (64, 5)])
    for p in probs:
        p["u_out"] = torch.empty_like(p["f"])
    options = dict(precision=ex.MIXED, fp32_min_unknowns=1 << 16)
    ex.resident_control(refuse=0)
    want = _solve(ex, probs, 1e-8, **options)
    ty, ms = ex.autotune_batch(probs, precision=ex.MIXED, reps=1, fp32_min_unknowns=1 << 16)
    assert ty in (4, 8) and ms > 0
    _same(_solve(ex, probs, 1e-8, **options), want)


def test_deferred_update_graphs_events_and_cg(ex):
    """The stored form with FP32 vectors at 64^3, its update deferred: in captured windows, launch
    by launch, and the CG specialisation, which does not defer it."""
    N, nl, bc = 64, 5, 2
    arr = make_arrays(config_problem(2), N, bc)
    f, g1, g2 = dev(arr.f), dev(arr.g1), dev(arr.g2)
    got = []
    for timed, method in ((False, ex.BICG), (True, ex.BICG), (False, ex.CG)):
        ex.set_timing(timed)
        u = torch.empty_like(f)
        rc, st = ex.solve_ex(N, nl, bc, f, g1, g2, 1e-9, u, precision=ex.MIXED, method=method,
                             fp32_min_unknowns=1, recompute_min_unknowns=1 << 30)
        assert rc == ex.OK, ex.last_error()
        assert ex.resident_counts() == (0, 0)
        if timed:
            assert ex.get_timing(nl - 1, 2)[1] > 0                # deferred updates
        got.append(([[(s["iterations"], s["runs"]) for s in st.levels()]], [u.cpu().numpy()]))
    assert got[0][0][0][-1][1] > 1
    _same(got[0], got[1])
    _same(got[0], got[2])
