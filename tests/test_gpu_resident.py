"""Bi-CG runs held on the chip (csrc/resident.hip) against the oracle and against the
launch-per-sweep form.

Both evaluate every element with the oracle's arithmetic, and the compensated dot products
equal the exactly rounded ones, so iterates and iteration counts are compared for equality.
The grids have one and several bricks, whole and partial ones, one to eight cells per thread."""
import numpy as np
import pytest

import oracle as O
from manufactured import config_problem, make_arrays
from manufactured.twod import family_2d, make_arrays_2d

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ex():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1901_05118_amd as ex
    ex.load()
    yield ex
    ex.set_timing(False)
    ex.finalize()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


# (cells, levels): 8^3 and 10^3 are the smallest grids the form takes
@pytest.mark.parametrize("N,levels", [(8, 3), (12, 3), (16, 3), (20, 3), (28, 3), (40, 4), (48, 5),
                                      (56, 4), (80, 5), (96, 6)])
@pytest.mark.parametrize("bc", [1, 2])
def test_run_equals_oracle(ex, N, levels, bc):
    print(f"resident N={N} bc={bc}", flush=True)
    ex.setup(N, levels, bc)
    rng = np.random.default_rng(N + bc)
    b, x0 = rng.standard_normal((2, (N - 1) ** 3))
    its = 12
    x = dev(x0)
    rc, it, rr = ex.bicg(levels - 1, dev(b), x, 0.0, its)
    xr, itr, rrr, rcr = O.bicg(N, bc, b, x0, 0.0, maxit=its)
    assert rc == ex.ENOCONV and it == itr == its
    assert rr == rrr
    np.testing.assert_array_equal(x.cpu().numpy(), xr)


@pytest.mark.parametrize("N,levels,bc", [(40, 4, 1), (64, 5, 2), (96, 6, 1), (96, 6, 2),
                                         (112, 5, 1), (128, 6, 2)])
def test_mixed_cascade_equals_sweeps(ex, N, levels, bc):
    """FP32 vectors on every level, with residual replacements (resumed runs).  Timed sweeps
    take the launch-per-sweep form."""
    print(f"resident mixed N={N} bc={bc}", flush=True)
    arr = make_arrays(config_problem(2), N, bc)
    f, g1, g2 = dev(arr.f), dev(arr.g1), dev(arr.g2)
    got = []
    for timed in (False, True):
        u = torch.empty_like(f)
        ex.set_timing(timed)
        rc, st = ex.solve_ex(N, levels, bc, f, g1, g2, 1e-7, u, precision=ex.MIXED,
                             fp32_min_unknowns=1)
        assert rc == ex.OK, ex.last_error()
        launches = ex.get_timing(levels - 1, 0)[1] + ex.get_timing(levels - 1, 2)[1]
        assert (launches > 0) == timed
        got.append((u.cpu().numpy(), [(s["iterations"], s["runs"]) for s in st.levels()]))
    ex.set_timing(False)
    assert got[0][1] == got[1][1]
    np.testing.assert_array_equal(got[0][0], got[1][0])


# planes: one brick (8, 24), whole and partial rows of bricks, one to eight cells per thread;
# 1024^2 is the largest plane the form takes
@pytest.mark.parametrize("N,levels", [(8, 3), (24, 3), (40, 4), (64, 5), (96, 5), (200, 4), (256, 7),
                                      (512, 6), (1024, 6)])
@pytest.mark.parametrize("bc", [1, 2])
def test_plane_run_equals_oracle(ex, N, levels, bc):
    print(f"resident plane N={N} bc={bc}", flush=True)
    ex.setup_2d(N, levels, bc)
    rng = np.random.default_rng(N + bc)
    b, x0 = rng.standard_normal((2, (N - 1) ** 2))
    its = 12
    x = dev(x0)
    rc, it, rr = ex.bicg(levels - 1, dev(b), x, 0.0, its)
    xr, itr, rrr, rcr = O.bicg_2d(N, bc, b, x0, 0.0, maxit=its)
    assert rc == ex.ENOCONV and it == itr == its
    assert rr == rrr
    np.testing.assert_array_equal(x.cpu().numpy(), xr)


@pytest.mark.parametrize("N,levels,bc", [(96, 5, 1), (512, 6, 1), (512, 6, 2), (1024, 6, 1)])
def test_mixed_plane_equals_sweeps(ex, N, levels, bc):
    print(f"resident mixed plane N={N} bc={bc}", flush=True)
    arr = make_arrays_2d(family_2d(5), N, bc)
    f, g1, g2 = dev(arr.f), dev(arr.g1), dev(arr.g2)
    got = []
    for timed in (False, True):
        u = torch.empty_like(f)
        ex.set_timing(timed)
        rc, st = ex.solve_ex_2d(N, levels, bc, f, g1, g2, 1e-9, u, precision=ex.MIXED,
                                fp32_min_unknowns=1)
        assert rc == ex.OK, ex.last_error()
        launches = ex.get_timing(levels - 1, 0)[1] + ex.get_timing(levels - 1, 2)[1]
        assert (launches > 0) == timed
        got.append((u.cpu().numpy(), [(s["iterations"], s["runs"]) for s in st.levels()]))
    ex.set_timing(False)
    assert got[0][1] == got[1][1]
    np.testing.assert_array_equal(got[0][0], got[1][0])


@pytest.mark.parametrize("case", ["fp64", "mixed", "mixed small", "capped"])
def test_batch_runs_equal_steps(ex, case):
    """Runs of a batch in shared launches (more of them than there are CUs for; 160^3 advances by
    steps beside them) against the persistent steps, which take all systems."""
    print(f"resident batch {case}", flush=True)
    sizes = [(16, 3), (24, 4), (40, 4), (48, 5), (64, 5), (64, 5), (80, 5), (96, 6), (28, 3), (32, 4)]
    sizes += {"fp64": [(112, 5)], "mixed": [(96, 5), (128, 6)], "capped": [(160, 6)]}.get(case, [])
    probs, fields = [], []
    for j, (N, nl) in enumerate(sizes):
        arr = make_arrays(config_problem(2), N, 1 + j % 2)
        fields.append([dev(arr.f), dev(arr.g1), dev(arr.g2)])
    options = {"fp64": {}, "mixed": dict(precision=ex.MIXED),
               "mixed small": dict(precision=ex.MIXED, fp32_min_unknowns=1),
               "capped": dict(max_iters=37)}[case]
    got = []
    for persistent in (False, True):
        probs = [dict(n_finest=N, n_levels=nl, bc_kind=1 + j % 2, f=f, g1=g1, g2=g2,
                      u_out=torch.empty_like(f), ut_out=torch.empty_like(f))
                 for j, ((N, nl), (f, g1, g2)) in enumerate(zip(sizes, fields))]
        rc, stats = ex.solve_batch(probs, 1e-7, persistent=persistent, **options)
        got.append((rc, [[(s["iterations"], s["runs"], s["status"]) for s in st.levels()] for st in stats],
                    [p["u_out"].cpu().numpy() for p in probs], [p["ut_out"].cpu().numpy() for p in probs]))
    assert got[0][0] == got[1][0]
    assert got[0][1] == got[1][1]
    for k in (2, 3):
        for a, b in zip(got[0][k], got[1][k]):
            np.testing.assert_array_equal(a, b)


# FP64 with 16 cells per thread (the iterate in memory, q* not kept)
@pytest.mark.parametrize("N,levels", [(112, 5), (128, 6)])
@pytest.mark.parametrize("bc", [1, 2])
def test_large_run_equals_oracle(ex, N, levels, bc):
    print(f"resident N={N} bc={bc}", flush=True)
    ex.setup(N, levels, bc)
    rng = np.random.default_rng(N + bc)
    b, x0 = rng.standard_normal((2, (N - 1) ** 3))
    for its in (1, 9):
        x = dev(x0)
        rc, it, rr = ex.bicg(levels - 1, dev(b), x, 0.0, its)
        xr, itr, rrr, rcr = O.bicg(N, bc, b, x0, 0.0, maxit=its)
        assert rc == ex.ENOCONV and it == itr == its
        assert rr == rrr
        np.testing.assert_array_equal(x.cpu().numpy(), xr)
