"""EXP_finite and EXP_true against the oracle at the edges of their tiles and marches (exact:
both evaluate the same formulas in the same order)."""
import numpy as np
import pytest

import oracle as O

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


# one cell; a tile less, exactly and more than 64 and 128 nodes wide; uneven last marches
@pytest.mark.parametrize("N", [4, 12, 60, 64, 68, 124, 128, 132, 196])
def test_tile_edges(ex, N):
    print(f"transfer N={N}", flush=True)
    rng = np.random.default_rng(N)
    u2, u1, u0 = (rng.standard_normal((N // s + 1,) * 3) for s in (1, 2, 4))
    d2, d1, d0 = (torch.from_numpy(a).cuda() for a in (u2, u1, u0))
    out = torch.full_like(d2, float("nan"))
    ex.exp_finite(N, d1, d0, out)
    np.testing.assert_array_equal(out.cpu().numpy(), O.exp_finite(N, u1, u0))
    out.fill_(float("nan"))
    ex.exp_true(N, d2, d1, out)
    np.testing.assert_array_equal(out.cpu().numpy(), O.exp_true(N, u2, u1))


def test_overlapping_calls(ex):
    """Calls from several threads at once: the kept intermediate grid serves one at a time."""
    import threading
    rng = np.random.default_rng(3)
    N = 64
    want, got, args = [], [None] * 4, []
    for k in range(4):
        u1 = rng.standard_normal((N // 2 + 1,) * 3)
        u0 = rng.standard_normal((N // 4 + 1,) * 3)
        want.append(O.exp_finite(N, u1, u0))
        args.append((torch.from_numpy(u1).cuda(), torch.from_numpy(u0).cuda(),
                     torch.empty((N + 1,) * 3, dtype=torch.float64, device="cuda")))

    def calls(k):
        same = True
        for _ in range(20):
            ex.exp_finite(N, *args[k])
            same = same and np.array_equal(args[k][2].cpu().numpy(), want[k])
        got[k] = same

    threads = [threading.Thread(target=calls, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert got == [True] * 4
