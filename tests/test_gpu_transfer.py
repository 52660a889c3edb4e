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
