"""DSOLVE on the smallest levels, on both sides of 32 unknowns, against the oracle (exact: the
factor and the substitutions subtract in the same order)."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# unknowns of level 0: 1, 4, 9, 16, 25, 36 in 2D; 1, 8, 27, 64 in 3D
@pytest.mark.parametrize("dim,N", [(2, 2), (2, 3), (2, 4), (2, 5), (2, 6), (2, 7), (3, 2), (3, 3),
                                   (3, 4), (3, 5)])
@pytest.mark.parametrize("bc", [1, 2])
def test_smallest_levels(dim, N, bc):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1901_05118_amd as ex
    (ex.setup if dim == 3 else ex.setup_2d)(N * 4, 3, bc)
    b = np.random.default_rng(N).standard_normal((N - 1) ** dim)
    for scale in (1.0, 2.0 ** -1015):
        x = torch.empty(b.size, dtype=torch.float64, device="cuda")
        ex.dsolve(0, torch.from_numpy(b * scale).cuda(), x)
        want = (O.dsolve if dim == 3 else O.dsolve_2d)(N, bc, b * scale)
        np.testing.assert_array_equal(x.cpu().numpy(), want)
    ex.finalize()
