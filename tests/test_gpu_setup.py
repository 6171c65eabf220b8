"""GPU parity of the operator set-up at the edges of its kernels: grids of
one voxel, one row or one plane (offsets missing from the singular corner),
bricks with the three edges apart.

Tolerance: each entry within 1e-10 of the largest entry of its offset, the
accuracy of the two independent quadratures against each other.
"""
import numpy as np
import pytest

from oracle import physics, toeplitz
from tests.layout import unique_from_octant

pytestmark = pytest.mark.gpu

F = 298e6
K = physics.k0(F)


@pytest.fixture(scope="module")
def vie():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_02196_amd as v
    return v


@pytest.mark.parametrize("N,D", [((1, 1, 1), (0.003, 0.004, 0.006)), ((1, 1, 2), (0.005,) * 3),
                                 ((2, 1, 1), (0.006, 0.004, 0.003)), ((1, 4, 1), (0.005, 0.002, 0.004)),
                                 ((3, 1, 2), (0.004, 0.005, 0.006))])
def test_assembly_on_degenerate_grids(vie, N, D):
    print("assembly %s" % (N,), flush=True)
    c = vie.Context(0)
    c.set_grid(N, D, F)
    lib = c.get_toeplitz()
    ref = unique_from_octant(toeplitz.toeplitz_octant(N, D, K))
    assert np.isfinite(lib).all()
    for iz in range(N[2]):
        for iy in range(N[1]):
            for ix in range(N[0]):
                a, b = lib[:, iz, iy, ix], ref[:, iz, iy, ix]
                assert np.abs(a - b).max() <= 1e-10 * np.abs(b).max(), (ix, iy, iz)
