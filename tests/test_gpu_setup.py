"""GPU parity of the operator set-up at the edges of its kernels: grids of
one voxel, one row or one plane (offsets missing from the singular corner),
bricks with the three edges apart.

Tolerance: each entry within 1e-10 of the largest entry of its offset, the
accuracy of the two independent quadratures against each other.
"""
import threading

import numpy as np
import pytest

import vie_inputs as vi
from oracle import physics, toeplitz
from tests.layout import unique_from_octant, vox_to_lib

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


@pytest.mark.parametrize("N", [(60, 24, 20), (50, 64, 48), (19, 120, 70), (18, 30, 40)])
def test_far_offsets_do_not_depend_on_the_run(vie, N):
    """The tensors of an offset depend on it alone; in a large grid the far
    offsets are evaluated in runs along x (of 2 to 16, with remainders, from
    the row's start or from where the band begins), in a grid of one plane
    one by one.  The sums are the same up to their order: 1e3 terms in FP64,
    1e-12 of the largest entry."""
    D = (0.003, 0.004, 0.005)
    print("far runs %s" % (N,), flush=True)
    c = vie.Context(0)
    c.set_grid(N, D, F)
    big = c.get_toeplitz()
    for n, part in (((N[0], N[1], 1), big[:, :1]), ((N[0], 1, N[2]), big[:, :, :1])):
        c.set_grid(n, D, F)
        ref = c.get_toeplitz()
        assert np.isfinite(part).all()
        assert (np.abs(part - ref).max(axis=0) <= 1e-12 * np.abs(ref).max(axis=0)).all(), n


def test_setup_beside_captured_solves(vie):
    """Graph captures of one thread's solves and the grid set-ups of another
    do not disturb each other: every call succeeds, every solution has the
    same bits."""
    import torch
    N, D = (6, 6, 6), (0.005,) * 3
    e, s = (vox_to_lib(v) for v in vi.sphere(N, D, 0.012, 50.0, 0.7))
    streams = [torch.cuda.Stream() for _ in range(2)]
    a, b = (vie.Context(0, st) for st in streams)
    a.set_grid(N, D, F)
    a.set_contrast(e, s)
    et = torch.empty(a.vec_shape(1), dtype=torch.complex128, device="cuda")
    x = torch.empty_like(et)
    a.incident_planewave(et)
    torch.cuda.synchronize()
    stop, errors, sols = threading.Event(), [], []

    def setups():
        try:
            while not stop.is_set():
                b.set_grid((5, 4, 6), D, F)
        except Exception as err:   # reported by the test
            errors.append(err)

    t = threading.Thread(target=setups)
    t.start()
    try:
        for _ in range(30):
            a.set_contrast(e, s)   # forgets the captured steps
            for _ in range(3):     # plain, captured, replayed
                code, _ = a.solve(et, x, mode=vie.SOLVE_FP32_IR, tol=1e-8, restart=12, graph=1)
                assert code == vie.VIE_OK
                with torch.cuda.stream(streams[0]):
                    sols.append(x.cpu().numpy())
    finally:
        stop.set()
        t.join()
    assert not errors, errors
    assert all(np.array_equal(v, sols[0]) for v in sols)


def test_grid_that_does_not_fit_leaves_the_context_usable(vie):
    """A grid whose tensors exceed the device's memory is refused after its
    first uploads are queued; the context then takes the next grid, with the
    bits of a context that never saw the other."""
    import torch
    N, D = (5, 4, 6), (0.003, 0.004, 0.005)
    print("grid beyond memory", flush=True)
    a, b = vie.Context(0), vie.Context(0)
    for _ in range(2):
        with pytest.raises(vie.VieError) as err:
            a.set_grid((2000, 2000, 2000), D, F)   # 7.7 TB of tensors
        assert err.value.code == vie.VIE_ENOMEM
    for c in (a, b):
        c.set_grid(N, D, F)
    assert np.array_equal(a.get_toeplitz(), b.get_toeplitz())
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.view_as_complex(torch.randn(a.vec_shape(1) + (2,), generator=g, device="cuda", dtype=torch.float64))
    ya, yb = torch.empty_like(x), torch.empty_like(x)
    for c, y in ((a, ya), (b, yb)):
        c.apply(x, y, op=vie.OP_N)
    assert torch.equal(ya, yb)
