"""GPU parity of the matrix-core x pass (variant 6) against the other
variants and torch's FFT, at every length along x that it is compiled for.

The reference is the circulant product formed with torch in complex128 from
the library's own block tensors, so that only the product is compared.
Tolerances from the arithmetic: a transform of length M and a sum of 12
terms in precision eps leave a relative error of about eps log2(M^3); 50 eps
(3e-6 complex64 in the 2-norm at eps = 6e-8, 6e-15 complex128) is several
times that at the largest M here.
"""
import numpy as np
import pytest

from tests.layout import UNIQUE_AB

pytestmark = pytest.mark.gpu

F = 298e6


def _smooth(n):
    for p in (2, 3, 5):
        while n % p == 0:
            n //= p
    return n == 1


# every even length 8 ... 256 made of 2, 3 and 5, and the three above
LENGTHS = [n for n in range(8, 257, 2) if _smooth(n)] + [320, 384, 512]


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


@pytest.fixture(scope="module")
def vie(torch):
    import paper_1902_02196_amd as v
    return v


def _sign(axis, a):
    p, l = divmod(a, 4)
    return (-1) ** ((p == axis) + (l == axis + 1))


def _unique_index():
    """(unique entry, sign) of every (a, b)."""
    u = {ab: e for e, ab in enumerate(UNIQUE_AB)}
    out = {}
    for a in range(12):
        for b in range(12):
            (p, l), (q, m) = divmod(a, 4), divmod(b, 4)
            k = (4 * min(p, q) + min(l, m), 4 * max(p, q) + max(l, m))
            out[a, b] = u[k], -1 if l > m == 0 else 1
    return out


def reference(torch, T, x):
    """N x by the circulant of 2 N per axis, complex128; T [60, Nz, Ny, Nx], x [n, 12, Nz, Ny, Nx]."""
    Nz, Ny, Nx = T.shape[1:]
    M = (2 * Nz, 2 * Ny, 2 * Nx)
    spec = []
    for a, b in UNIQUE_AB:
        C = torch.zeros(M, dtype=torch.complex128, device="cuda")
        t = T[len(spec)]
        for dim, axis, n in ((0, 2, Nz), (1, 1, Ny), (2, 0, Nx)):
            mirror = _sign(axis, a) * _sign(axis, b) * t.narrow(dim, 1, n - 1).flip(dim)
            gap = torch.zeros_like(t.narrow(dim, 0, 1))
            t = torch.cat([t, gap, mirror], dim)
        C.copy_(t)
        spec.append(torch.fft.fftn(C))
    X = torch.fft.fftn(x.to(torch.complex128), s=M, dim=(2, 3, 4))
    idx = _unique_index()
    Y = torch.zeros_like(X)
    for (a, b), (e, s) in idx.items():
        Y[:, a] += s * spec[e] * X[:, b]
    return torch.fft.ifftn(Y, dim=(2, 3, 4))[:, :, :Nz, :Ny, :Nx]


@pytest.mark.parametrize("M", LENGTHS)
def test_every_length(vie, torch, M):
    """Ragged rows (Nx below M / 2), odd and even extents in y and z (single
    and paired siblings), two right-hand sides, both precisions."""
    for N in ((M // 2, 3, 2), (max(1, M // 2 - 3), 2, 3)):
        c = vie.Context(0)
        c.set_grid(N, (0.003, 0.004, 0.005), F, fft_size=(M, 2 * N[1], 2 * N[2]))
        T = torch.from_numpy(c.get_toeplitz()).cuda()
        g = torch.Generator(device="cuda").manual_seed(M)
        x = torch.view_as_complex(torch.randn(c.vec_shape(2) + (2,), generator=g, device="cuda", dtype=torch.float64))
        ref = reference(torch, T, x)
        for prec, dtype, eps in ((vie.C64, torch.complex64, 6e-8), (vie.C128, torch.complex128, 1.2e-16)):
            print("M %d N %s %s" % (M, N, dtype), flush=True)
            try:
                c.set_tuning(dict(variant=6, sib_blocks=1, tile_z=8, tile_y=8), prec, 2)
            except vie.VieError:
                assert prec == vie.C128 and M == 512   # its rows do not fit LDS
                continue
            xd = x.to(dtype).contiguous()
            y = torch.full_like(xd, float("nan"))
            c.apply(xd, y, op=vie.OP_N)
            r = ref if dtype == torch.complex128 else reference(torch, T, xd)
            err = ((y.to(torch.complex128) - r).norm() / r.norm()).item()
            assert err < 50 * eps, (N, dtype, err)
