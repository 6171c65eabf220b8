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


def _circulant(torch, T, members, reflect, x):
    """The 12 x 12 block circulant product, complex128: T [n, Nz, Ny, Nx] unique
    tensors, members {(a, b): (tensor, sign)}, reflect(tensor, axis) the sign of
    its mirror, x [nrhs, 12, Nz, Ny, Nx]."""
    Nz, Ny, Nx = T.shape[1:]
    spec = []
    for e in range(T.shape[0]):
        t = T[e]
        for dim, axis, n in ((0, 2, Nz), (1, 1, Ny), (2, 0, Nx)):
            mirror = reflect(e, axis) * t.narrow(dim, 1, n - 1).flip(dim)
            t = torch.cat([t, torch.zeros_like(t.narrow(dim, 0, 1)), mirror], dim)
        spec.append(torch.fft.fftn(t))
    X = torch.fft.fftn(x.to(torch.complex128), s=(2 * Nz, 2 * Ny, 2 * Nx), dim=(2, 3, 4))
    Y = torch.zeros_like(X)
    for (a, b), (e, s) in members.items():
        Y[:, a] += s * spec[e] * X[:, b]
    return torch.fft.ifftn(Y, dim=(2, 3, 4))[:, :, :Nz, :Ny, :Nx]


def reference(torch, T, x):
    """N x from the 60 block tensors."""
    return _circulant(torch, T, _unique_index(),
                      lambda e, i: _sign(i, UNIQUE_AB[e][0]) * _sign(i, UNIQUE_AB[e][1]), x)


def curl_reference(torch, TK, x):
    """K x from the 30 curl tensors: K^{pl,ql'} = eps_pkq Q_k^{ll'}, mirrored
    with -sigma_i(a) sigma_i(b)."""
    members, rep = {}, {}
    for (a, b), (e, s) in _unique_index().items():
        p, q = a // 4, b // 4
        if p != q:
            k = 3 - p - q
            members[a, b] = (10 * k + e % 10, s * (1 if (k - p) % 3 == 1 else -1))
            rep[10 * k + e % 10] = (a, b)
    return _circulant(torch, TK, members, lambda e, i: -_sign(i, rep[e][0]) * _sign(i, rep[e][1]), x)


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
            if prec == vie.C128 and M in (240, 250):
                with pytest.raises(vie.VieError):   # lengths the complex128 product has never taken
                    c.apply(x, torch.empty_like(x), op=vie.OP_N)
                continue
            xd = x.to(dtype).contiguous()
            y = torch.full_like(xd, float("nan"))
            c.apply(xd, y, op=vie.OP_N)
            r = ref if dtype == torch.complex128 else reference(torch, T, xd)
            err = ((y.to(torch.complex128) - r).norm() / r.norm()).item()
            assert err < 50 * eps, (N, dtype, err)


@pytest.mark.parametrize("M", [8, 16, 32, 64, 96, 128, 160, 192, 256, 320, 384, 512])
def test_pwc_every_length(vie, torch, M):
    """The PWC product (the pulse functions alone, a = 4 p) at every length it
    takes: ragged rows, single and paired siblings in y and z, two right-hand
    sides, both precisions."""
    for N in ((M // 2, 3, 2), (max(1, M // 2 - 3), 2, 3)):
        c = vie.Context(0)
        c.set_grid(N, (0.003, 0.004, 0.005), F, fft_size=(M, 2 * N[1], 2 * N[2]))
        Th = c.get_toeplitz()
        T = torch.from_numpy(Th).cuda()
        c.set_basis(3)
        c.set_toeplitz(Th)
        x = _random(torch, torch.Generator(device="cuda").manual_seed(M + 1), c.vec_shape(2))
        for dtype, eps in ((torch.complex64, 6e-8), (torch.complex128, 1.2e-16)):
            print("M %d N %s %s" % (M, N, dtype), flush=True)
            xd = x.to(dtype).contiguous()
            y = torch.full_like(xd, float("nan"))
            c.apply(xd, y, op=vie.OP_N)
            x12 = torch.zeros((2, 12) + tuple(xd.shape[2:]), dtype=torch.complex128, device="cuda")
            x12[:, ::4] = xd
            r = reference(torch, T, x12)[:, ::4]
            err = ((y.to(torch.complex128) - r).norm() / r.norm()).item()
            assert err < 50 * eps, (N, dtype, err)


def _random(torch, g, shape):
    return torch.view_as_complex(torch.randn(tuple(shape) + (2,), generator=g, device="cuda", dtype=torch.float64))


@pytest.mark.parametrize("M", [n for n in LENGTHS if n <= 256])
def test_curl_and_coupled_products(vie, torch, M):
    """The curl operator's product (magnetic field, complex128) and the coupled
    sums of the J-M product (A x, both precisions) at every length they take."""
    w = 2 * np.pi * F
    ce, cm = 1j * w * 8.8541878128e-12, 1j * w * 1.25663706212e-6
    dv = 0.003 * 0.004 * 0.005
    for N in ((M // 2, 3, 2), (max(1, M // 2 - 3), 2, 3)):
        g = torch.Generator(device="cuda").manual_seed(M)
        fft = (M, 2 * N[1], 2 * N[2])
        c = vie.Context(0)
        c.set_grid(N, (0.003, 0.004, 0.005), F, fft_size=fft)
        T = torch.from_numpy(c.get_toeplitz()).cuda()
        TK = torch.from_numpy(c.get_curl_toeplitz()).cuda()
        G = torch.tensor([dv, dv / 12, dv / 12, dv / 12] * 3, device="cuda", dtype=torch.float64).view(1, 12, 1, 1, 1)
        x, ht = _random(torch, g, c.vec_shape(2)), torch.zeros(c.vec_shape(2), dtype=torch.complex128, device="cuda")
        h = torch.full_like(x, float("nan"))
        print("M %d N %s curl" % (M, N), flush=True)
        c.magnetic_field(ht, x, h)
        r = curl_reference(torch, TK, x) / G
        err = ((h - r).norm() / r.norm()).item()
        assert err < 50 * 1.2e-16, (N, err)

        c = vie.Context(0)
        c.set_basis(24)
        c.set_grid(N, (0.003, 0.004, 0.005), F, fft_size=fft)
        shape = x.shape[2:]
        eps, sig, mu, mi = (torch.rand(shape, generator=g, device="cuda", dtype=torch.float64) for _ in range(4))
        eps, mu = 1 + 40 * eps, 1 + 2 * mu
        c.set_contrast(eps, sig)
        c.set_magnetic_contrast(mu.cpu().numpy(), mi.cpu().numpy())
        er, mr = torch.complex(eps, -sig / (w * 8.8541878128e-12)), torch.complex(mu, -mi)
        x = _random(torch, g, c.vec_shape(2))
        x[:, 12:] *= 1e-3   # magnetic currents are of another size: both couplings count
        for dtype, e in ((torch.complex64, 6e-8), (torch.complex128, 1.2e-16)):
            print("M %d N %s J-M %s" % (M, N, dtype), flush=True)
            if dtype == torch.complex128 and M in (240, 250):
                continue   # complex128 takes no PWL product of these lengths
            xd = x.to(dtype).contiguous()
            y = torch.full_like(xd, float("nan"))
            c.apply(xd, y, op=vie.OP_A)
            xj, xm = xd[:, :12].to(torch.complex128), xd[:, 12:].to(torch.complex128)
            rj = er * G * xj - (er - 1) * (reference(torch, T, xj) - ce * curl_reference(torch, TK, xm))
            rm = mr * G * xm - (mr - 1) * (reference(torch, T, xm) + cm * curl_reference(torch, TK, xj))
            for part, r in ((y[:, :12], rj), (y[:, 12:], rm)):
                err = ((part.to(torch.complex128) - r).norm() / r.norm()).item()
                assert err < 50 * e, (N, dtype, err)


@pytest.mark.parametrize("nx", [1, 2, 3, 45])
def test_autotuned_shape_can_be_installed(vie, torch, nx):
    """x lengths of the run-time kernel (2, 4, 6) and one of the matrix-core
    kernel alone (90): what the autotuner returns is a shape vie_set_tuning
    takes, and gives the product it gave."""
    c = vie.Context(0)
    c.set_grid((nx, 3, 4), (0.003, 0.004, 0.005), F)
    x = _random(torch, torch.Generator(device="cuda").manual_seed(nx), c.vec_shape(2))
    for prec, dtype in ((vie.C64, torch.complex64), (vie.C128, torch.complex128)):
        choice, _ = c.autotune(prec, 2)
        print("nx %d %s %s" % (nx, dtype, choice), flush=True)
        xd = x.to(dtype).contiguous()
        ya, yb = torch.empty_like(xd), torch.full_like(xd, float("nan"))
        c.apply(xd, ya, op=vie.OP_N)
        c.set_tuning(choice, prec, 2)
        c.apply(xd, yb, op=vie.OP_N)
        assert torch.equal(ya, yb)


@pytest.mark.parametrize("M", [320, 384, 512])
def test_coupled_products_of_long_rows(vie, torch, M):
    """The coupled sums of the J-M product (A x, complex64) at the lengths
    above 256 that have a kernel, full and ragged rows."""
    w = 2 * np.pi * F
    ce, cm = 1j * w * 8.8541878128e-12, 1j * w * 1.25663706212e-6
    dv = 0.003 * 0.004 * 0.005
    for N in ((M // 2, 3, 2), (M // 2 - 3, 2, 3)):
        g = torch.Generator(device="cuda").manual_seed(M)
        c = vie.Context(0)
        c.set_basis(24)
        c.set_grid(N, (0.003, 0.004, 0.005), F, fft_size=(M, 2 * N[1], 2 * N[2]))
        T = torch.from_numpy(c.get_toeplitz()).cuda()
        TK = torch.from_numpy(c.get_curl_toeplitz()).cuda()
        G = torch.tensor([dv, dv / 12, dv / 12, dv / 12] * 3, device="cuda", dtype=torch.float64).view(1, 12, 1, 1, 1)
        x = _random(torch, g, c.vec_shape(2)).to(torch.complex64)
        x[:, 12:] *= 1e-3   # magnetic currents are of another size: both couplings count
        shape = x.shape[2:]
        eps, sig, mu, mi = (torch.rand(shape, generator=g, device="cuda", dtype=torch.float64) for _ in range(4))
        eps, mu = 1 + 40 * eps, 1 + 2 * mu
        c.set_contrast(eps, sig)
        c.set_magnetic_contrast(mu.cpu().numpy(), mi.cpu().numpy())
        er, mr = torch.complex(eps, -sig / (w * 8.8541878128e-12)), torch.complex(mu, -mi)
        print("M %d N %s J-M" % (M, N), flush=True)
        y = torch.full_like(x, float("nan"))
        c.apply(x, y, op=vie.OP_A)
        xj, xm = x[:, :12].to(torch.complex128), x[:, 12:].to(torch.complex128)
        rj = er * G * xj - (er - 1) * (reference(torch, T, xj) - ce * curl_reference(torch, TK, xm))
        rm = mr * G * xm - (mr - 1) * (reference(torch, T, xm) + cm * curl_reference(torch, TK, xj))
        for part, r in ((y[:, :12], rj), (y[:, 12:], rm)):
            err = ((part.to(torch.complex128) - r).norm() / r.norm()).item()
            assert err < 50 * 6e-8, (N, err)


@pytest.mark.parametrize("N", [(16, 12, 10), (24, 20, 12), (5, 3, 6)])
def test_matrix_core_shape_matches_oracle(vie, torch, N):
    """Variant 6, installed explicitly, against the oracle's FFT product from
    its own blocks, three right-hand sides (the other variants:
    test_every_launch_shape_matches_oracle)."""
    import vie_inputs as vi
    from oracle import matvec, physics, toeplitz
    from tests.layout import relerr, unique_from_full, vec_from_lib, vec_to_lib
    D = (0.005, 0.004, 0.006)
    T = toeplitz.toeplitz_full(N, D, physics.k0(F))
    c = vie.Context(0)
    c.set_grid(N, D, F)
    c.set_toeplitz(unique_from_full(T))
    xs = [vi.complex_normal(40 + r, (12,) + N) for r in range(3)]
    Ch = matvec.circulant_spectrum(T, tuple(2 * n for n in N))
    x = torch.from_numpy(np.stack([vec_to_lib(v) for v in xs]))
    for dtype, prec, tile, tol in ((torch.complex64, vie.C64, 16, 1e-5), (torch.complex128, vie.C128, 8, 1e-11)):
        print("N %s %s" % (N, dtype), flush=True)
        xd = x.to("cuda", dtype)
        y = torch.full_like(xd, float("nan"))
        c.set_tuning(dict(variant=6, sib_blocks=1, tile_z=tile, tile_y=tile), prec, 3)
        c.apply(xd, y, op=vie.OP_N)
        for r in range(3):
            assert relerr(vec_from_lib(y[r].cpu().numpy()), matvec.fft_N(Ch, xs[r])) < tol, (dtype, r)


@pytest.mark.parametrize("M", [96, 128, 160, 192, 320, 384, 512])
def test_default_x_pass_of_thin_and_thick_grids(vie, torch, M):
    """Without a named shape, thin grids (few octant rows) and thicker ones run
    different x passes at these lengths: both sides of the rules, PWL and PWC
    in both precisions, and a vector's bits do not depend on its batch."""
    for N in ((M // 2 - 3, 3, 2), (M // 2, 6, 10), (M // 2 - 1, 15, 16), (M // 2 - 3, 18, 20)):
        c = vie.Context(0)
        c.set_grid(N, (0.003, 0.004, 0.005), F, fft_size=(M, 2 * N[1], 2 * N[2]))
        Th = c.get_toeplitz()
        T = torch.from_numpy(Th).cuda()
        g = torch.Generator(device="cuda").manual_seed(M)
        x = _random(torch, g, c.vec_shape(3))
        ref = reference(torch, T, x[:1])
        x3 = x[:, ::4].contiguous()
        x12 = torch.zeros_like(x[:1])
        x12[:, ::4] = x3[:1]
        ref3 = reference(torch, T, x12)[:, ::4]
        for basis, v, r in ((12, x, ref), (3, x3, ref3)):
            c.set_basis(basis)
            for dtype, eps in ((torch.complex64, 6e-8), (torch.complex128, 1.2e-16)):
                print("M %d N %s basis %d %s" % (M, N, basis, dtype), flush=True)
                vd = v.to(dtype).contiguous()
                y, one = torch.full_like(vd, float("nan")), torch.full_like(vd[:1], float("nan"))
                c.apply(vd, y, op=vie.OP_N)
                c.apply(vd[:1].contiguous(), one, op=vie.OP_N)
                assert torch.equal(y[:1], one), (N, basis, dtype)
                err = ((one.to(torch.complex128) - r).norm() / r.norm()).item()
                # the inputs' own rounding to complex64 adds one eps
                assert err < 51 * eps, (N, basis, dtype, err)
