"""GPU parity of the strided passes (along y and z) at every length they are
compiled for, against torch's FFT in complex128 on the same block tensors.

Tolerances as derived in test_gpu_xpass.py: 50 eps in the 2-norm.
"""
import pytest

from tests.test_gpu_xpass import F, LENGTHS, reference, torch, vie  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", LENGTHS + [768])
def test_every_length(vie, torch, M):  # noqa: F811
    """Full and ragged pencils, an inner extent that is no multiple of a tile
    (and one below it), the plain epilogue and the one with x and contrast."""
    for N, axis in (((5, M // 2, 2), 1), ((17, 2, max(1, M // 2 - 3)), 2)):
        c = vie.Context(0)
        fft = [2 * n for n in N]
        fft[0] = 16 if N[0] == 5 else 36
        fft[axis] = M
        c.set_grid(N, (0.003, 0.004, 0.005), F, fft_size=fft)
        T = torch.from_numpy(c.get_toeplitz()).cuda()
        g = torch.Generator(device="cuda").manual_seed(M)
        x = torch.view_as_complex(torch.randn(c.vec_shape(2) + (2,), generator=g, device="cuda", dtype=torch.float64))
        shape = x.shape[2:]
        eps_r = torch.rand(shape, generator=g, device="cuda", dtype=torch.float64) * 40 + 1
        sig = torch.rand(shape, generator=g, device="cuda", dtype=torch.float64)
        c.set_contrast(eps_r, sig)
        er = torch.complex(eps_r, -sig / (2 * 3.141592653589793 * F * 8.8541878128e-12))
        dv = 0.003 * 0.004 * 0.005
        G = torch.tensor([dv, dv / 12, dv / 12, dv / 12] * 3, device="cuda", dtype=torch.float64).view(1, 12, 1, 1, 1)
        for dtype, eps in ((torch.complex64, 6e-8), (torch.complex128, 1.2e-16)):
            print("M %d N %s %s" % (M, N, dtype), flush=True)
            xd = x.to(dtype).contiguous()
            w = reference(torch, T, xd)
            for op, r in ((vie.OP_N, w), (vie.OP_A, er * G * xd - (er - 1) * w)):
                y = torch.full_like(xd, float("nan"))
                c.apply(xd, y, op=op)
                err = ((y.to(torch.complex128) - r).norm() / r.norm()).item()
                assert err < 50 * eps, (N, dtype, op, err)


@pytest.mark.parametrize("M", [2, 6, 270, 288, 300, 768])
def test_every_tile_of_the_lengths_with_a_choice(vie, torch, M):  # noqa: F811
    """The lengths whose tile the caller picks (the run-time kernel's and 768;
    every other length has one kernel with its own tile): each accepted tile
    gives the product, in z and in y."""
    for N, axis in (((5, max(1, M // 2), 2), 1), ((17, 2, max(1, M // 2 - 3)), 2)):
        c = vie.Context(0)
        fft = [2 * n for n in N]
        fft[0] = 16 if N[0] == 5 else 36
        fft[axis] = M
        c.set_grid(N, (0.003, 0.004, 0.005), F, fft_size=fft)
        T = torch.from_numpy(c.get_toeplitz()).cuda()
        g = torch.Generator(device="cuda").manual_seed(M)
        x = torch.view_as_complex(torch.randn(c.vec_shape(2) + (2,), generator=g, device="cuda", dtype=torch.float64))
        for dtype, prec, eps in ((torch.complex64, vie.C64, 6e-8), (torch.complex128, vie.C128, 1.2e-16)):
            xd = x.to(dtype).contiguous()
            ref = reference(torch, T, xd)
            ran = []
            for tile in (1, 2, 4, 8, 16, 32):
                shape = dict(variant=6, sib_blocks=1, tile_z=8, tile_y=8)
                shape["tile_y" if axis == 1 else "tile_z"] = tile
                try:
                    c.set_tuning(shape, prec, 2)
                except vie.VieError:
                    continue   # does not fit LDS
                ran.append(tile)
                y = torch.full_like(xd, float("nan"))
                c.apply(xd, y, op=vie.OP_N)
                err = ((y.to(torch.complex128) - ref).norm() / ref.norm()).item()
                assert err < 50 * eps, (N, dtype, tile, err)
            print("M %d N %s %s tiles %s" % (M, N, dtype, ran), flush=True)
            assert len(ran) >= 3
