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
