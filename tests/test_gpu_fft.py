"""The 2D FFT solve of the circulant mesh systems at the edges of its lengths: small
sides, odd powers of two (one radix-2 pass), the largest power of two, Bluestein lengths
just above and at their limit, different kinds on the two sides; one to three fields.
Through the mass P2M of the paper-exact 2D methods, against the same right-hand side (the
lumped P2M times the cell area) solved by numpy's FFT in FP64: the system's condition
number is 4, so 1e-13."""
import numpy as np
import pytest

from paper_1610_05258_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nx,ny,F", [(8, 32, 2), (5, 64, 1), (128, 9, 3), (90, 90, 1),
                                     (96, 250, 2), (2048, 16, 1), (16, 2048, 1), (1023, 20, 1), (20, 1024, 2),
                                     (513, 40, 1), (40, 700, 1)])
def test_mass_p2m(nx, ny, F):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_05258_amd import binding as B
    print(f"[fft] {nx}x{ny} F={F}", flush=True)
    lx, ly = nx / 16.0, ny / 16.0   # square cells: stretched ones leave the stars' radius
    x, y = wl.stratified_2d(nx + ny, nx, ny, 4, lx, ly)
    A = np.random.Generator(np.random.PCG64(3)).standard_normal((F, x.size))
    ctx = B.Context(0)
    try:
        d = B.Particles(dim=2, nx=nx, ny=ny, lx=lx, ly=ly, x=torch.tensor(x, device="cuda"),
                        y=torch.tensor(y, device="cuda"))
        v = torch.tensor(A, device="cuda")
        out, rep = B.p2m_x2d_assign(ctx, d, B.X1D_MASS, v)
        r = B.read_report(rep, F)
        lumped, _ = B.p2m_x2d_assign(ctx, d, B.X1D_LUMPED, v)
        torch.cuda.synchronize()
        assert (r.iters == 0).all()
        assert r.flags == 0
        tx = 2 * np.pi * np.arange(nx)[None, :] / nx
        ty = 2 * np.pi * np.arange(ny)[:, None] / ny
        symbol = 0.5 + (np.cos(tx) + np.cos(ty) + np.cos(tx + ty)) / 6.0
        b = lumped.cpu().numpy().reshape(F, ny, nx)
        want = np.fft.ifft2(np.fft.fft2(b) / symbol).real.reshape(F, -1)
        got = out.cpu().numpy()
        for f in range(F):
            assert np.linalg.norm(got[f] - want[f]) <= 1e-13 * np.linalg.norm(want[f])
    finally:
        ctx.close()
