"""The particle mass system of the paper-exact 2D M2P (eq. (20)) through the Chebyshev
iteration at the edges of its forms: below and above the one-launch limit of 32,768 rows,
one to three fields, against the oracle (relative l2 <= 1e-11: the residual 1e-14 times
the condition of the matrix, 10 to 160).  Calls it leaves to the CG behind it (an
iteration cap below its step count, a wait that gives up) end as the CG ends them."""
import numpy as np
import pytest

from oracle import paper2d as p2
from paper_1610_05258_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_05258_amd import binding
    binding.lib()
    return binding


def problem(B, nx, ny, ppc):
    x, y = wl.stratified_2d(nx + 7 * ny, nx, ny, ppc, 1.0, 1.0)
    return x, y, B.Particles(dim=2, nx=nx, ny=ny, lx=1.0, ly=1.0, x=torch.tensor(x, device="cuda"),
                             y=torch.tensor(y, device="cuda"))


@pytest.mark.parametrize("nx,ny,ppc,F", [(64, 65, 1, 1), (40, 40, 1, 3), (128, 128, 2, 2), (113, 145, 2, 1),
                                         (96, 97, 4, 3)])
def test_particle_mass_solve(B, nx, ny, ppc, F):
    print(f"[pmass] {nx}x{ny} x {ppc}, F={F}", flush=True)
    x, y, d = problem(B, nx, ny, ppc)
    nodal = np.random.Generator(np.random.PCG64(5)).standard_normal((F, nx * ny))
    ctx = B.Context(0)
    try:
        out, rep = B.p2m_x2d_interpolate(ctx, d, B.X1D_MASS, torch.tensor(nodal, device="cuda"))
        r = B.read_report(rep, F)
        assert r.flags == 0 and (r.iters > 0).all() and (r.rel_residual <= 1e-14).all()
        want = p2.Paper2D(x, y, nx, ny, 1.0, 1.0).m2p_mass(nodal)
        got = out.cpu().numpy()
        for f in range(F):
            assert np.linalg.norm(got[f] - want[f]) <= 1e-11 * np.linalg.norm(want[f])
    finally:
        ctx.close()


def test_left_to_the_cg(B):
    x, y, d = problem(B, 96, 97, 4)
    nodal = torch.tensor(np.random.Generator(np.random.PCG64(6)).standard_normal((1, 96 * 97)), device="cuda")
    ctx = B.Context(0)
    try:
        out, rep = B.p2m_x2d_interpolate(ctx, d, B.X1D_MASS, nodal,
                                         opts=B.solve_opts(tol=1e-14, maxit=5, max_refine=3, fp64=True))
        r = B.read_report(rep, 1)
        assert r.flags & B.FLAG_NOT_CONVERGED and 0 < r.iters[0] <= 5
        _, _, small = problem(B, 70, 70, 1)
        ctx.set_solve_spin(-1)
        out, rep = B.p2m_x2d_interpolate(ctx, small, B.X1D_MASS, nodal[:, :4900].contiguous())
        r = B.read_report(rep, 1)
        assert r.flags & B.FLAG_BREAKDOWN and torch.isfinite(out).all()
    finally:
        ctx.close()
