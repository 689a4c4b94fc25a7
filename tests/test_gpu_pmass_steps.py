"""That the Chebyshev iteration, and not the CG behind it, solves the particle mass system of
the paper-exact 2D M2P: the reported iterations are its step count, ceil(log3(4 / tol)), for
one to three fields on either side of its one-launch limit, and of its smallest size."""
import math

import numpy as np
import pytest

from test_gpu_pmass import problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nx,ny,ppc,F,tol", [(65, 64, 1, 1, 1e-14), (46, 45, 1, 2, 1e-10), (37, 37, 1, 3, 1e-14),
                                             (128, 128, 2, 2, 1e-12), (128, 129, 2, 3, 1e-14), (181, 182, 1, 1, 1e-8)])
def test_steps(nx, ny, ppc, F, tol):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_05258_amd import binding as B
    print(f"[pmass steps] {nx}x{ny} x {ppc} F={F} {tol}", flush=True)
    _, _, d = problem(B, nx, ny, ppc)
    nodal = np.random.default_rng(2).standard_normal((F, nx * ny))
    ctx = B.Context(0)
    try:
        _, rep = B.p2m_x2d_interpolate(ctx, d, B.X1D_MASS, torch.tensor(nodal, device="cuda"),
                                       opts=B.solve_opts(tol=tol, maxit=2000, max_refine=20, fp64=True))
        r = B.read_report(rep, F)
    finally:
        ctx.close()
    assert r.flags == 0 and list(r.iters) == [math.ceil(math.log(4 / tol) / math.log(3))] * F
    assert (r.refines == 1).all() and (r.rel_residual <= tol).all()
