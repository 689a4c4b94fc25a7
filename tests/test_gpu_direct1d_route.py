"""The 1D solve by cyclic reduction where it has to run: from the FLIP start under AUTO and
RESIDENT_CHEB (which is AUTO where it does not apply), and after p2m_tune, whose plan must not
be slower than no plan.  That it is the reduction that solves, and not the conjugate gradients
behind it, shows in the iterations: none or one, at the edges of its forms too (the whole
period in a workgroup, overlapping windows, several of them), against at least 8 without it.
Orphans and both types with it."""
import numpy as np
import pytest

from test_gpu_direct1d import _case

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def solve(B, ctx, x, A, n, dt):
    d = B.Particles(dim=1, nx=n, ny=1, lx=1.0, ly=1.0, x=torch.tensor(x.astype(dt), device="cuda"))
    out, rep = B.p2m_mass_assign(ctx, d, torch.tensor(A.astype(dt), device="cuda"),
                                 B.solve_opts(tol=1e-12 if dt == "f8" else 1e-9, maxit=4000, max_refine=20, fp64=dt == "f8"))
    return out.clone(), B.read_report(rep, 2)


@pytest.mark.parametrize("n,ppc,empty,dt", [(2, 4, 0, "f8"), (3, 4, 0, "f8"), (17, 6, 0, "f8"), (64, 8, 0, "f8"),
                                            (64, 8, 1, "f8"), (255, 8, 0, "f4"), (256, 8, 0, "f8"), (257, 8, 0, "f8"),
                                            (511, 8, 0, "f8"), (513, 8, 0, "f4"), (1030, 8, 1, "f8"),
                                            (5000, 8, 0, "f8")])
def test_iterations(n, ppc, empty, dt):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_05258_amd import binding as B
    print(f"[direct1d route] {n} {ppc} {empty} {dt}", flush=True)
    x, A = _case(n, ppc, empty, n + ppc)
    got = {}
    for mode in (B.SOLVER_AUTO, B.SOLVER_RESIDENT_CHEB, B.SOLVER_STREAMING):
        ctx = B.Context(0)
        try:
            ctx.set_solver(mode)
            got[mode] = solve(B, ctx, x, A, n, dt)
        finally:
            ctx.close()
    (a, ra), (c, rc), (_, rs) = (got[m] for m in (B.SOLVER_AUTO, B.SOLVER_RESIDENT_CHEB, B.SOLVER_STREAMING))
    print(ra.iters, rs.iters, flush=True)
    assert ra.flags & ~B.FLAG_ORPHAN == 0 and (ra.iters <= 1).all()
    assert n < 17 or (rs.iters >= 8).all()
    assert torch.equal(a, c) and list(ra.iters) == list(rc.iters)


def test_tuned():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_05258_amd import binding as B
    x, A = _case(300, 8, 0, 4)
    ctx = B.Context(0)
    try:
        before, r0 = solve(B, ctx, x, A, 300, "f8")
        d = B.Particles(dim=1, nx=300, ny=1, lx=1.0, ly=1.0, x=torch.tensor(x, device="cuda"))
        plan, out, rep = B.p2m_tune(ctx, d, torch.tensor(A, device="cuda"),
                                    B.solve_opts(tol=1e-12, maxit=4000, max_refine=20, fp64=True))
        after, r1 = solve(B, ctx, x, A, 300, "f8")
        print(plan, flush=True)
        assert plan.solver == B.SOLVER_AUTO and list(r0.iters) == list(r1.iters) and (r1.iters <= 1).all()
        assert torch.equal(before, after)
    finally:
        ctx.close()
