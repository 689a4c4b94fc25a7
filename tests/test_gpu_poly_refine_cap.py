"""One correction allowed (max_refine = 1): the polynomial solve converges where the diagonal
solvers do, though its recurrence stalls on the way (random particles, 1.5 and 2 per cell) or
its scaled residual reaches the goal before the true one does (particles of very different
volumes), FP64 and FP32, alone and in a batch; max_refine = 0 still returns the start."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def case(n, m, ppc, seed, vol):
    g = np.random.default_rng(seed)
    N = int(n * m * ppc)
    x, y = np.minimum(g.random(N), 0.9999999), np.minimum(g.random(N), 0.9999999)
    return x, y, (g.uniform(0.03, 1.0, N) ** 4 / N if vol else None), np.sin(6 * x) * np.cos(6 * y)


@pytest.mark.parametrize("n,m,ppc,seed,vol,bits,tol", [(200, 200, 2, 7, 0, 64, 1e-11), (16, 200, 1.5, 3, 0, 64, 1e-6),
                                                       (64, 64, 2, 5, 0, 64, 1e-10), (100, 130, 4, 2, 1, 64, 1e-10),
                                                       (300, 300, 2, 9, 0, 64, 1e-9), (100, 130, 6, 2, 1, 32, 1e-5),
                                                       (600, 560, 2, 4, 0, 32, 1e-5), (150, 150, 2, 4, 0, 32, 1e-5)])
def test_converges(n, m, ppc, seed, vol, bits, tol):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_05258_amd import binding as B
    print(f"[refine cap] {n}x{m} {ppc} {vol} FP{bits}", flush=True)
    dt = torch.float64 if bits == 64 else torch.float32
    x, y, v, A = (None if a is None else torch.tensor(a, device="cuda").to(dt) for a in case(n, m, ppc, seed, vol))
    d = B.Particles(dim=2, nx=n, ny=m, lx=1.0, ly=1.0, x=x, y=y, vol=v)
    opts = B.solve_opts(tol=tol, inner_rtol=0.0, maxit=4000, max_refine=1, fp64=bits == 64)
    res = {}
    for mode in (B.SOLVER_AUTO, B.SOLVER_RESIDENT if bits == 32 else B.SOLVER_STREAMING):
        ctx = B.Context(0)
        try:
            ctx.set_solver(mode)
            out, rep = B.p2m_mass_assign(ctx, d, A[None], opts)
            res[mode] = r = B.read_report(rep, 1)
            print(f"  solver {mode}: {r.rel_residual[0]:.2e} after {r.iters[0]}, {r.refines[0]} residuals", flush=True)
            if mode == B.SOLVER_AUTO and bits == 32:
                outs, bt = B.p2m_mass_assign_batched(ctx, [d, d], [A[None], A[None]], opts)
                assert torch.equal(outs[1], out) and bt.reports()[1].refines[0] == r.refines[0]
            opts0 = B.solve_opts(tol=1e-12, inner_rtol=0.0, maxit=4000, max_refine=0, fp64=bits == 64)
            _, rep = B.p2m_mass_assign(ctx, d, A[None], opts0)
            assert B.read_report(rep, 1).refines[0] == 1 and B.read_report(rep, 1).iters[0] == 0
        finally:
            ctx.close()
    a, b = res.values()
    assert not (b.flags & B.FLAG_NOT_CONVERGED), "the case is to be one that the diagonal solver converges on"
    assert not (a.flags & B.FLAG_NOT_CONVERGED) and a.rel_residual[0] <= tol and a.refines[0] <= 4
