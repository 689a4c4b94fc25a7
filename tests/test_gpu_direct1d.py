"""The 1D mass assignment by cyclic reduction: periods shorter than a distance, the whole
period in one workgroup (up to 256 nodes), the first sizes of the overlapping windows and
several of them; FP32 and FP64; orphan nodes (empty cells); a matrix without full rank,
where the reduction gives way to the conjugate gradients.  Against a dense FP64 solve
of the same particles; the bound is the requested residual times the condition number."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _case(n, ppc, empty, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    c = np.repeat(np.arange(n), ppc)
    if empty:
        c = c[(c % 7 != 2) & (c % 7 != 3)]
    x = (c + rng.uniform(0.0, 1.0, c.size)) / n
    return np.minimum(x, np.nextafter(1.0, 0.0)), rng.standard_normal((2, c.size))


def _dense(n, x, A, dt):
    x = x.astype(dt).astype(np.float64)
    i = np.minimum(np.floor(x * n).astype(int), n - 1)
    a = x * n - i
    P = np.zeros((x.size, n))
    np.add.at(P, (np.arange(x.size), i), 1.0 - a)
    np.add.at(P, (np.arange(x.size), (i + 1) % n), a)
    return P.T @ P, P.T @ A.T.astype(np.float64)


@pytest.mark.parametrize("n,ppc,empty,dt", [(2, 4, 0, "f8"), (3, 4, 0, "f8"), (17, 3, 0, "f8"), (64, 4, 0, "f8"),
                                            (64, 4, 1, "f8"), (255, 5, 0, "f4"), (256, 3, 0, "f8"),
                                            (257, 3, 0, "f8"), (300, 6, 1, "f4"), (511, 3, 0, "f8"),
                                            (513, 4, 0, "f8"), (1030, 3, 1, "f8"), (1500, 8, 0, "f4")])
def test_mass_1d(n, ppc, empty, dt):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_05258_amd import binding as B
    print(f"[direct1d] n={n} ppc={ppc} empty={empty} {dt}", flush=True)
    dt = np.dtype(dt)
    x, A = _case(n, ppc, empty, n + ppc)
    A = A.astype(dt)
    M, b = _dense(n, x, A, dt)
    live = np.diag(M) > 0
    lam = np.linalg.eigvalsh(M[np.ix_(live, live)])
    kappa = lam[-1] / lam[0]
    tol = 1e-13 if dt == np.float64 else 1e-9
    ctx = B.Context(0)
    try:
        d = B.Particles(dim=1, nx=n, ny=1, lx=1.0, ly=1.0, x=torch.tensor(x.astype(dt), device="cuda"))
        opts = B.solve_opts(tol=tol, maxit=4000, max_refine=20, fp64=dt == np.float64)
        out, rep = B.p2m_mass_assign(ctx, d, torch.tensor(A, device="cuda"), opts)
        r = B.read_report(rep, 2)
        assert not (r.flags & (B.FLAG_NOT_CONVERGED | B.FLAG_BREAKDOWN))
        assert (r.rel_residual <= tol).all()
        got = out.cpu().numpy().astype(np.float64)
        want = np.zeros((2, n))
        want[:, live] = np.linalg.solve(M[np.ix_(live, live)], b[live]).T
        assert not got[:, ~live].any()
        # residual, assembly (weights and sums in the type) and the result's rounding
        eps = np.finfo(dt).eps
        bound = kappa * (tol + 32 * eps) + eps
        for f in range(2):
            err = np.linalg.norm(got[f] - want[f]) / np.linalg.norm(want[f])
            print(f"  kappa {kappa:.1f} iters {r.iters[f]} err {err:.2e} bound {bound:.2e}", flush=True)
            assert err <= bound
    finally:
        ctx.close()


def test_mass_1d_rank_deficient():
    """One particle to two cells: half the rank.  The same answer as the conjugate
    gradients' own (the streaming solver), which stay in the start's affine space."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_05258_amd import binding as B
    n = 128
    x = (np.arange(0, n, 2) + 0.37) / n
    A = np.random.Generator(np.random.PCG64(5)).standard_normal((1, x.size))
    outs = []
    for mode in (B.SOLVER_AUTO, B.SOLVER_STREAMING):
        ctx = B.Context(0)
        try:
            ctx.set_solver(mode)
            d = B.Particles(dim=1, nx=n, ny=1, lx=1.0, ly=1.0, x=torch.tensor(x, device="cuda"))
            out, rep = B.p2m_mass_assign(ctx, d, torch.tensor(A, device="cuda"),
                                         B.solve_opts(tol=1e-12, maxit=1000, max_refine=5, fp64=True))
            outs.append((out.cpu().numpy(), B.read_report(rep, 1)))
        finally:
            ctx.close()
    assert np.array_equal(outs[0][0], outs[1][0]) and outs[0][1].flags == outs[1][1].flags
