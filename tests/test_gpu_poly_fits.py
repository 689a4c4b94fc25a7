"""The polynomial solve runs wherever the header says it does, not where its state happens to
fit the other solvers' workspace: FP64 meshes of one tile, of a few nodes across and with a
tile of a few nodes' remainder, tall FP32 strips.  Its iterations are at most half of the
diagonal solver's to the same residual (a polynomial of degree 2 or 4 in each), its result
within the other tile tests' bounds (FP64 1e-12, FP32 1e-6) of the FP64 oracle.  A problem
that just fits the static scratch is still taken by the call that uses it, with the bits of
the call that is given a workspace."""
import ctypes

import numpy as np
import pytest

from oracle import metrics
from test_gpu_poly import problem, reference

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(9, 5, 1, 64), (9, 9, 1, 64), (13, 11, 2, 64), (33, 36, 2, 64), (37, 34, 3, 64), (6, 400, 1, 64),
          (400, 6, 3, 64), (3, 16500, 1, 32)]


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_05258_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("nx,ny,F,bits", SHAPES)
def test_runs(B, nx, ny, F, bits):
    print(f"[poly fits] {nx}x{ny} F={F} FP{bits}", flush=True)
    prob, vals = problem(nx, ny, 5, F, np.float32 if bits == 32 else np.float64)
    its = []
    for mode in (B.SOLVER_AUTO, B.SOLVER_STREAMING):
        ctx = B.Context(0)
        try:
            ctx.set_solver(mode)
            opts = B.solve_opts(tol=1e-8 if bits == 32 else 1e-13, maxit=2000, max_refine=20, fp64=bits == 64)
            out, rep = B.p2m_mass_assign(ctx, B.particles_from(prob), torch.as_tensor(vals).cuda(), opts)
            torch.cuda.synchronize()
            r = B.read_report(rep, F)
            assert not (r.flags & (B.FLAG_BREAKDOWN | B.FLAG_NOT_CONVERGED))
            its.append(r.iters)
            for f, ref in enumerate(reference(prob, vals)):
                e = metrics.rel_l2(out[f].cpu().numpy().astype(np.float64), ref)
                assert e <= (1e-6 if bits == 32 else 1e-12), (mode, f, e)
        finally:
            ctx.close()
    assert (2 * its[0] <= its[1]).all(), its


def test_static_scratch_edge(B):
    """33 x 36 FP64, F = 2: the most particles whose workspace fits the static scratch."""
    nx, ny, F = 33, 36, 2
    ctx = B.Context(0)
    try:
        def size(np_):
            p = B.CProblem(2, nx, ny, B.P2M_F64, 1.0, 1.0, np_, 256, 256, None)
            n = ctypes.c_size_t()
            assert B.lib().p2m_workspace_size(ctx.handle, ctypes.byref(p), F, ctypes.byref(n)) == 0
            return n.value
        lo, hi = 1000, 10_000_000
        assert size(lo) <= B.SCRATCH_BYTES < size(hi)
        while hi - lo > 1:
            mid = (lo + hi) // 2
            lo, hi = (mid, hi) if size(mid) <= B.SCRATCH_BYTES else (lo, mid)
        # 12 bytes a particle in the layout: key, rank, perm, in units of 256 bytes, so the
        # edge lies where it lay without the solve's added bytes
        assert B.SCRATCH_BYTES - size(lo) < 3 * 256
        g = np.random.default_rng(1)
        x, y = (torch.tensor(np.minimum(g.random(lo), 0.9999999), device="cuda") for _ in range(2))
        d = B.Particles(dim=2, nx=nx, ny=ny, lx=1.0, ly=1.0, x=x, y=y)
        v = torch.stack([torch.sin(6 * x), y])
        opts = B.solve_opts(tol=1e-12, maxit=1000, max_refine=10, fp64=True)
        a, _ = B.p2m_mass_assign_noalloc(ctx, d, v, opts)
        b, rep = B.p2m_mass_assign(ctx, d, v, opts)
        torch.cuda.synchronize()
        assert torch.equal(a, b) and B.read_report(rep, F).flags == 0
    finally:
        ctx.close()
