"""The polynomial-preconditioned mass solve (AUTO) at the edges of its tiles and dispatch
rules, against the FP64 oracle (Sec. 2.4 under the particle quadrature): 32 x 32 tiles up
to 256 of them, 64 x 64 tiles resident and streamed beyond, meshes narrower than the
three-deep ring of a tile, remainders of one node, one to three fields, FP32 (relative l2
<= 1e-6) and FP64 (<= 1e-12); a batch that mixes both tile sizes equals its single calls
bit for bit, and forced RESIDENT batches keep the diagonal solver's bits."""
import numpy as np
import pytest

from oracle import metrics
from oracle import p1
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


def problem(nx, ny, ppc, F, dtype):
    x, y = wl.stratified_2d(nx * 1000 + ny, nx, ny, ppc, 2.0, 1.5)
    vals = wl.taylor_green(np.pi * x, np.pi * y / 0.75)[:F]
    return dict(dim=2, nx=nx, ny=ny, lx=2.0, ly=1.5, x=x.astype(dtype), y=y.astype(dtype),
                vol=None), vals.astype(dtype)


def reference(prob, vals):
    pr = dict(prob, x=np.asarray(prob["x"], np.float64), y=np.asarray(prob["y"], np.float64))
    st = p1.assemble_stencil(pr, vals.astype(np.float64))
    M = p1.regularised_matrix(p1.stencil_matrix(pr, st), st["w"])
    return [p1.cg_fp64(M, b, rtol=1e-14)[0] for b in st["b"]]


@pytest.mark.parametrize("nx,ny,F,bits", [
    (2, 2, 1, 32), (3, 40, 2, 32), (5, 33, 3, 32), (31, 32, 1, 32), (32, 32, 3, 32), (33, 65, 2, 32),
    (34, 98, 3, 32), (512, 512, 1, 32), (513, 512, 2, 32), (576, 641, 3, 32), (1030, 1100, 1, 32),
    (64, 64, 1, 64), (65, 97, 3, 64), (200, 130, 2, 64), (300, 257, 1, 64)])
def test_tile_edges(B, nx, ny, F, bits):
    print(f"[poly] {nx}x{ny} F={F} FP{bits}", flush=True)
    dtype = np.float32 if bits == 32 else np.float64
    prob, vals = problem(nx, ny, 5, F, dtype)
    ctx = B.Context(0)
    try:
        d = B.particles_from(prob)
        v = torch.as_tensor(vals).cuda()
        opts = B.solve_opts(tol=1e-9 if bits == 32 else 1e-14, maxit=2000, max_refine=20, fp64=bits == 64)
        out, rep = B.p2m_mass_assign(ctx, d, v, opts)
        out = out.clone()
        again, _ = B.p2m_mass_assign(ctx, d, v, opts)
        torch.cuda.synchronize()
        assert torch.equal(out, again)
        r = B.read_report(rep, F)
        assert not (r.flags & B.FLAG_BREAKDOWN)
        for f, ref in enumerate(reference(prob, vals)):
            assert metrics.rel_l2(out[f].cpu().numpy().astype(np.float64), ref) <= (1e-6 if bits == 32 else 1e-12)
    finally:
        ctx.close()


@pytest.mark.parametrize("solver", ["AUTO", "RESIDENT"])
def test_batch_of_both_tile_sizes(B, solver):
    insts = [problem(nx, ny, ppc, 2, np.float32) for nx, ny, ppc in ((600, 560, 3), (40, 70, 4), (33, 31, 6))]
    ctx = B.Context(0)
    try:
        ctx.set_solver(getattr(B, "SOLVER_" + solver))
        probs = [B.particles_from(p) for p, _ in insts]
        vals = [torch.as_tensor(v).cuda() for _, v in insts]
        opts = B.solve_opts(tol=1e-9, maxit=2000, max_refine=20)
        outs, bt = B.p2m_mass_assign_batched(ctx, probs, vals, opts)
        outs = [o.clone() for o in outs]
        for k in range(len(insts)):
            one, rep = B.p2m_mass_assign(ctx, probs[k], vals[k], opts)
            torch.cuda.synchronize()
            assert torch.equal(outs[k], one), k
            a, b = bt.reports()[k], B.read_report(rep, 2)
            assert list(a.iters) == list(b.iters) and list(a.rel_residual) == list(b.rel_residual)
    finally:
        ctx.close()
