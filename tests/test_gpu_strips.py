"""Long thin FP32 meshes (more than 256 square solver tiles that are mostly empty): a batch
with such strips beside ordinary meshes of both tile sizes equals its single calls bit for
bit, values and reports, and AUTO takes the diagonal solve there (the bits of RESIDENT)."""
import numpy as np
import pytest

from test_gpu_poly import problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

STRIPS = [(16500, 2), (2, 16500), (16386, 16), (65537, 5)]


@pytest.mark.parametrize("F,strips", [(1, STRIPS), (2, [(20000, 16), (4, 17000)]), (3, [(16500, 3), (40000, 4)])])
def test_batch_equals_single(F, strips):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_05258_amd import binding as B
    insts = [problem(nx, ny, 4, F, np.float32) for nx, ny in [(40, 33)] + strips + [(600, 560)]]
    ctx = B.Context(0)
    try:
        probs = [B.particles_from(p) for p, _ in insts]
        vals = [torch.as_tensor(v).cuda() for _, v in insts]
        opts = B.solve_opts(tol=1e-8, maxit=2000, max_refine=20)
        outs, bt = B.p2m_mass_assign_batched(ctx, probs, vals, opts)
        outs, reps = [o.clone() for o in outs], bt.reports()
        for k, (p, _) in enumerate(insts):
            print(f"[strips] {p['nx']}x{p['ny']} F={F}", flush=True)
            one, rep = B.p2m_mass_assign(ctx, probs[k], vals[k], opts)
            torch.cuda.synchronize()
            a, b = reps[k], B.read_report(rep, F)
            assert not (b.flags & (B.FLAG_BREAKDOWN | B.FLAG_NOT_CONVERGED))
            assert torch.equal(outs[k], one), k
            assert list(a.iters) == list(b.iters) and list(a.rel_residual) == list(b.rel_residual)
            if p["nx"] > 16384 and -(-p["nx"] // 128) * -(-p["ny"] // 32) <= 256:
                ctx.set_solver(B.SOLVER_RESIDENT)
                res, _ = B.p2m_mass_assign(ctx, probs[k], vals[k], opts)
                torch.cuda.synchronize()
                ctx.set_solver(B.SOLVER_AUTO)
                assert torch.equal(res, one), k
    finally:
        ctx.close()
