"""FLIP and PIC whose result lies over an input: the values are read whole before the
result is written, as with buffers of their own; and the orphan count of both forms."""
import numpy as np
import pytest

from paper_1610_05258_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dim,nx,ny,dt", [(2, 33, 47, torch.float32), (2, 40, 30, torch.float64),
                                          (1, 700, 1, torch.float64)])
@pytest.mark.parametrize("offset", [0, 5, -3])
def test_in_place(dim, nx, ny, dt, offset):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_05258_amd import binding as B
    print(f"[final overlap] {dim}D {nx}x{ny} {dt} offset={offset}", flush=True)
    rng = np.random.Generator(np.random.PCG64(nx))
    if dim == 2:
        x, y = wl.stratified_2d(nx + ny, nx, ny, 3, 1.0, 1.0)
        keep = x > 4.0 / nx   # empty columns: orphans
        x, y = x[keep], y[keep]
    else:
        x, y = rng.uniform(0.1, 1.0, 3 * nx), None
    n = x.size
    d = B.Particles(dim=dim, nx=nx, ny=ny, lx=1.0, ly=1.0, x=torch.tensor(x, device="cuda", dtype=dt),
                    y=torch.tensor(y, device="cuda", dtype=dt) if dim == 2 else None)
    ctx = B.Context(0)
    try:
        for kind in (B.FLIP, B.PIC):
            buf = torch.zeros(n + 16, dtype=dt, device="cuda")
            vals = buf[8:8 + n]
            vals.copy_(torch.tensor(rng.standard_normal(n), dtype=dt))
            want, rep = B.p2m_assign(ctx, d, kind, vals.clone()[None])
            out = buf[8 + offset:8 + offset + nx * ny][None]
            _, rep2 = B.p2m_assign(ctx, d, kind, vals[None], out=out)
            assert torch.equal(out, want)
            r, r2 = B.read_report(rep, 1), B.read_report(rep2, 1)
            assert r.n_orphan == r2.n_orphan > 0 and r.flags == r2.flags
    finally:
        ctx.close()
