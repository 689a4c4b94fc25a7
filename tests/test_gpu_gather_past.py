"""The node-major gather around the size from which its positions bypass the caches (288 MB of
positions and results): just below and above it, with 16-byte accesses and without, FP32 and
FP64; against the same interpolation in FP64 torch, rounding of three products and two sums
(8 eps)."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EDGE = (288 << 20) // 4 // 6     # particles, FP32, F = 4


@pytest.mark.parametrize("F,dt,n", [(4, torch.float32, EDGE // 4 * 4), (4, torch.float32, EDGE // 4 * 4 + 4),
                                    (4, torch.float32, EDGE + 3), (2, torch.float64, (288 << 20) // 8 // 4),
                                    (2, torch.float64, (288 << 20) // 8 // 4 + 1)])
def test_gather(F, dt, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_05258_amd import binding as B
    print(f"[gather past] F={F} {dt} n={n}", flush=True)
    nx, ny = 61, 40
    g = torch.Generator("cuda").manual_seed(F)
    x, y = (torch.rand(n, generator=g, device="cuda", dtype=torch.float64).clamp_(max=0.999999).to(dt) for _ in range(2))
    x[n // 2] = float("nan")
    nodal = torch.randn((F, nx * ny), generator=g, device="cuda", dtype=torch.float64).to(dt)
    ctx = B.Context(0)
    try:
        d = B.Particles(dim=2, nx=nx, ny=ny, lx=1.0, ly=1.0, x=x, y=y)
        ws = torch.empty(F * nx * ny * 8, dtype=torch.uint8, device="cuda")
        out, rep = B.p2m_interpolate(ctx, d, nodal, ws=ws)
        r = B.read_report(rep, F)
    finally:
        ctx.close()
    assert r.n_invalid == 0 and r.flags == B.FLAG_NONFINITE and bool(out[:, n // 2].isnan().all())
    x[n // 2] = 0.5
    tx, ty = x.double() * nx, y.double() * ny
    i, j = tx.floor().long(), ty.floor().long()
    a, b = tx - i, ty - j
    i1, j1 = (i + 1) % nx, (j + 1) % ny
    low = a >= b
    w = [1 - torch.where(low, a, b), torch.where(low, a - b, b - a), torch.where(low, b, a)]
    k = [i + nx * j, torch.where(low, i1 + nx * j, i + nx * j1), i1 + nx * j1]
    eps = torch.finfo(dt).eps
    for f in range(F):
        A = nodal[f].double()
        want = sum(w[c] * A[k[c]] for c in range(3))
        scale = sum(w[c] * A[k[c]].abs() for c in range(3))
        err = (out[f].double() - want).abs() - 8 * eps * scale
        err[n // 2] = 0
        assert float(err.max()) <= 1e-300
