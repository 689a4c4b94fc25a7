"""Paper-exact 1D in one launch before the solve (up to 3072 particles and cells) against
the general path, which the same particles take when particles that cannot be located
are appended until there are more than 3072: the same operations, so the same bits
before the solve; the solves agree to their residual's order."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,np_,how", [(2, 5, "any"), (3, 1, "any"), (64, 256, "any"), (64, 1000, "one"),
                                       (1024, 1025, "any"), (1025, 40, "any"), (3072, 3072, "any"),
                                       (300, 3072, "few"), (50, 200, "bad")])
@pytest.mark.parametrize("F", [1, 3])
def test_same_as_general(n, np_, how, F):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_05258_amd import binding as B
    print(f"[x1d_small] n={n} np={np_} {how} F={F}", flush=True)
    rng = np.random.Generator(np.random.PCG64(n + np_))
    x = (np.arange(np_) + rng.uniform(0.1, 0.9, np_)) / np_
    if how == "one":
        x = (7 + x) / n
    if how == "few":
        x = x * 40 / n
    x = rng.permutation(x)
    if how == "bad":
        x[::7] = np.nan
        x[3::7] = -2.0
    A = rng.standard_normal((F, np_))
    pad = 3073 - np_
    xg, Ag = np.concatenate([x, np.full(pad, np.nan)]), np.concatenate([A, np.zeros((F, pad))], 1)
    nodal = torch.tensor(rng.standard_normal((F, n)), device="cuda")
    ctx = B.Context(0)
    try:
        ds = [B.Particles(dim=1, nx=n, ny=1, lx=1.0, ly=1.0, x=torch.tensor(v, device="cuda")) for v in (x, xg)]
        vs = [torch.tensor(v, device="cuda") for v in (A, Ag)]
        for quad in (B.QUAD_EXACT, B.QUAD_APPB):
            for kind in (B.X1D_DELTA, B.X1D_LUMPED, B.X1D_MASS):
                o = [B.p2m_x1d_assign(ctx, d, kind, quad, v) for d, v in zip(ds, vs)]
                q = [B.p2m_x1d_interpolate(ctx, d, kind, quad, nodal) for d in ds]
                f = [B.read_report(r[1], F) for r in o]
                assert f[0].flags == (f[1].flags if how == "bad" else f[1].flags & ~B.FLAG_NONFINITE)
                assert f[0].n_invalid == f[1].n_invalid - pad
                got, want = o[0][0].cpu().numpy(), o[1][0].cpu().numpy()
                gq, wq = q[0][0].cpu().numpy(), q[1][0].cpu().numpy()[:, :np_]
                assert np.array_equal(np.isnan(gq), np.isnan(wq))
                if kind == B.X1D_MASS:
                    assert np.abs(got - want).max() <= 1e-12 * np.abs(want).max()
                    assert np.nanmax(np.abs(gq - wq)) <= 1e-12 * np.nanmax(np.abs(wq))
                else:
                    assert np.array_equal(got, want)
                    assert np.array_equal(gq, wq, equal_nan=True)
        va = [B.p2m_x1d_volumes(ctx, d).cpu().numpy() for d in ds]
        assert np.array_equal(va[0], va[1][:np_], equal_nan=True)
    finally:
        ctx.close()
