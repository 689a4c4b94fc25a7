"""Paper-exact 1D results written over the positions they were computed from (volumes, and the
mesh to particle kinds), small problems and large, with particles that cannot be located:
the bits of a call with a result array of its own."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,np_", [(64, 300), (3000, 3072), (700, 5000), (9000, 40000), (500000, 2000000)])
@pytest.mark.parametrize("what", ["volumes", "delta", "mass", "lumped"])
def test_result_over_positions(n, np_, what):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_05258_amd import binding as B
    print(f"[x1d in place] {n} {np_} {what}", flush=True)
    g = np.random.default_rng(n)
    x = np.minimum(g.random(np_), 0.9999999)
    x[g.random(np_) < 0.05] = np.nan
    x[g.random(np_) < 0.05] = 7.0
    nodal = torch.tensor(g.standard_normal((1, n)), device="cuda")
    ctx = B.Context(0)
    try:
        got = []
        for over in (False, True):
            d = B.Particles(dim=1, nx=n, ny=1, lx=1.0, ly=1.0, x=torch.tensor(x, device="cuda"))
            out = d.x if over else torch.empty(np_, dtype=torch.float64, device="cuda")
            rep = ctx.new_report()
            if what == "volumes":
                cp = d.cstruct()
                wp, wn = B._x1d_ws(ctx, d, 1, None)
                assert B.lib().p2m_x1d_volumes(ctx.handle, ctypes.byref(cp), ctypes.c_void_p(out.data_ptr()),
                                               ctypes.c_void_p(rep.data_ptr()), wp, wn, B._stream_ptr(None)) == 0
            else:
                B.p2m_x1d_interpolate(ctx, d, getattr(B, "X1D_" + what.upper()), B.QUAD_APPB, nodal, rep=rep,
                                      out=out[None])
            r = B.read_report(rep, 1)
            got.append(out.cpu().numpy().copy())
            assert r.flags & (B.FLAG_RANGE | B.FLAG_NONFINITE)
        bad = np.isnan(x) | (x == 7.0)
        assert np.array_equal(np.isnan(got[0]), bad)
        assert np.array_equal(got[0], got[1], equal_nan=True)
    finally:
        ctx.close()
