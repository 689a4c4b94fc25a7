"""The periodic Delaunay triangulation over its dispatch: the four-lane kernel (meshes of
at least 9 cells a side), what it leaves to the general kernel (stars that reach beyond
its radius, lists that overflow, few and many of them) and the meshes the general kernel
takes whole, on even and strongly uneven particle sets.  The triangles and the volumes
equal those of the oracle (particle numbers and image shifts, named canonically)."""
import numpy as np
import pytest

from oracle import paper2d as p2
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


def positions(kind, nx, ny, ppc):
    g = np.random.Generator(np.random.PCG64(nx * 100 + ny))
    n = nx * ny * ppc
    if kind == "even":
        return wl.stratified_2d(nx + ny, nx, ny, ppc, 1.0, 1.0)
    if kind == "graded":      # dense towards one corner, sparse away from it
        return g.random(n) ** 2, g.random(n) ** 2
    c = np.repeat(np.arange(nx * ny), ppc)   # "clusters": a tight one in every cell
    return ((c % nx + 0.5 + 0.02 * g.standard_normal(n)) / nx,
            (c // nx + 0.5 + 0.02 * g.standard_normal(n)) / ny)


@pytest.mark.parametrize("kind,nx,ny,ppc", [("even", 9, 9, 1), ("even", 9, 12, 6), ("even", 8, 9, 3),
                                            ("even", 33, 17, 2), ("graded", 20, 20, 5),
                                            ("graded", 9, 30, 12), ("clusters", 10, 10, 60),
                                            ("clusters", 12, 9, 20)])
def test_triangulation(B, kind, nx, ny, ppc):
    print(f"[x2d star] {kind} {nx}x{ny} x {ppc}", flush=True)
    x, y = positions(kind, nx, ny, ppc)
    ctx = B.Context(0)
    try:
        d = B.Particles(dim=2, nx=nx, ny=ny, lx=1.0, ly=1.0, x=torch.tensor(x, device="cuda"),
                        y=torch.tensor(y, device="cuda"))
        deg, nbr, sh, rep = B.p2m_x2d_triangulation(ctx, d)
        vol, _ = B.p2m_x2d_volumes(ctx, d)
        flags = B.read_report(rep, 1).flags
        deg, nbr, sh, vol = (t.cpu().numpy() for t in (deg, nbr, sh, vol))
    finally:
        ctx.close()
    tri, shifts = p2.periodic_delaunay(x, y, 1.0, 1.0)
    want = {p2._canonical(i, s) for i, s in zip(tri, shifts)}
    # a star that no search of 8 rings closes, or of more than 32 neighbours, is flagged;
    # every star that is given is the oracle's
    assert flags == 0 or (flags == B.FLAG_TRIANGULATION and kind == "clusters")
    seen = {}
    for mu in np.nonzero(deg)[0]:
        for j in range(deg[mu]):
            j1 = (j + 1) % deg[mu]
            s = np.array([[0, 0]] + [[(sh[mu, q] & 255) - 128, ((sh[mu, q] >> 8) & 255) - 128]
                                     for q in (j, j1)])
            key = p2._canonical(np.array([mu, nbr[mu, j], nbr[mu, j1]]), s)
            seen[key] = seen.get(key, 0) + 1
    assert set(seen) <= want
    if flags == 0:
        assert set(seen) == want and set(seen.values()) == {3}
        assert abs(vol.sum() - 1.0) <= 1e-12
