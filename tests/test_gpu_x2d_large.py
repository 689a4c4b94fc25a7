"""The exported triangulation of 67,240,000 particles: its 32 entries a particle number more
than 2^31.  (73 GB of device memory.)  Every particle has a star, and for the first, the last
and a spread of the others each neighbour lists the particle back at the opposite image."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_export_beyond_int32_entries():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if torch.cuda.mem_get_info()[0] < 90 << 30:
        pytest.skip("needs 90 GB of free device memory")
    from paper_1610_05258_amd import binding as B
    n, ppc = 4100, 4
    N = n * n * ppc
    assert N * B.X2D_MAXDEG > 2 ** 31
    g = torch.Generator("cuda").manual_seed(3)
    c = torch.arange(N, device="cuda") // ppc
    x = ((c % n).double() + torch.rand(N, generator=g, device="cuda", dtype=torch.float64)) / n
    y = ((c // n).double() + torch.rand(N, generator=g, device="cuda", dtype=torch.float64)) / n
    del c
    ctx = B.Context(0)
    try:
        d = B.Particles(dim=2, nx=n, ny=n, lx=1.0, ly=1.0, x=x.clamp_(max=1 - 1e-12), y=y.clamp_(max=1 - 1e-12))
        print(f"[x2d large] {N} particles, workspace {B.x2d_workspace_size(ctx, d, 1) / 1e9:.1f} GB", flush=True)
        deg, nbr, sh, rep = B.p2m_x2d_triangulation(ctx, d)
        torch.cuda.synchronize()
        assert B.read_report(rep, 1).flags == 0 and int(deg.min()) >= 3 and int(deg.max()) <= B.X2D_MAXDEG
        assert int(deg.long().sum()) == 6 * N   # a triangulation of the torus
        p = torch.cat([torch.arange(0, 2000), torch.arange(N - 2000, N), torch.arange(0, N, 33617)]).cuda()
        live = torch.arange(B.X2D_MAXDEG, device="cuda")[None] < deg[p][:, None]
        assert bool((nbr[p][~live] == -1).all())
        who, j = torch.nonzero(live, as_tuple=True)
        q, s = nbr[p[who], j].long(), sh[p[who], j]
        back = ((128 - (s & 255)) + 128) | (((128 - ((s >> 8) & 255)) + 128) << 8)
        hit = (nbr[q] == p[who][:, None].int()) & (sh[q] == back[:, None].int())
        assert bool(hit.any(1).all())
    finally:
        ctx._ws = None
        ctx.close()
        torch.cuda.empty_cache()
