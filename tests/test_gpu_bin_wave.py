"""Binning in one launch with cells on either side of its three sorts (a thread up to 16
particles, a wave up to 64, the workgroup beyond), in reversed and shuffled particle order,
with fewer and with more cells than the workgroup has threads.  Integers: exactly the
stable order by cell."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nx,counts", [(40, [16, 17, 63, 64, 65, 1, 0, 33, 130, 2]), (400, [17, 20]), (127, [64]),
                                       (1500, [1, 0, 18, 0, 2])])
@pytest.mark.parametrize("order", ["reversed", "shuffled"])
def test_order(nx, counts, order):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_05258_amd import binding as B
    print(f"[bin wave] {nx} {counts} {order}", flush=True)
    cell = np.repeat(np.arange(nx), np.resize(counts, nx))[:8192]
    cell = cell[::-1].copy() if order == "reversed" else np.random.default_rng(nx).permutation(cell)
    ctx = B.Context(0)
    try:
        d = B.Particles(dim=1, nx=nx, ny=1, lx=float(nx), ly=1.0, x=torch.tensor(cell + 0.5, device="cuda").float())
        perm, cs, rep = B.p2m_bin(ctx, d)
        assert np.array_equal(perm.cpu().numpy(), np.argsort(cell, kind="stable").astype(np.int32))
        assert np.array_equal(np.diff(cs.cpu().numpy()), np.bincount(cell, minlength=nx))
        assert B.read_report(rep, 1).flags == 0
    finally:
        ctx.close()
