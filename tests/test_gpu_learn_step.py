"""The training step at the edges of its row blocks (64 rows, the gradient sums in groups
of 32 blocks) and with parameters at every alignment of a float: loss and gradient
against the FP64 oracle with the bounds of the network's other gradient test (1e-3 and
1e-2, BF16 products), and the same bits whatever the alignment."""
import numpy as np
import pytest

from oracle import metrics, mlp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("rows", [1, 15, 16, 63, 64, 65, 130, 2048, 2100])
def test_rows_and_alignment(rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_05258_amd import binding as B
    print(f"[learn step] rows={rows}", flush=True)
    g = np.random.default_rng(rows)
    N = rows + 7
    X = torch.as_tensor(g.normal(0, 0.5, (N, mlp.N_IN)).astype(np.float32)).cuda().to(torch.bfloat16)
    t = g.normal(0, 1, N).astype(np.float32)
    sel = g.permutation(N)[:rows].astype(np.int32)
    th = np.asarray(mlp.init_params(rows), np.float32)
    Xo = X.float().cpu().numpy().astype(np.float64)[sel]
    lo, go, _ = mlp.loss_and_grad(th.astype(np.float64), Xo, t[sel].astype(np.float64))
    ctx = B.Context(0)
    try:
        outs = []
        for off in range(4):
            buf = torch.zeros(B.LEARNED_NPARAM + 4, dtype=torch.float32, device="cuda")
            P = buf[off:off + B.LEARNED_NPARAM]
            P.copy_(torch.as_tensor(th))
            tr = B.Trainer(ctx, P, batch=rows)
            grad = torch.empty(B.LEARNED_NPARAM, dtype=torch.float32, device="cuda")
            loss = tr.run(X, torch.as_tensor(t).cuda(), torch.as_tensor(sel).cuda(), apply=False, grad=grad).item()
            y = B.learned_forward(ctx, P, X)
            outs.append((loss, grad.cpu().numpy(), y.cpu().numpy()))
    finally:
        ctx.close()
    assert abs(outs[0][0] - lo) <= 1e-3 * lo
    assert metrics.rel_l2(outs[0][1].astype(np.float64), go) <= 1e-2
    for o in outs[1:]:
        assert o[0] == outs[0][0] and np.array_equal(o[1], outs[0][1]) and np.array_equal(o[2], outs[0][2])
