"""The measured workloads of the assignment library: what a particle program calls per time step.

Every case is one pass of a loop that a user's program runs thousands of times: particles
have moved, their values go to the mesh (FLIP or the mass assignment) and come back.  The
sizes are those of this repository's configurations and benchmark legs; draw() spreads the
same families over their ranges, ragged sides and field counts among them.

prepare() makes the inputs on the GPU from the seed with plain torch; run() calls the public
entry points of paper_1610_05258_amd.binding; exact() is the same method in 64 bits, in plain
torch, without the library.
"""
from __future__ import annotations

import math

import torch

from paper_1610_05258_amd import binding as B

TWO_PI = 2.0 * math.pi
DEV = "cuda"
F64 = torch.float64


# ----------------------------------------------------------------------------
# the cases
# ----------------------------------------------------------------------------
def listed():
    return [
        # the 1D top-hat: 64 elements, 256 random particles, FP64, mass P2M and M2P; the
        # smallest problem a program has, where launches and the host path count
        dict(name="tophat_1d", kind="step", dim=1, nx=64, ny=1, ppc=4, fields=1, dtype="f64", p2m="mass"),
        # the paper's Table 2 set-up with the particle hats: full mass there and back, one
        # field, Appendix-B quadrature
        dict(name="table2_1d", kind="exact1d", nx=64, ppc=4, fields=1),
        # an ordinary particle-in-cell step (FLIP and interpolation) on a ragged mesh
        dict(name="pic_333x217", kind="step", dim=2, nx=333, ny=217, ppc=5, fields=2, dtype="f32",
             p2m="flip"),
        # the slotted disk: 256 x 256, 4 per cell, one field, mass P2M and M2P each step
        dict(name="zalesak_256", kind="step", dim=2, nx=256, ny=256, ppc=4, fields=1, dtype="f32",
             p2m="mass"),
        # the headline: Taylor-Green u, v, p at 1024 x 1024, 8 per cell, mass P2M and M2P
        dict(name="tg_1024", kind="step", dim=2, nx=1024, ny=1024, ppc=8, fields=3, dtype="f32",
             p2m="mass"),
        # the same fields on four times the mesh: 33.5 million particles, more solver tiles
        # than compute units; the largest call
        dict(name="tg_2048", kind="step", dim=2, nx=2048, ny=2048, ppc=8, fields=3, dtype="f32",
             p2m="mass"),
        # the plain double-precision form on an ordinary mesh
        dict(name="fp64_512", kind="step", dim=2, nx=512, ny=512, ppc=8, fields=1, dtype="f64",
             p2m="mass"),
        # 64 independent meshes of side 32 to 512 with 2 to 16 per cell in one graph launch
        dict(name="uneven_batch", kind="batch", count=64, side_lo=32, side_hi=512, fields=2),
        # one time step of the Taylor-Green vortex sheet, mass P2M, Courant 0.5
        dict(name="fluid_256", kind="fluid", nx=256, ny=256, ppc=4, p2m="mass"),
        # the paper's slotted disk with the particle triangulation, full mass there and back
        dict(name="exact2d_90", kind="exact2d", nx=90, ny=90, ppc=1, fields=1),
        # the same at a million particles
        dict(name="exact2d_512", kind="exact2d", nx=512, ny=512, ppc=4, fields=1),
        # one training step (forward, backward, Adam) of the warm-start network
        dict(name="train_4096", kind="train", rows=4096),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step1d", "flip", "mass", "mass", "mass64", "batch", "fluid", "exact1d", "exact2d",
                       "train"])
    if kind == "step1d":
        return dict(kind="step", dim=1, nx=_log(rng, 16, 4096), ny=1, ppc=rng.randint(3, 8),
                    fields=rng.randint(1, 3), dtype="f64", p2m="mass")
    if kind in ("flip", "mass", "mass64"):
        hi = 768 if kind == "mass64" else 2048
        nx = _log(rng, 32, hi)
        ny = max(32, min(hi, int(nx * rng.uniform(0.5, 1.5))))
        return dict(kind="step", dim=2, nx=nx, ny=ny, ppc=rng.randint(4, 8), fields=rng.randint(1, 3),
                    dtype="f64" if kind == "mass64" else "f32", p2m="flip" if kind == "flip" else "mass")
    if kind == "batch":
        lo = rng.randint(32, 96)
        return dict(kind="batch", count=rng.randint(4, 64), side_lo=lo, side_hi=rng.randint(lo + 32, 512),
                    fields=rng.randint(1, 2))
    if kind == "fluid":
        n = _log(rng, 64, 768)
        return dict(kind="fluid", nx=n, ny=n, ppc=rng.randint(4, 6), p2m=rng.choice(["mass", "flip"]))
    if kind == "exact1d":
        return dict(kind="exact1d", nx=_log(rng, 32, 16384), ppc=rng.randint(2, 8), fields=rng.randint(1, 2))
    if kind == "exact2d":
        nx = _log(rng, 32, 448)
        return dict(kind="exact2d", nx=nx, ny=max(32, int(nx * rng.uniform(0.75, 1.1))),
                    ppc=rng.randint(1, 4), fields=rng.randint(1, 2))
    return dict(kind="train", rows=_log(rng, 512, 16384))


# ----------------------------------------------------------------------------
# inputs (plain torch, from the seed alone)
# ----------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 13)
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV, dtype=F64)


def _stratified(g, nx, ny, ppc, lx, ly):
    """ppc uniform particles in every cell, cell by cell, FP64."""
    c = torch.arange(nx * ny, device=DEV).repeat_interleave(ppc)
    u = _rand(g, 2, nx * ny * ppc)
    return (c % nx + u[0]) * (lx / nx), (c // nx + u[1]) * (ly / ny)


def _taylor_green(x, y):
    return torch.stack([torch.sin(x) * torch.cos(y), -torch.cos(x) * torch.sin(y),
                        0.25 * (torch.cos(2.0 * x) + torch.cos(2.0 * y))])


def _advect(x, y, steps, dt):
    """Midpoint steps in the Taylor-Green velocity, wrapped into [0, 2 pi)."""
    for _ in range(steps):
        u, v = torch.sin(x) * torch.cos(y), -torch.cos(x) * torch.sin(y)
        xm, ym = x + 0.5 * dt * u, y + 0.5 * dt * v
        u, v = torch.sin(xm) * torch.cos(ym), -torch.cos(xm) * torch.sin(ym)
        x, y = torch.remainder(x + dt * u, TWO_PI), torch.remainder(y + dt * v, TWO_PI)
    return x, y


def _disk(x, y):
    """Zalesak's slotted disk in the unit square: radius 0.15, slot 0.05 wide."""
    inside = (x - 0.5) ** 2 + (y - 0.75) ** 2 <= 0.15 ** 2
    slot = ((x - 0.5).abs() <= 0.025) & (y <= 0.85)
    return (inside & ~slot).to(F64)


def _rotate(x, y, angle):
    """Rigid rotation of the particles within the moving circle of the slotted-disk runs."""
    dx, dy = x - 0.5, y - 0.5
    move = dx * dx + dy * dy <= (0.5 * 1.4 / 1.5) ** 2
    c, s = math.cos(angle), math.sin(angle)
    return (torch.where(move, 0.5 + c * dx - s * dy, x), torch.where(move, 0.5 + s * dx + c * dy, y))


def _step_inputs(case, seed):
    """(x, y or None, values, lx, ly) in the case's type."""
    g = _gen(seed)
    dt = F64 if case["dtype"] == "f64" else torch.float32
    nx, ny, ppc, F = case["nx"], case["ny"], case["ppc"], case["fields"]
    if case["dim"] == 1:
        x = _rand(g, nx * ppc)
        if nx * ppc > 512:   # long segments: stratified, so that no node is left without particles
            x = (torch.arange(nx * ppc, device=DEV) // ppc + x) / nx
        top = ((x >= 0.25) & (x < 0.5)).to(F64)
        vals = torch.stack([top, torch.sin(TWO_PI * x), torch.cos(TWO_PI * x)])[:F]
        return x.to(dt), None, vals.to(dt).contiguous(), 1.0, 1.0
    x, y = _stratified(g, nx, ny, ppc, TWO_PI, TWO_PI)
    vals = _taylor_green(x, y)[:F]
    if F == 1:   # the slotted disk, on the same box
        vals = _disk(x / TWO_PI, y / TWO_PI)[None]
    vals = vals + 1e-3 * torch.randn(vals.shape, generator=g, device=DEV, dtype=F64)
    x, y = _advect(x, y, 20, 2.5e-3)
    return x.to(dt), y.to(dt), vals.to(dt).contiguous(), TWO_PI, TWO_PI


def _batch_inputs(case, seed):
    """[(nx, x, y, values)]: square meshes, side log-uniform, 2 to 16 per cell.  The sides and
    counts are the case's, the positions and fields the seed's."""
    sizes = torch.Generator()
    sizes.manual_seed(1000 + case["count"])
    g = _gen(seed)
    out = []
    for _ in range(case["count"]):
        u = torch.rand(2, generator=sizes, dtype=F64).tolist()
        n = int(round(case["side_lo"] * (case["side_hi"] / case["side_lo"]) ** u[0]))
        ppc = 2 + int(15 * u[1])
        x, y = _stratified(g, n, n, ppc, TWO_PI, TWO_PI)
        ph = _rand(g, 2) * TWO_PI
        v = _taylor_green(x + ph[0], y + ph[1])[:case["fields"]]
        out.append((n, x.float(), y.float(), v.float().contiguous()))
    return out


def _fluid_inputs(case, seed):
    """Unit box, particles carrying the Taylor-Green velocity, disordered by a few steps."""
    x, y = _stratified(_gen(seed), case["nx"], case["ny"], case["ppc"], 1.0, 1.0)
    x, y = _advect(x * TWO_PI, y * TWO_PI, 10, 2.5e-3)
    x, y = (x / TWO_PI).float(), (y / TWO_PI).float()
    kx, ky = TWO_PI * x.double(), TWO_PI * y.double()
    vel = torch.stack([torch.sin(kx) * torch.cos(ky), -torch.cos(kx) * torch.sin(ky)]).float()
    return x, y, vel.contiguous()


def _exact1d_inputs(case, seed):
    g = _gen(seed)
    n = case["nx"] * case["ppc"]
    x = (torch.arange(n, device=DEV) + _rand(g, n)) / n   # distorted regular spacing, any order
    x = x[torch.randperm(n, generator=g, device=DEV)].contiguous()
    v = torch.stack([((x > 0.25) & (x < 0.75)).to(F64), torch.sin(TWO_PI * x)])[:case["fields"]]
    return x, v.contiguous()


def _exact2d_inputs(case, seed):
    g = _gen(seed)
    x, y = _stratified(g, case["nx"], case["ny"], case["ppc"], 1.0, 1.0)
    v = torch.stack([_disk(x, y), torch.sin(TWO_PI * x) * torch.cos(TWO_PI * y)])[:case["fields"]]
    x, y = _rotate(x, y, float(_rand(g, 1)) * TWO_PI)
    return x.contiguous(), y.contiguous(), v.contiguous()


def _train_inputs(case, seed):
    """Feature rows like those of learned_features (8 particles in each of a node's four cells),
    targets, network weights and an Adam state in the middle of a training."""
    g = _gen(seed)
    table = 4 * case["rows"]
    n = (torch.randn(table, generator=g, device=DEV) * 3 + 32).round().clamp(1, B.LEARNED_KMAX)
    on = torch.arange(B.LEARNED_KMAX, device=DEV)[None] < n[:, None]
    X = torch.zeros(table, B.LEARNED_NIN, device=DEV)
    for j in range(3):
        r = torch.rand(table, B.LEARNED_KMAX, generator=g, device=DEV) * 2 - 1
        X[:, j:3 * B.LEARNED_KMAX:3] = torch.where(on, r * (1.7 if j == 2 else 1.0), torch.zeros_like(r))
    X[:, 3 * B.LEARNED_KMAX] = n / B.LEARNED_KMAX
    target = 0.25 * torch.randn(table, generator=g, device=DEV)
    H, NI, NF = B.LEARNED_HIDDEN, B.LEARNED_NIN, 3 * B.LEARNED_KMAX + 1
    w1 = torch.randn(H, NI, generator=g, device=DEV) * math.sqrt(2.0 / NF)
    w1[:, NF:] = 0.0
    w2, w3 = (torch.randn(H, H, generator=g, device=DEV) * math.sqrt(2.0 / H) for _ in range(2))
    w4 = 0.1 * torch.randn(H, generator=g, device=DEV)
    b = 0.05 * torch.randn(3 * H + 1, generator=g, device=DEV)
    params = torch.cat([w1.reshape(-1), b[:H], w2.reshape(-1), b[H:2 * H], w3.reshape(-1), b[2 * H:3 * H],
                        w4, b[3 * H:]])
    m = 1e-4 * torch.randn(params.shape, generator=g, device=DEV)
    v = 1e-5 * (0.5 + torch.rand(params.shape, generator=g, device=DEV))
    rows = torch.randint(0, table, (case["rows"],), generator=g, device=DEV, dtype=torch.int32)
    return X.bfloat16(), target, params, m, v, rows


TRAIN_STEP, TRAIN_LR = 1000, 2e-3
NU = 0.005


# ----------------------------------------------------------------------------
# prepare and run
# ----------------------------------------------------------------------------
def _opts(case):
    """The benchmark's tolerances: 1e-8 in FP32 (FP64 residual), 1e-13 in FP64."""
    if case.get("dtype") == "f64":
        return B.solve_opts(tol=1e-13, maxit=2000, max_refine=10, fp64=True)
    if case["kind"] == "batch":   # the 2-per-cell instances need the tighter residual
        return B.solve_opts(tol=1e-9, inner_rtol=1e-4, maxit=2000, max_refine=10)
    return B.solve_opts(tol=1e-8, inner_rtol=1e-4, maxit=2000, max_refine=10)


def prepare(case, seed):
    ctx = B.Context(0)
    s = dict(case=case, ctx=ctx)
    kind = case["kind"]
    if kind == "step":
        x, y, vals, lx, ly = _step_inputs(case, seed)
        p = B.Particles(case["dim"], case["nx"], case["ny"], lx, ly, x, y)
        F = case["fields"]
        s.update(prob=p, vals=vals, opts=_opts(case), rep=ctx.new_report(), rep2=ctx.new_report(),
                 ws=ctx.workspace(ctx.workspace_size(p, F)),
                 nodal=torch.empty((F, p.n_nodes), dtype=x.dtype, device=DEV),
                 back=torch.empty((F, p.n_particles), dtype=x.dtype, device=DEV))
    elif kind == "batch":
        inst = _batch_inputs(case, seed)
        probs = [B.Particles(2, n, n, TWO_PI, TWO_PI, x, y) for n, x, y, _ in inst]
        s.update(batch=B.Batch(ctx, probs, [v for _, _, _, v in inst], _opts(case)))
    elif kind == "fluid":
        x, y, vel = _fluid_inputs(case, seed)
        p = B.Particles(2, case["nx"], case["ny"], 1.0, 1.0, x, y)
        s.update(prob=p, vel=vel, opts=B.solve_opts(tol=1e-8, maxit=4000, max_refine=20),
                 dt=0.5 / case["nx"], x_out=torch.empty_like(x), y_out=torch.empty_like(y),
                 mesh=torch.empty((2, p.n_nodes), dtype=torch.float32, device=DEV),
                 reps=torch.zeros((3, B.REPORT_BYTES), dtype=torch.uint8, device=DEV),
                 ws=ctx.workspace(B.ns_workspace_size(ctx, p)),
                 method=B.NS_MASS if case["p2m"] == "mass" else B.NS_FLIP)
    elif kind == "exact1d":
        x, vals = _exact1d_inputs(case, seed)
        p = B.Particles(1, case["nx"], 1, 1.0, 1.0, x)
        s.update(prob=p, vals=vals, rep=ctx.new_report(), rep2=ctx.new_report(),
                 ws=ctx.workspace(B.x1d_workspace_size(ctx, p, case["fields"])),
                 nodal=torch.empty((case["fields"], p.n_nodes), dtype=F64, device=DEV),
                 back=torch.empty((case["fields"], p.n_particles), dtype=F64, device=DEV))
    elif kind == "exact2d":
        x, y, vals = _exact2d_inputs(case, seed)
        p = B.Particles(2, case["nx"], case["ny"], 1.0, 1.0, x, y)
        s.update(prob=p, vals=vals, reps=torch.zeros((2, B.REPORT_BYTES), dtype=torch.uint8, device=DEV),
                 ws=ctx.workspace(B.x2d_workspace_size(ctx, p, case["fields"])),
                 nodal=torch.empty((case["fields"], p.n_nodes), dtype=F64, device=DEV),
                 back=torch.empty((case["fields"], p.n_particles), dtype=F64, device=DEV))
    else:
        X, target, params, m, v, rows = _train_inputs(case, seed)
        tr = B.Trainer(ctx, params, case["rows"])
        tr.m, tr.v, tr.step = m, v, TRAIN_STEP
        s.update(X=X, target=target, rows=rows, trainer=tr, grad=torch.empty_like(params))
    return s


def run(s):
    case, ctx = s["case"], s["ctx"]
    kind = case["kind"]
    if kind == "step":
        p = s["prob"]
        if case["p2m"] == "mass":
            B.p2m_mass_assign(ctx, p, s["vals"], s["opts"], ws=s["ws"], rep=s["rep"], out=s["nodal"])
        else:
            B.p2m_assign(ctx, p, B.FLIP, s["vals"], ws=s["ws"], rep=s["rep"], out=s["nodal"])
        B.p2m_interpolate(ctx, p, s["nodal"], ws=s["ws"], rep=s["rep2"], out=s["back"])
        return s["nodal"], s["back"]
    if kind == "batch":
        return s["batch"].run()
    if kind == "fluid":
        B.p2m_ns_step(ctx, s["prob"], s["vel"], s["method"], s["dt"], NU, s["opts"], x_out=s["x_out"],
                      y_out=s["y_out"], mesh_vel=s["mesh"], reps=s["reps"], ws=s["ws"])
        return s["mesh"], s["vel"], s["x_out"], s["y_out"]
    if kind == "exact1d":
        p = s["prob"]
        B.p2m_x1d_assign(ctx, p, B.X1D_MASS, B.QUAD_APPB, s["vals"], ws=s["ws"], rep=s["rep"], out=s["nodal"])
        B.p2m_x1d_interpolate(ctx, p, B.X1D_MASS, B.QUAD_APPB, s["nodal"], ws=s["ws"], rep=s["rep2"],
                              out=s["back"])
        return s["nodal"], s["back"]
    if kind == "exact2d":
        B.p2m_x2d_round_trip(ctx, s["prob"], B.X1D_MASS, B.X1D_MASS, s["vals"], ws=s["ws"], reps=s["reps"],
                             nodal=s["nodal"], out=s["back"])
        return s["nodal"], s["back"]
    tr = s["trainer"]
    tr.run(s["X"], s["target"], s["rows"], lr=TRAIN_LR, grad=s["grad"])
    return tr.loss, s["grad"], tr.params, tr.m, tr.v


def work(case):
    """Inputs read once and outputs written once; the operations of the method itself."""
    kind = case["kind"]
    if kind == "train":
        n, P = case["rows"], B.LEARNED_NPARAM
        return dict(bytes=float(n * (2 * B.LEARNED_NIN + 8) + 4 * P * 7), flops=6.0 * P * n)
    if kind == "batch":
        sizes = torch.Generator()
        sizes.manual_seed(1000 + case["count"])
        b = fl = 0.0
        for _ in range(case["count"]):
            u = torch.rand(2, generator=sizes, dtype=F64).tolist()
            n = int(round(case["side_lo"] * (case["side_hi"] / case["side_lo"]) ** u[0]))
            np_ = n * n * (2 + int(15 * u[1]))
            b += np_ * 4 * (2 + case["fields"]) + 4 * case["fields"] * n * n
            fl += np_ * (30 + 6 * case["fields"])
        return dict(bytes=b, flops=fl)
    nn = case["nx"] * case.get("ny", 1)
    np_, F = nn * case["ppc"], case.get("fields", 2)
    e = 8 if kind.startswith("exact") or case.get("dtype") == "f64" else 4
    d = 1 if kind == "exact1d" or case.get("dim") == 1 else 2
    moved = 2 * d if kind == "fluid" else d     # positions in; the fluid step writes new ones
    return dict(bytes=float(e * (np_ * (moved + 2 * F) + nn * F)),
                flops=float(np_ * (60 + 24 * F) + nn * 20 * F))


# ----------------------------------------------------------------------------
# the same in 64 bits, plain torch
# ----------------------------------------------------------------------------
def _locate(x, n, length):
    t = x * (n / length)
    c = torch.floor(t)
    return c.long() % n, t - c


def _corners(x, y, nx, ny, lx, ly):
    """Node numbers [4, np] and P1 weights [4, np] of the "/"-split square (corner 00, 10, 11, 01)."""
    i, a = _locate(x, nx, lx)
    j, b = _locate(y, ny, ly)
    ip, jp = (i + 1) % nx, (j + 1) % ny
    low = a >= b
    zero = torch.zeros_like(a)
    w = torch.stack([1 - torch.maximum(a, b), torch.where(low, a - b, zero), torch.minimum(a, b),
                     torch.where(low, zero, b - a)])
    return torch.stack([i + nx * j, ip + nx * j, ip + nx * jp, i + nx * jp]), w


def _interp(nodal, x, y, nx, ny, lx, ly):
    k, w = _corners(x, y, nx, ny, lx, ly)
    return sum(nodal[:, k[c]] * w[c] for c in range(4))


def _cg(matvec, diag, b, x):
    """Diagonally preconditioned CG on every row of b, to a relative residual of 1e-15."""
    stop = (1e-15 * b.norm(dim=1)) ** 2
    r = b - matvec(x)
    z = r / diag
    p, rz = z.clone(), (r * z).sum(1)
    for it in range(2000):
        q = matvec(p)
        pq = (p * q).sum(1)
        a = torch.where(pq > 0, rz / pq, torch.zeros_like(pq))[:, None]
        x = x + a * p
        r = r - a * q
        if it % 4 == 3 and bool(((r * r).sum(1) <= stop).all()):
            break
        z = r / diag
        new = (r * z).sum(1)
        p = z + torch.where(rz > 0, new / rz, torch.zeros_like(rz))[:, None] * p
        rz = new
    return x


def _p2m(x, y, vals, nx, ny, lx, ly, mass):
    """FLIP or the mass assignment with the particle quadrature, uniform volumes."""
    nn, vol = nx * ny, lx * ly / x.numel()
    k, w = _corners(x, y, nx, ny, lx, ly)
    b = torch.zeros(vals.shape[0], nn, dtype=F64, device=DEV)
    s = torch.zeros(nn, dtype=F64, device=DEV)
    m = torch.zeros(4, nn, dtype=F64, device=DEV)   # diagonal, +x, +y, +x+y
    for c in range(4):
        s.index_add_(0, k[c], vol * w[c])
        for f in range(vals.shape[0]):
            b[f].index_add_(0, k[c], vol * w[c] * vals[f])
        if mass:
            m[0].index_add_(0, k[c], vol * w[c] * w[c])
    if not mass:
        return torch.where(s > 0, b / s, torch.zeros_like(b))
    for q, u, v in ((1, 0, 1), (1, 3, 2), (2, 0, 3), (2, 1, 2), (3, 0, 2)):
        m[q].index_add_(0, k[u], vol * w[u] * w[v])
    m = m.reshape(4, ny, nx)
    empty = s == 0
    diag = torch.where(empty, torch.ones_like(s), m[0].reshape(-1))

    def matvec(p):
        g = p.reshape(-1, ny, nx)
        out = diag.reshape(ny, nx) * g
        for q, dy, dx in ((1, 0, 1), (2, 1, 0), (3, 1, 1)):
            out = out + m[q] * torch.roll(g, (-dy, -dx), (1, 2)) + torch.roll(m[q] * g, (dy, dx), (1, 2))
        return out.reshape(p.shape)
    return _cg(matvec, diag, b, torch.where(empty, torch.zeros_like(b), b / s))


def _p2m_1d(x, vals, n):
    i, a = _locate(x, n, 1.0)
    j, vol = (i + 1) % n, 1.0 / x.numel()
    b = torch.zeros(vals.shape[0], n, dtype=F64, device=DEV)
    s, d, e = (torch.zeros(n, dtype=F64, device=DEV) for _ in range(3))
    for k, w in ((i, 1 - a), (j, a)):
        s.index_add_(0, k, vol * w)
        d.index_add_(0, k, vol * w * w)
        for f in range(vals.shape[0]):
            b[f].index_add_(0, k, vol * w * vals[f])
    e.index_add_(0, i, vol * a * (1 - a))
    d = torch.where(s > 0, d, torch.ones_like(d))
    x0 = torch.where(s > 0, b / s, torch.zeros_like(b))
    return _cg(lambda p: d * p + e * torch.roll(p, -1, 1) + torch.roll(e * p, 1, 1), d, b, x0)


def _exact_fluid(case, seed):
    x, y, vel = (t.double() for t in _fluid_inputs(case, seed))
    n, dt = case["nx"], 0.5 / case["nx"]
    h = 1.0 / n
    th = TWO_PI * torch.arange(n, device=DEV, dtype=F64) / n
    K = 4 - 2 * torch.cos(th)[None] - 2 * torch.cos(th)[:, None]

    def solve(r, symbol, zero_mean):
        t = torch.fft.fft2(r.reshape(-1, n, n))
        t = t / torch.where(symbol == 0, torch.ones_like(symbol), symbol)
        if zero_mean:
            t[:, 0, 0] = 0
        return torch.fft.ifft2(t).real

    def grad(p):   # integral of psi_i grad p over the triangles of node i
        p10, p01 = torch.roll(p, -1, -1), torch.roll(p, -1, -2)
        p11 = torch.roll(p10, -1, -2)
        out = []
        for low, up in ((p10 - p, p11 - p01), (p11 - p10, p01 - p)):
            out.append(h / 6 * (low + torch.roll(low, 1, -1) + torch.roll(low, (1, 1), (-2, -1)) + up
                                + torch.roll(up, 1, -2) + torch.roll(up, (1, 1), (-2, -1))))
        return out
    U = _p2m(x, y, vel, n, n, 1.0, 1.0, case["p2m"] == "mass")
    U = solve(U, 1 + dt * NU / h ** 2 * K, False)
    p = solve(-(grad(U[0])[0] + grad(U[1])[1]) / dt, K, True)[0]
    U = (U - dt / h ** 2 * torch.stack(grad(p))).reshape(2, -1)
    new = _interp(U, x, y, n, n, 1.0, 1.0)
    xm, ym = torch.remainder(x + 0.5 * dt * new[0], 1.0), torch.remainder(y + 0.5 * dt * new[1], 1.0)
    mid = _interp(U, xm, ym, n, n, 1.0, 1.0)
    return U, new, torch.remainder(x + dt * mid[0], 1.0), torch.remainder(y + dt * mid[1], 1.0)


def _exact_1d(case, seed):
    """Full mass with the particle hats, Appendix-B rule, both ways."""
    x, vals = _exact1d_inputs(case, seed)
    n, order = case["nx"], torch.argsort(x)
    xs, A = x[order], vals[:, order]
    N, h = xs.numel(), 1.0 / n
    gap = torch.remainder(torch.roll(xs, -1) - xs, 1.0)

    def particle_interp(t):
        k = (torch.searchsorted(xs, t, right=True) - 1) % N
        u = torch.remainder(t - xs[k], 1.0) / gap[k]
        return A[:, k] * (1 - u) + A[:, (k + 1) % N] * u
    grid = torch.arange(n, device=DEV, dtype=F64) * h
    fn, fm = particle_interp(grid), particle_interp(grid + 0.5 * h)
    b = h / 6 * (2 * fn + 2 * fm + 2 * torch.roll(fm, 1, 1))
    th = TWO_PI * torch.arange(n, device=DEV, dtype=F64) / n
    nodal = torch.fft.ifft(torch.fft.fft(b) / (h * (2 + torch.cos(th)) / 3)).real

    def mesh_interp(t):
        i, a = _locate(torch.remainder(t, 1.0), n, 1.0)
        return nodal[:, i] * (1 - a) + nodal[:, (i + 1) % n] * a
    fk, fg = mesh_interp(xs), mesh_interp(xs + 0.5 * gap)
    lo = gap / 6 * (fk + 2 * fg)                              # gap k to its lower end's hat
    hi = torch.roll(gap / 6 * (torch.roll(fk, -1, 1) + 2 * fg), 1, 1)
    d, e = (gap + torch.roll(gap, 1)) / 3, gap / 6
    sol = _cg(lambda p: d * p + e * torch.roll(p, -1, 1) + torch.roll(e * p, 1, 1), d, lo + hi,
              mesh_interp(xs))
    back = torch.empty_like(sol)
    back[:, order] = sol
    return nodal, back


def _delaunay(x, y, nx, ny):
    """Periodic Delaunay stars in the unit box by gift wrapping: neighbour numbers [N, 32]
    counter-clockwise (-1 past the degree) and their offsets [N, 32, 2] from the particle."""
    N, W = x.numel(), 32
    cx, cy = _locate(x, nx, 1.0)[0], _locate(y, ny, 1.0)[0]
    order = torch.argsort(cx + nx * cy)
    count = torch.bincount(cx + nx * cy, minlength=nx * ny)
    start = torch.cumsum(count, 0) - count
    P = int(count.max())
    nbr = torch.full((N, W), -1, dtype=torch.long, device=DEV)
    off = torch.zeros(N, W, 2, dtype=F64, device=DEV)
    left, ring = torch.arange(N, device=DEV), 2
    while left.numel():
        redo, cells = [], (2 * ring + 1) ** 2
        step = max(1, 24_000_000 // (cells * P))
        for k in left.split(step):
            dj, di = torch.meshgrid(*[torch.arange(-ring, ring + 1, device=DEV)] * 2, indexing="ij")
            i, j = cx[k, None] + di.reshape(1, -1), cy[k, None] + dj.reshape(1, -1)
            cell = i % nx + nx * (j % ny)
            s = torch.arange(P, device=DEV)
            ok = (s < count[cell][..., None]).reshape(k.numel(), -1)
            c = order[(start[cell][..., None] + s).clamp(max=N - 1)].reshape(k.numel(), -1)
            sx = torch.floor_divide(i, nx)[..., None].expand(-1, -1, P).reshape(c.shape)
            sy = torch.floor_divide(j, ny)[..., None].expand(-1, -1, P).reshape(c.shape)
            ex, ey = (x[c] + sx) - x[k, None], (y[c] + sy) - y[k, None]
            d2 = ex * ex + ey * ey
            ok &= d2 > 0
            at = torch.where(ok, d2, torch.inf).argmin(1, keepdim=True)
            first, big = at, torch.zeros(k.numel(), dtype=F64, device=DEV)
            done = torch.zeros(k.numel(), dtype=torch.bool, device=DEV)
            for w in range(W):
                ux, uy = ex.gather(1, at), ey.gather(1, at)
                nbr[k, w] = torch.where(done, -1, c.gather(1, at)[:, 0])
                off[k, w] = torch.cat([ux, uy], 1)
                cr = ux * ey - uy * ex
                good = ok & (cr > 0)
                good.scatter_(1, at, False)
                t = torch.where(good, (d2 - ux * ex - uy * ey) / (2 * torch.where(good, cr, 1.0)), torch.inf)
                tm, nxt = t.min(1, keepdim=True)
                radius = ((ux / 2 - tm * uy) ** 2 + (uy / 2 + tm * ux) ** 2).sqrt()[:, 0]
                big = torch.where(done, big, torch.maximum(big, radius))
                done = done | (nxt == first)[:, 0]
                at = nxt
                if bool(done.all()):
                    break
            redo.append(k[~done | ~(2 * big <= ring * min(1.0 / nx, 1.0 / ny))])
        left, ring = torch.cat(redo), ring + 1
        nbr[left], off[left] = -1, 0.0
        if ring > 9:
            raise RuntimeError("a Voronoi cell does not close")
    return nbr, off


def _exact_2d(case, seed):
    """Full mass on the particle triangulation, Appendix-B rule, both ways."""
    x, y, A = _exact2d_inputs(case, seed)
    nx, ny = case["nx"], case["ny"]
    N, F = x.numel(), A.shape[0]
    nbr, off = _delaunay(x, y, nx, ny)
    has = nbr >= 0
    deg = has.sum(1)
    nxt = torch.where(torch.arange(32, device=DEV)[None] + 1 < deg[:, None], torch.arange(1, 33, device=DEV)[None],
                      0).clamp(max=31)
    nb2 = nbr.gather(1, nxt)
    off2 = off.gather(1, nxt[..., None].expand(-1, -1, 2))
    area = torch.where(has, 0.5 * (off[..., 0] * off2[..., 1] - off[..., 1] * off2[..., 0]), 0.0)
    # the particle interpolant on the half-spacing grid: every triangle once, its grid points
    k, w = torch.nonzero(has & (torch.arange(N, device=DEV)[:, None] < nbr)
                         & (torch.arange(N, device=DEV)[:, None] < nb2), as_tuple=True)
    gx, gy = 0.5 / nx, 0.5 / ny
    ax, ay = off[k, w, 0], off[k, w, 1]
    bx, by = off2[k, w, 0], off2[k, w, 1]
    det = ax * by - ay * bx
    tri = torch.stack([k, nbr[k, w], nb2[k, w]])
    zero = torch.zeros_like(ax)
    i0 = torch.ceil((x[k] + torch.minimum(torch.minimum(ax, bx), zero)) / gx - 1e-9)
    j0 = torch.ceil((y[k] + torch.minimum(torch.minimum(ay, by), zero)) / gy - 1e-9)
    i1 = torch.floor((x[k] + torch.maximum(torch.maximum(ax, bx), zero)) / gx + 1e-9)
    j1 = torch.floor((y[k] + torch.maximum(torch.maximum(ay, by), zero)) / gy + 1e-9)
    H = torch.full((F, 2 * ny, 2 * nx), torch.nan, dtype=F64, device=DEV)
    for dj in range(int((j1 - j0).max()) + 1):
        for di in range(int((i1 - i0).max()) + 1):
            q = torch.nonzero((i0 + di <= i1) & (j0 + dj <= j1))[:, 0]
            px, py = (i0[q] + di) * gx - x[k[q]], (j0[q] + dj) * gy - y[k[q]]
            u = (px * by[q] - py * bx[q]) / det[q]
            v = (ax[q] * py - ay[q] * px) / det[q]
            inside = (u >= -1e-11) & (v >= -1e-11) & (u + v <= 1 + 1e-11)
            q, u, v = q[inside], u[inside], v[inside]
            t = tri[:, q]
            H[:, (j0[q] + dj).long() % (2 * ny), (i0[q] + di).long() % (2 * nx)] = (
                A[:, t[0]] * (1 - u - v) + A[:, t[1]] * u + A[:, t[2]] * v)
    n00, mx, my, mxy = H[:, ::2, ::2], H[:, ::2, 1::2], H[:, 1::2, ::2], H[:, 1::2, 1::2]
    e, n = (lambda t: torch.roll(t, -1, 2)), (lambda t: torch.roll(t, -1, 1))
    T = 0.5 / (nx * ny)
    b = torch.zeros(F, ny, nx, dtype=F64, device=DEV)

    def rule(a, p, q, ap, aq, pq):
        return T * (a / 30 - (p + q) / 60 + 2 * (ap + aq) / 15 + pq / 15)
    n10, n01, n11 = e(n00), n(n00), e(n(n00))
    for va, vb, vc, mab, mac, mbc, sb, sc in (
            (n00, n10, n11, mx, mxy, e(my), (0, 1), (1, 1)),     # lower triangle 00, 10, 11
            (n00, n11, n01, mxy, my, n(mx), (1, 1), (1, 0))):    # upper triangle 00, 11, 01
        b += rule(va, vb, vc, mab, mac, mbc)
        b += torch.roll(rule(vb, va, vc, mab, mbc, mac), sb, (1, 2))
        b += torch.roll(rule(vc, va, vb, mac, mbc, mab), sc, (1, 2))
    tx = TWO_PI * torch.arange(nx, device=DEV, dtype=F64)[None] / nx
    ty = TWO_PI * torch.arange(ny, device=DEV, dtype=F64)[:, None] / ny
    symbol = (0.5 + (torch.cos(tx) + torch.cos(ty) + torch.cos(tx + ty)) / 6) / (nx * ny)
    nodal = torch.fft.ifft2(torch.fft.fft2(b) / symbol).real.reshape(F, -1)

    def mesh(px, py):
        return _interp(nodal, torch.remainder(px, 1.0), torch.remainder(py, 1.0), nx, ny, 1.0, 1.0)
    c, at = torch.zeros(F, N, dtype=F64, device=DEV), mesh(x, y)
    for w in range(int(deg.max())):
        o, p = off[:, w], off2[:, w]
        v = (at / 30 - (mesh(x + o[:, 0], y + o[:, 1]) + mesh(x + p[:, 0], y + p[:, 1])) / 60
             + 2 * (mesh(x + o[:, 0] / 2, y + o[:, 1] / 2) + mesh(x + p[:, 0] / 2, y + p[:, 1] / 2)) / 15
             + mesh(x + (o[:, 0] + p[:, 0]) / 2, y + (o[:, 1] + p[:, 1]) / 2) / 15)
        c += area[:, w] * v
    diag = area.sum(1) / 6
    width = int(deg.max())
    col, wa = nbr[:, :width].clamp(min=0), area[:, :width] / 12
    wb = torch.zeros_like(wa).scatter_add_(1, nxt[:, :width].clamp(max=width - 1), wa)

    def matvec(p):
        out = diag * p
        for w in range(width):
            out = out + (wa[:, w] + wb[:, w]) * p[:, col[:, w]]
        return out
    return nodal, _cg(matvec, diag, c, at)


def _exact_train(case, seed):
    X, target, params, m, v, rows = _train_inputs(case, seed)
    th = params.double().requires_grad_(True)
    H, NI = B.LEARNED_HIDDEN, B.LEARNED_NIN
    w1, b1, w2, b2, w3, b3, w4, b4 = th.split([H * NI, H, H * H, H, H * H, H, H, 1])
    h = torch.relu(X[rows.long()].double() @ w1.reshape(H, NI).t() + b1)
    h = torch.relu(h @ w2.reshape(H, H).t() + b2)
    h = torch.relu(h @ w3.reshape(H, H).t() + b3)
    loss = ((h @ w4 + b4 - target[rows.long()].double()) ** 2).mean()
    loss.backward()
    g, t = th.grad, TRAIN_STEP + 1
    m = 0.9 * m.double() + 0.1 * g
    v = 0.999 * v.double() + 0.001 * g * g
    new = th.detach() - TRAIN_LR * (m / (1 - 0.9 ** t)) / ((v / (1 - 0.999 ** t)).sqrt() + 1e-8)
    return loss.detach().reshape(1), g, new, m, v


def exact(case, seed):
    kind = case["kind"]
    if kind == "step":
        x, y, vals, lx, ly = _step_inputs(case, seed)
        x, vals, n = x.double(), vals.double(), case["nx"]
        if case["dim"] == 1:
            nodal = _p2m_1d(x, vals, n)
            i, a = _locate(x, n, 1.0)
            return nodal, nodal[:, i] * (1 - a) + nodal[:, (i + 1) % n] * a
        y = y.double()
        nodal = _p2m(x, y, vals, n, case["ny"], lx, ly, case["p2m"] == "mass")
        return nodal, _interp(nodal, x, y, n, case["ny"], lx, ly)
    if kind == "batch":
        return [_p2m(x.double(), y.double(), v.double(), n, n, TWO_PI, TWO_PI, True)
                for n, x, y, v in _batch_inputs(case, seed)]
    if kind == "fluid":
        return _exact_fluid(case, seed)
    if kind == "exact1d":
        return _exact_1d(case, seed)
    if kind == "exact2d":
        return _exact_2d(case, seed)
    return _exact_train(case, seed)
