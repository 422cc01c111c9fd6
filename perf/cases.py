"""Performance cases of the DDPS solver: what its users have it do.

Every case builds a sparse system on the GPU from a seed (matrix coefficients
and the solution x* both follow the seed), sets up a `Solver` on it and runs
one pass through the public entry points: a solve with kept factors, or a
whole step (new matrix values, factorisation, solve), or one epoch of the
learned guess's training.

kind        system
grid2d      upwind convection-diffusion on nx x ny, slabs of whole grid rows
            ("rows" each, or uneven heights lo..hi)
euler2d     one implicit Euler step of a rotating convection-diffusion problem
grid3d      7-point upwind convection-diffusion on nx x ny x nz
diff3d      7-point lognormal diffusion with a reaction term on nx x ny x nz
mesh        a randomly triangulated mesh with shuffled numbering, reordered
            and partitioned by GeneralSystem
guess       the learned guess's network (4t+2 -> 512 -> 512 -> 512 -> 2t)

op "solve": factors kept, one solve of k right-hand sides.
op "step": refactor_values + factor + solve, as a time step or a Newton step
does.
"""
import functools
import math

import numpy as np
import torch

from paper_1008_1700_amd import ddps

DEV = "cuda"


def listed():
    return [
        # the smallest call: one right-hand side on a 64 x 64 grid, factors kept; launches and host waits count
        dict(name="solve_small", kind="grid2d", op="solve", nx=64, ny=64, rows=16, k=1, dtype="f64", tol=1e-10,
             inner_tol=1e-12),
        # a whole step of a small ragged system (odd plane, uneven slabs): many short launches
        dict(name="step_small_ragged", kind="grid2d", op="step", nx=93, ny=121, lo=3, hi=17, k=2, dtype="f64",
             tol=1e-11, inner_tol=1e-12),
        # one step of an implicit time integration, 64 slabs of 16 grid rows, mixed precision
        dict(name="euler_step", kind="euler2d", op="step", nx=1024, ny=1024, rows=16, k=1, dtype="bf16x3", tol=1e-12,
             inner_tol=1e-6),
        # the paper's method in plain FP64, one right-hand side, spikes kept
        dict(name="step_3d_f64", kind="grid3d", op="step", nx=32, ny=32, nz=512, planes=8, k=1, dtype="f64",
             tol=1e-10, inner_tol=1e-9),
        # the same system in mixed precision
        dict(name="step_3d_mixed", kind="grid3d", op="step", nx=32, ny=32, nz=512, planes=8, k=1, dtype="bf16x3",
             tol=1e-11, inner_tol=1e-6),
        # the benchmark's system at a quarter of its length: mixed precision, 8 right-hand sides
        dict(name="step_diff_mixed_8rhs", kind="diff3d", op="step", nx=40, ny=40, nz=1024, planes=8, k=8,
             dtype="bf16x3", tol=1e-10, inner_tol=1e-4, inner_prec=1),
        # plain FP64 on the same cross-section: spike tips only, retrieval by a second block solve
        dict(name="step_diff_f64_tips", kind="diff3d", op="step", nx=40, ny=40, nz=256, planes=8, k=8, dtype="f64",
             tol=1e-11, inner_tol=1e-9, retrieval=1),
        # uneven slabs of a wide 2D grid in FP32 (tall blocks, a band that is no multiple of the tile)
        dict(name="step_uneven_f32", kind="euler2d", op="step", nx=1500, ny=420, lo=4, hi=28, k=1, dtype="f32",
             tol=1e-12, inner_tol=1e-6),
        # many right-hand sides against kept factors: 5 columns (an odd count), odd plane
        dict(name="solve_5rhs_mixed", kind="diff3d", op="solve", nx=33, ny=37, nz=512, planes=8, k=5,
             dtype="bf16x3", tol=1e-10, inner_tol=1e-4, inner_prec=1),
        # a general sparse matrix with a drop tolerance: outer BiCGStab
        dict(name="step_mesh_drop", kind="mesh", op="step", nx=250, ny=240, p=16, k=1, dtype="f64", tol=1e-11,
             inner_tol=1e-10, delta=0.1, outer="bicgstab", sigma=1.0),
        # incomplete block factors: cheap factorisation, many outer iterations, 8 right-hand sides
        dict(name="step_ilu_8rhs", kind="grid3d", op="step", nx=32, ny=32, nz=256, planes=8, k=8, dtype="f32",
             tol=1e-12, inner_tol=1e-4, inner_prec=1, retrieval=1, block_factor="ilu0", outer="bicgstab"),
        # one epoch of the learned guess's training: 32 minibatches of 512 interface pairs
        dict(name="guess_epoch", kind="guess", op="train", t=1024, batch=512, steps=32, lr=1e-3),
    ]


def _log(rng, a, b):
    return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))


def draw(rng):
    kind = rng.choice(["grid2d", "grid2d", "euler2d", "grid3d", "diff3d", "diff3d", "mesh", "ilu", "guess"])
    if kind == "guess":
        return dict(kind="guess", op="train", t=64 * _log(rng, 1, 20), batch=_log(rng, 40, 700),
                    steps=_log(rng, 4, 32), lr=1e-3)
    op = rng.choice(["solve", "step", "step"])
    k = rng.choice([1, 1, 2, 3, 5, 8])
    dtype = rng.choice(["f64", "f32", "bf16x3", "bf16x3"])
    c = dict(kind=kind, op=op, k=k, dtype=dtype, tol=1e-11, inner_tol=1e-9 if dtype == "f64" else 1e-5)
    # factor flops are about 8 n b^2: bounded per type so that no drawn case costs more than the largest listed one
    most = {"f64": 4e12, "f32": 5e12, "bf16x3": 2e13}[dtype]
    if kind in ("grid2d", "euler2d"):
        nx = _log(rng, 40, 200 if kind == "grid2d" else 1400)
        rows = max(rng.randint(4, 20), -(-2 * 64 * -(-nx // 64) // nx))
        p = max(2, min(_log(rng, 2, 64), int(most / (8.0 * nx * rows * nx * nx))))
        c.update(nx=nx, ny=rows * p, rows=rows, tol=1e-12)
        if rng.random() < 0.4:
            del c["rows"]
            c.update(lo=max(3, -(-2 * 64 * -(-nx // 64) // nx)), hi=max(12, rows))
        return c
    if kind in ("grid3d", "diff3d", "ilu"):
        nx, ny = _log(rng, 9, 40), _log(rng, 9, 40)
        b = nx * ny
        planes = max(rng.randint(4, 10), -(-2 * 64 * -(-b // 64) // b))
        p = max(2, min(_log(rng, 2, 96), int(most / (8.0 * b * planes * b * b))))
        c.update(nx=nx, ny=ny, nz=planes * p, planes=planes)
        if kind == "ilu":
            c.update(kind="grid3d", op="step", nz=planes * min(p, 24), dtype="f32", tol=1e-12, inner_tol=1e-4,
                     inner_prec=1, retrieval=1, block_factor="ilu0", outer="bicgstab")
        elif k > 2:
            c["inner_prec"] = 1
        if kind == "diff3d" and dtype == "f64":
            c["retrieval"] = rng.choice([0, 1])
        return c
    nx = _log(rng, 60, 240)
    c.update(nx=nx, ny=_log(rng, nx, 2 * nx), p=rng.randint(4, 16), k=1, dtype=rng.choice(["f64", "bf16x3"]), tol=1e-11,
             inner_tol=1e-10, delta=rng.choice([0.01, 0.1, 0.3]), outer="bicgstab", sigma=1.0)
    return c


# ---------------------------------------------------------------- systems
class System:
    """CSR arrays on the host, as Solver takes them."""

    def __init__(self, n, row_ptr, col, val):
        self.n, self.row_ptr, self.col, self.val = n, row_ptr, col, val


@functools.lru_cache(maxsize=32)
def _pattern(nx, ny, nz):
    """Row pointers and columns of the 5- or 7-point stencil (x fastest), the
    offsets in column order and which of them each row has (on the GPU)."""
    n = nx * ny * nz
    i = torch.arange(n, device=DEV)
    ix, iy, iz = i % nx, (i // nx) % ny, i // (nx * ny)
    offs = [(-nx * ny, iz > 0), (-nx, iy > 0), (-1, ix > 0), (0, ix >= 0), (1, ix < nx - 1), (nx, iy < ny - 1),
            (nx * ny, iz < nz - 1)]
    if nz == 1:
        offs = offs[1:-1]
    has = torch.stack([m for _, m in offs], dim=1)
    cols = i[:, None] + torch.tensor([o for o, _ in offs], device=DEV)[None, :]
    row_ptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(has.sum(dim=1).cpu().numpy(), out=row_ptr[1:])
    return row_ptr, cols[has].to(torch.int32).cpu().numpy(), [o for o, _ in offs], has


def _upwind(v, h):
    a = abs(v) * h
    return -1.0 - (a if v > 0 else 0.0), -1.0 - (a if v < 0 else 0.0), 2.0 + a


def _coefficients(c, g):
    """(n, offsets) stencil coefficients, h^2-scaled; random parts from g."""
    nx, ny, nz = c["nx"], c["ny"], c.get("nz", 1)
    h = 1.0 / (nx + 1)
    _, _, offs, has = _pattern(nx, ny, nz)
    n = has.shape[0]
    if c["kind"] == "diff3d":
        a = torch.exp(torch.randn(n, generator=g, device=DEV, dtype=torch.float64))
        pad = nx * ny
        ap = torch.ones(n + 2 * pad, device=DEV, dtype=torch.float64)
        ap[pad:pad + n] = a
        co, diag = torch.empty(n, len(offs), device=DEV, dtype=torch.float64), torch.full_like(a, 0.1 * h * h)
        for q, o in enumerate(offs):
            if o == 0:
                continue
            nb = ap[pad + o:pad + o + n]
            t = torch.where(has[:, q], 2.0 * a * nb / (a + nb), 2.0 * a)
            co[:, q] = -t
            diag += t
        co[:, offs.index(0)] = diag
        return co
    # convection with the seed's velocity direction; the time step's matrix is I + dt L
    u = torch.rand(2, generator=g, device=DEV, dtype=torch.float64).cpu().tolist()
    th = 2.0 * math.pi * u[0]
    speed = {"grid2d": 28.0, "euler2d": 50.0, "grid3d": 10.0}[c["kind"]]
    x, y = _upwind(speed * math.cos(th), h), _upwind(speed * math.sin(th), h)
    z = _upwind(10.0 * u[1], h)
    row = [y[0], x[0], x[2] + y[2], x[1], y[1]]
    if nz > 1:
        row = [z[0], y[0], x[0], x[2] + y[2] + z[2], x[1], y[1], z[1]]
    if c["kind"] == "euler2d":
        row = [v * 1e-3 / (h * h) for v in row]
        row[2] += 1.0
    return torch.tensor(row, device=DEV, dtype=torch.float64).expand(n, len(row))


def _heights(total, lo, hi):
    """Uneven slab heights lo..hi, the same for every seed."""
    r, out = np.random.RandomState(2), []
    while total > hi:
        out.append(int(r.randint(lo, min(hi, total - lo) + 1)))
        total -= out[-1]
    return out + [total]


def _stencil(c, g):
    """System, partition, x* (k, n) and f = A x* (k, n) of a stencil case."""
    nx, ny, nz = c["nx"], c["ny"], c.get("nz", 1)
    row_ptr, col, offs, has = _pattern(nx, ny, nz)
    n = has.shape[0]
    co = torch.where(has, _coefficients(c, g), 0.0)
    if "lo" in c:
        heights = _heights(ny, c["lo"], c["hi"])
    else:
        per = c["planes"] if nz > 1 else c["rows"]
        heights = [per] * ((nz if nz > 1 else ny) // per)
    part = np.concatenate([[0], np.cumsum(heights)]).astype(np.int64) * (nx * ny if nz > 1 else nx)
    xs = torch.rand(c["k"], n, generator=g, device=DEV, dtype=torch.float64) * 2 - 1
    pad = max(offs)
    xp = torch.nn.functional.pad(xs, (pad, pad))
    f = torch.zeros_like(xs)
    for q, o in enumerate(offs):
        f += co[:, q] * xp[:, pad + o:pad + o + n]
    return System(n, row_ptr, col, co[has].cpu().numpy()), part, xs, f


@functools.lru_cache(maxsize=8)
def _mesh_pattern(nx, ny):
    """Edges (both directions) of an nx x ny lattice with one random diagonal
    per cell, under a random numbering; sorted by row, then column."""
    r = np.random.RandomState(7)
    i = np.arange(nx * ny).reshape(ny, nx)
    flip = r.rand(ny - 1, nx - 1) < 0.5
    a = [i[:, :-1].ravel(), i[:-1].ravel(), np.where(flip, i[:-1, :-1], i[:-1, 1:]).ravel()]
    b = [i[:, 1:].ravel(), i[1:].ravel(), np.where(flip, i[1:, 1:], i[1:, :-1]).ravel()]
    new = r.permutation(nx * ny)
    a, b = new[np.concatenate(a)], new[np.concatenate(b)]
    d = np.arange(nx * ny)
    row, col = np.concatenate([a, b, d]), np.concatenate([b, a, d])
    order = np.lexsort((col, row))
    row, col = row[order], col[order]
    row_ptr = np.zeros(nx * ny + 1, dtype=np.int64)
    np.cumsum(np.bincount(row, minlength=nx * ny), out=row_ptr[1:])
    return row, row_ptr, col.astype(np.int32)


def _mesh(c, seed):
    r = np.random.RandomState(seed % (1 << 31))
    row, row_ptr, col = _mesh_pattern(c["nx"], c["ny"])
    n = len(row_ptr) - 1
    off = row != col
    val = np.where(off, -np.exp(c["sigma"] * r.randn(len(row))), 0.0)
    rs = np.bincount(row, weights=-val, minlength=n)
    cs = np.bincount(col, weights=-val, minlength=n)
    val[~off] = np.maximum(rs, cs) + 0.02 + 0.02 * r.rand(n)
    xs = r.uniform(-1.0, 1.0, n)
    f = np.bincount(row, weights=val * xs[col], minlength=n)
    gs = ddps.GeneralSystem(n, row_ptr, col, val, c["p"])
    xs, f = (torch.from_numpy(np.ascontiguousarray(gs.to_perm(v)))[None, :].to(DEV) for v in (xs, f))
    return gs, gs.part_ptr, xs, f


def _system(c, seed):
    if c["kind"] == "mesh":
        return _mesh(c, seed)
    return _stencil(c, torch.Generator(device=DEV).manual_seed(int(seed)))


# ---------------------------------------------------------------- the passes
class Net:
    """The network's handle and one epoch of training pairs."""

    def __init__(self, c, seed):
        g = torch.Generator(device=DEV).manual_seed(int(seed))
        t, b, s = c["t"], c["batch"], c["steps"]
        self.X = torch.randn(s, b, 4 * t + 2, generator=g, device=DEV)
        self.T = 0.25 * torch.randn(s, b, 2 * t, generator=g, device=DEV)
        self.h = ddps.ddps_mlp_create(4 * t + 2, 512, 2 * t, b, seed=int(seed),
                                      stream=torch.cuda.current_stream().cuda_stream)

    def __del__(self):
        ddps.ddps_mlp_destroy(self.h)


def prepare(case, seed):
    c = case
    if c["kind"] == "guess":
        return dict(case=c, net=Net(c, seed))
    A, part, xs, f = _system(c, seed)
    S = ddps.Solver(A, part, dtype=c["dtype"], delta=c.get("delta", 0.0), inner_tol=c["inner_tol"],
                    outer=c.get("outer", "refine"), max_rhs=c["k"], inner_prec=c.get("inner_prec", 0),
                    retrieval=c.get("retrieval", 0), block_factor=c.get("block_factor", "lu"))
    val = S.val.clone()
    if c["op"] == "solve":
        S.factor()
    return dict(case=c, S=S, val=val, f=f, x=torch.zeros_like(f))


def run(state):
    c = state["case"]
    if c["kind"] == "guess":
        net = state["net"]
        for s in range(c["steps"]):
            ddps.ddps_mlp_train_step(net.h, c["batch"], net.X[s], net.T[s], c["lr"], want_loss=False)
        return ddps.ddps_mlp_get_params(net.h)
    S, f, x = state["S"], state["f"], state["x"]
    if c["op"] == "step":
        ddps.ddps_refactor_values(S.h, state["val"])
        S.factor()
    if c["k"] == 1:
        S.solve(f, x, c["tol"])
    else:
        ddps.ddps_solve_many(S.h, f, x, c["tol"])
    return x


def exact(case, seed):
    """x*: f was formed from it, so it solves the system up to the rounding of f."""
    if case["kind"] == "guess":
        return None   # rounded weights after an epoch of Adam have no value in 64 bits
    return _system(case, seed)[2]


def work(case):
    """A step cannot do without the band LU of the blocks (2 n b^2 flops), the
    spikes (6 n b^2) and the CSR, right-hand sides and solutions once; a solve
    with kept factors reads the band factors and the spikes once."""
    c = case
    if c["kind"] == "guess":
        t, b, s = c["t"], c["batch"], c["steps"]
        d, params = 6 * t + 2, (6 * t + 2) * 512 + 2 * 512 * 512 + 3 * 512 + 2 * t
        # forward and weight gradients of every layer, input gradients of all but the first
        flops = s * b * 2.0 * (3 * (d * 512 + 2 * 512 * 512) - (4 * t + 2) * 512)
        return {"bytes": s * (4.0 * b * d + 28.0 * params), "flops": flops}
    n = c["nx"] * c["ny"] * c.get("nz", 1)
    k, elt = c["k"], 8 if c["dtype"] == "f64" else 4
    b = c["nx"] * (c["ny"] if c.get("nz", 1) > 1 else 1)
    nnz = n * (5 if c.get("nz", 1) == 1 else 7)
    if c["kind"] == "mesh":
        b, nnz = min(c["nx"], c["ny"]), 7 * n
    io = 12.0 * nnz + 8.0 * n + 16.0 * n * k
    if c.get("block_factor") == "ilu0":
        return {"bytes": io + 4.0 * n * b, "flops": 4.0 * nnz * b}
    if c["op"] == "solve":
        return {"bytes": io + 4.0 * n * b * elt, "flops": 8.0 * n * b * k}
    return {"bytes": io, "flops": 8.0 * n * b * b}
