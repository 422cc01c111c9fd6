"""The solve phase's products where their dispatch changes: launches below and
above the counts at which a workgroup takes fewer waves or fewer rows, packed
tip rows of one to four pieces per wave, the longest packed rows, and
reductions taken up by the kernels that read them or by a kernel of their own.
Checked against float64 on the host."""
import numpy as np
import pytest

from tests.gpu_util import dev_vec, host, torch_cuda
from workloads import pde

pytestmark = pytest.mark.gpu

UNIT = {"f64": 2.0 ** -53, "f32": 2.0 ** -24}


def system(p, t, seed):
    """p blocks of 2t, 2t + 1, ... rows, five diagonals at 0, +-1, +-t."""
    rng = np.random.default_rng(seed)
    sizes = 2 * t + np.arange(p) % 3
    part = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    n = int(part[-1])
    row = np.arange(n)
    offs = [-t, -1, 0, 1, t]
    vals = [rng.uniform(-1, 1, n) for _ in offs]
    vals[2] = rng.uniform(4, 5, n)
    return pde.stencil_csr(n, offs, vals, [(row + o >= 0) & (row + o < n) for o in offs]), part


# 2 (p - 1) t / 64 workgroups per reduced product, p t / 64 per sweep step
@pytest.mark.parametrize("p,t", [(2, 64), (3, 192), (2, 2048), (9, 512), (17, 512), (18, 512), (33, 512), (10, 1024),
                                 (7, 1536), (6, 2048), (1100, 64), (2100, 64)])
@pytest.mark.parametrize("dtype,k", [("f64", 1), ("f64", 2), ("f64", 5), ("f32", 1), ("f32", 2), ("f32", 5)])
def test_products_at_dispatch_edges(p, t, dtype, k):
    from paper_1008_1700_amd import ddps
    torch = torch_cuda()
    A, part = system(p, t, 10 * p + t)
    As = A.scipy()
    S = ddps.Solver(A, part, dtype=dtype, max_rhs=k, inner_tol=1e-8)
    try:
        S.factor()
        m, ts, _ = ddps.ddps_reduced_layout(S.h)
        assert ts == t and m == 2 * (p - 1) * t
        mask = torch.empty(m, dtype=torch.float64, device="cuda")
        ddps.ddps_reduced_layout(S.h, torch.empty(m, dtype=torch.int64, device="cuda"), mask)
        on = host(mask) > 0
        rng = np.random.default_rng(t)
        # reduced product: an error bound of sums of 2t + 1 products on the stored spikes
        X = rng.uniform(-1, 1, (k, m)) * on
        V = torch.empty(k, m, dtype=torch.float64, device="cuda")
        ddps.ddps_reduced_matvec(S.h, k, dev_vec(X), V)
        V = host(V)
        u = UNIT["f64"] if k <= 2 else UNIT[dtype]
        Xp = np.concatenate([np.zeros((k, t)), X, np.zeros((k, t))], axis=1)
        some = {0, 1, p // 2, p - 2, p - 1} if p > 32 else set(range(p))
        for i in sorted(some):
            N = int(part[i + 1] - part[i])
            G = torch.empty(2 * t, N, dtype=torch.float64, device="cuda")
            ddps.ddps_get_spikes(S.h, i, G)
            G = host(G).T
            # values on c beside block i: the last t rows of block i-1, the first t rows of block i+1
            lo = (2 * i - 1) * t if i else 0
            xl = Xp[:, lo:lo + t] if i else np.zeros((k, t))
            xr = Xp[:, (2 * i + 2) * t:(2 * i + 3) * t] if i < p - 1 else np.zeros((k, t))
            x = np.concatenate([xl, xr], axis=1)
            for half, rows in ((0, G[:t]), (1, G[N - t:])):
                if (half == 0 and i == 0) or (half == 1 and i == p - 1):
                    continue
                ro = (2 * i - 1 + half) * t
                sel = on[ro:ro + t]
                exp = X[:, ro:ro + t] + x @ rows.T
                bound = (2 * t + 4) * u * (np.abs(X[:, ro:ro + t]) + np.abs(x) @ np.abs(rows).T)
                assert np.all((np.abs(V[:, ro:ro + t] - exp) <= bound)[:, sel])
        # block solves: normwise backward error of the block diagonal
        Y = rng.uniform(-1, 1, (k, A.n))
        g = torch.empty(k, A.n, dtype=torch.float64, device="cuda")
        ddps.ddps_block_solve(S.h, k, dev_vec(Y), g)
        g = host(g)
        C = As.tocoo()
        own = np.searchsorted(part, C.row, "right") == np.searchsorted(part, C.col, "right")
        D = type(C)((C.data[own], (C.row[own], C.col[own])), shape=C.shape).tocsr()
        nd = np.max(np.abs(D).sum(axis=1))
        back = np.linalg.norm((D @ g.T).T - Y, axis=1) / (nd * np.linalg.norm(g, axis=1))
        print(f"p {p} t {t} {dtype} k {k}: block solve {back.max():.2e}")
        assert back.max() <= 128 * UNIT[dtype]
        # full solves: the reductions steer both iterations
        Xs = rng.uniform(-1, 1, (k, A.n))
        Z = torch.zeros(k, A.n, dtype=torch.float64, device="cuda")
        rc, info = ddps.ddps_solve_many(S.h, dev_vec((As @ Xs.T).T), Z, 1e-11)
        assert rc == 0 and info.relres_inf <= 1e-11
        assert np.max(np.abs(host(Z) - Xs)) <= 1e-8
    finally:
        S.close()
