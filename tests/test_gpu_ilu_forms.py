"""Incomplete factors at the edges of their kernels: blocks that just fit in
LDS and blocks that do not, levels of one row up to more rows than a workgroup
has threads, rows with more entries than the held ones, near and far spike
entries.  Diagonals 0, +-d alone give no fill, so there ILU(0) is the exact
factorisation and the block solve is checked by its backward error; general
patterns are checked against the oracle."""
import numpy as np
import pytest

from tests.gpu_util import dev_vec, host, make_solver, relerr, torch_cuda
from workloads import pde

pytestmark = pytest.mark.gpu


def system(sizes, offs, seed):
    rng = np.random.default_rng(seed)
    part = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    n = int(part[-1])
    row = np.arange(n)
    vals = [rng.uniform(-1, 1, n) if o else rng.uniform(1.5, 2, n) * (len(offs) - 1) for o in offs]
    A = pde.stencil_csr(n, offs, vals, [(row + o >= 0) & (row + o < n) for o in offs])
    return dict(A=A, part_ptr=part)


@pytest.mark.parametrize("d,sizes", [(1, [20479, 300]), (1, [20480, 300]), (40, [257, 900, 511]), (190, [777, 400]),
                                     (300, [1300, 701]), (700, [2801, 1409]), (1500, [3100, 5001])])
@pytest.mark.parametrize("k", [1, 3])
def test_block_solve_without_fill(d, sizes, k):
    from paper_1008_1700_amd import ddps
    torch = torch_cuda()
    s = system(sizes, [-d, 0, d], d)
    A, part = s["A"], s["part_ptr"]
    S = make_solver(s, dtype="f64", max_rhs=k, retrieval=1, block_factor="ilu0", outer="bicgstab")
    try:
        S.factor()
        Y = np.random.default_rng(d + k).uniform(-1, 1, (k, A.n))
        g = torch.empty(k, A.n, dtype=torch.float64, device="cuda")
        ddps.ddps_block_solve(S.h, k, dev_vec(Y), g)
        g = host(g)
        C = A.scipy().tocoo()
        own = np.searchsorted(part, C.row, "right") == np.searchsorted(part, C.col, "right")
        D = type(C)((C.data[own], (C.row[own], C.col[own])), shape=C.shape).tocsr()
        # rows of three entries, diagonally dominant: a few roundings per entry
        assert np.max(np.abs((D @ g.T).T - Y)) <= 16 * 2.0 ** -53 * np.max(np.abs(D).sum(axis=1)) * np.max(np.abs(g))
        # the whole method: spikes of the exact factors make the preconditioner exact
        x = np.random.default_rng(d).uniform(-1, 1, A.n)
        z = torch.zeros(A.n, dtype=torch.float64, device="cuda")
        rc, info = ddps.ddps_solve(S.h, dev_vec(A.scipy() @ x), z, 1e-12)
        assert rc == 0 and info.outer_iters <= 2 and relerr(host(z), x) <= 1e-9
    finally:
        S.close()


@pytest.mark.parametrize("offs", [[-17, -16, -1, 0, 1, 16, 17],                       # either side of the near ring
                                  [-60, -50, -40, -30, -9, 0, 9, 30, 40, 50, 60],     # four far, one near
                                  [-5, -4, -3, -2, -1, 0, 1, 2, 3, 4, 5],             # more near than held
                                  [-63, -50, -45, -40, -35, -30, -25, -2, -1, 0, 1, 2, 25, 30, 35, 40, 45, 50, 63]])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_general_rows(offs, dtype):
    from oracle import ddps_oracle as O
    from paper_1008_1700_amd import ddps
    torch = torch_cuda()
    s = system([333, 130, 200], offs, len(offs))
    A = s["A"]
    P = O.Preconditioner(A.n, A.row_ptr, A.col, A.val, s["part_ptr"], 0.0, block_factor="ilu0")
    S = make_solver(s, dtype=dtype, max_rhs=2, retrieval=1, block_factor="ilu0", outer="bicgstab")
    try:
        S.factor()
        Y = np.random.default_rng(1).standard_normal((2, A.n))
        g = torch.empty(2, A.n, dtype=torch.float64, device="cuda")
        ddps.ddps_block_solve(S.h, 2, dev_vec(Y), g)
        g = host(g)
        for j in range(2):
            exp = np.concatenate([O.solve_with(f, Y[j, b.lo:b.hi]) for f, b in zip(P.factors, P.blocks)])
            assert relerr(g[j], exp) <= 1e-12
        m, t, _ = ddps.ddps_reduced_layout(S.h)
        c = torch.empty(m, dtype=torch.int64, device="cuda")
        mask = torch.empty(m, dtype=torch.float64, device="cuda")
        ddps.ddps_reduced_layout(S.h, c, mask)
        on = host(mask) > 0
        assert np.array_equal(host(c)[on], P.c)
        x = np.random.default_rng(2).standard_normal(m) * on
        v = torch.empty(m, dtype=torch.float64, device="cuda")
        ddps.ddps_reduced_matvec(S.h, 1, dev_vec(x), v)
        # FP32 spikes are rounded to 24 bits row by row
        assert relerr(host(v)[on], P.ghat_matvec(x[on])) <= (1e-12 if dtype == "f64" else 64 * 2.0 ** -24)
    finally:
        S.close()
