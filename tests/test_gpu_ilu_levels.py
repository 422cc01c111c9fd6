"""Incomplete-factor block solves on levels of many more rows than a workgroup
has threads, whose rows have fewer and more entries than the packed four."""
import numpy as np
import pytest

from tests.gpu_util import dev_vec, host, make_solver, relerr, torch_cuda
from tests.test_gpu_ilu_forms import system

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offs", [[-1500, 0, 1500], [-1504, -1503, -1500, 0, 1500, 1502, 1504],
                                  [-1900, -1800, -1700, -1650, -1600, -1550, 0, 1550, 1600, 1650, 1700, 1800, 1900]])
@pytest.mark.parametrize("k", [1, 2])
def test_wide_levels(offs, k):
    from oracle import ddps_oracle as O
    from paper_1008_1700_amd import ddps
    torch = torch_cuda()
    s = system([6000, 4100], offs, len(offs))
    A = s["A"]
    P = O.Preconditioner(A.n, A.row_ptr, A.col, A.val, s["part_ptr"], 0.0, block_factor="ilu0")
    S = make_solver(s, dtype="f64", max_rhs=k, retrieval=1, block_factor="ilu0", outer="bicgstab")
    try:
        S.factor()
        Y = np.random.default_rng(k).standard_normal((k, A.n))
        g = torch.empty(k, A.n, dtype=torch.float64, device="cuda")
        ddps.ddps_block_solve(S.h, k, dev_vec(Y), g)
        g = host(g)
        for j in range(k):
            exp = np.concatenate([O.solve_with(f, Y[j, b.lo:b.hi]) for f, b in zip(P.factors, P.blocks)])
            assert relerr(g[j], exp) <= 1e-12
    finally:
        S.close()
