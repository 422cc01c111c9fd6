"""The packed-tip product on rows with an infinite entry: the infinity is the
row's result, whatever pieces of the row other lanes do not have."""
import numpy as np
import pytest

from tests.gpu_util import dev_vec, host, torch_cuda
from tests.test_gpu_gemv_forms import system

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,t", [(3, 192), (10, 1024), (9, 1216), (90, 192)])
@pytest.mark.parametrize("k", [1, 2])
def test_infinite_entry_stays_infinite(p, t, k):
    from paper_1008_1700_amd import ddps
    torch = torch_cuda()
    A, part = system(p, t, t)
    # row r = n0 - t of block 0: 0.05 x_r + 1e38 x_n0, and x_r in no other row of it:
    # the first right coupling column's spike overflows FP32 in that row alone
    n0 = int(part[1])
    r = n0 - t
    inside = np.arange(len(A.val)) < A.row_ptr[n0]
    A.val[inside & (A.col == r)] = 0.0
    lo, hi = A.row_ptr[r], A.row_ptr[r + 1]
    A.val[lo:hi] = np.where(A.col[lo:hi] == r, 0.05, np.where(A.col[lo:hi] == n0, 1e38, 0.0))
    S = ddps.Solver(A, part, dtype="f32", max_rhs=k)
    try:
        S.factor()
        m, ts, _ = ddps.ddps_reduced_layout(S.h)
        assert ts == t
        G = torch.empty(2 * t, n0, dtype=torch.float64, device="cuda")
        ddps.ddps_get_spikes(S.h, 0, G)
        G = host(G).T[n0 - t:, t:]
        assert np.isinf(G[0, 0]) and np.isfinite(G[1:]).all() and np.isfinite(G[:, 1:]).all()
        X = np.random.default_rng(p).uniform(0.5, 1, (k, m))
        V = torch.empty(k, m, dtype=torch.float64, device="cuda")
        ddps.ddps_reduced_matvec(S.h, k, dev_vec(X), V)
        V = host(V)
        assert (V[:, 0] == np.sign(G[0, 0]) * np.inf).all()
        assert np.isfinite(V[:, 1:t]).all()
    finally:
        S.close()
