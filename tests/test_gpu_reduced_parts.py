"""Direct solve of the reduced system whose products are cut into column ranges
of odd length: tips of 448 over 3 and 1 interfaces (6 and 2 ranges), 320 over 2
(4 ranges), 576 over 4 (8 ranges), each with one and several right-hand sides."""
import numpy as np
import pytest

from tests.gpu_util import dev_vec, host, make_solver, oracle_prec, relerr, torch_cuda
from workloads import configs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,p", [(430, 4), (430, 2), (300, 3), (550, 5)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_parts_of_odd_length(b, p, dtype):
    from paper_1008_1700_amd import ddps
    torch = torch_cuda()
    t = (b + 63) // 64 * 64
    d = configs.small_banded(p, [2 * t + 10 * (i % 2) for i in range(p)], b, 29)
    P = oracle_prec(d)
    n = d["A"].n
    Y = np.random.default_rng(b).standard_normal((5, n))
    want = np.array([P.apply(y, reduced="dense")[0] for y in Y])
    # FP32 tips: the rounding of sums over t columns, 16 of them one after another
    tol = 1e-11 if dtype == "f64" else 16 * t * 2.0 ** -24
    S = make_solver(d, reduced="direct", dtype=dtype, max_rhs=8)
    try:
        S.factor()
        assert ddps.ddps_reduced_layout(S.h)[1] == t
        for k in (1, 2, 5):
            Z = torch.empty(k, n, dtype=torch.float64, device="cuda")
            ddps.ddps_apply_preconditioner(S.h, k, dev_vec(Y[:k]), Z)
            assert relerr(host(Z), want[:k]) <= tol, (k, relerr(host(Z), want[:k]))
    finally:
        S.close()
