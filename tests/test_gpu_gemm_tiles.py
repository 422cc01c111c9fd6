"""The grouped products at the edges of their tiles: block factors and spikes
of systems whose tile size is one 64-row sub-tile, a whole number of 128- or
256-row tiles, and those plus 64, 128 or 192 rows, on ragged (padded) blocks.
Checked by normwise backward errors of the block solves and the spikes,
against float64 on the host."""
import numpy as np
import pytest

from tests.gpu_util import host, torch_cuda
from workloads import configs

pytestmark = pytest.mark.gpu

# 64 units of the arithmetic's rounding: FP64, FP32, and two bfloat16 terms
# per operand (hi + lo keep 16 bits, the dropped lo * lo term is below them)
TOL = {"f64": 64 * 2.0 ** -52, "f32": 64 * 2.0 ** -23, "bf16x3": 64 * 2.0 ** -17, "bf16": 64 * 2.0 ** -8}


@pytest.fixture(scope="module")
def systems():
    cache = {}

    def get(b):
        if b not in cache:
            t = -(-b // 64) * 64
            # one block padded by a few rows, one whose padding is nearly a tile
            cache[b] = configs.small_banded(2, [3 * t - 5, 2 * t + 1], b, 100 + b)
        return cache[b]
    return get


@pytest.mark.parametrize("b", [50, 128, 190, 256, 320, 384, 448, 512, 570, 700])
@pytest.mark.parametrize("dtype,policy", [("f64", 0), ("f64", 1), ("f32", 0), ("f32", 1), ("bf16x3", 0),
                                          ("bf16x3", 5), ("bf16", 5)])
def test_block_factors_at_tile_edges(systems, b, dtype, policy):
    from paper_1008_1700_amd import ddps
    torch = torch_cuda()
    d = systems(b)
    A, part = d["A"], d["part_ptr"]
    As = A.scipy().toarray()
    S = ddps.Solver(A, part, dtype=dtype, max_rhs=2)
    try:
        if policy:
            ddps.ddps_set_execution(S.h, 1, False, policy)
        S.factor()
        y = np.random.default_rng(b).uniform(-1, 1, (2, A.n))
        yd = torch.from_numpy(y).cuda()
        g = torch.empty_like(yd)
        ddps.ddps_block_solve(S.h, 2, yd, g)
        g = host(g)
        _, t, _ = ddps.ddps_reduced_layout(S.h)
        for i in range(2):
            lo, hi = int(part[i]), int(part[i + 1])
            Aii, x = As[lo:hi, lo:hi], g[:, lo:hi].T
            na = np.linalg.norm(Aii, np.inf)
            r = np.linalg.norm(Aii @ x - y[:, lo:hi].T) / (na * np.linalg.norm(x))
            G = torch.empty(2 * t, hi - lo, dtype=torch.float64, device="cuda")
            ddps.ddps_get_spikes(S.h, i, G)
            G = host(G).T
            R = np.zeros_like(G)
            if i == 1:
                R[:, :t] = As[lo:hi, lo - t:lo]
            else:
                R[:, t:] = As[lo:hi, hi:hi + t]
            rg = np.linalg.norm(Aii @ G - R) / (na * np.linalg.norm(G))
            print(f"b {b} {dtype} policy {policy} block {i}: solve {r:.2e}, spikes {rg:.2e}")
            assert r <= TOL[dtype] and rg <= TOL[dtype]
    finally:
        S.close()
