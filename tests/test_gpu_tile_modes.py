"""Each tile of the grouped products on the launches of whole factorisations,
forced through recorded per-launch tiles: 128 x 128 and 256 x 256 tiles on
problems of every side that is 64, 128 or 192 past a multiple of them, narrow
ones included (which the size rule takes too).  FP64 and FP32 by backward
errors against float64 on the host; the bf16 kernels give the same bits whatever
the tile, so those are compared bit by bit with the 64 x 64 one."""
import numpy as np
import pytest

from tests.gpu_util import host, torch_cuda
from workloads import configs

pytestmark = pytest.mark.gpu

# 64 units of the arithmetic's rounding
TOL = {"f64": 64 * 2.0 ** -52, "f32": 64 * 2.0 ** -23}


def system(b):
    t = -(-b // 64) * 64
    return configs.small_banded(2, [3 * t - 5, 2 * t + 1], b, 100 + b), t


def gemm_launches(S):
    from paper_1008_1700_amd import ddps
    ddps.ddps_timing_enable(S.h, 0, True)
    S.factor()
    r = ddps.ddps_timing_read(S.h, 0)
    ddps.ddps_timing_enable(S.h, 0, False)
    return r["launches"], r["flops"]


def recorded(S, dtype, t, digits, path):
    """The handle's form from a tuner cache with one tile digit for all launches."""
    from paper_1008_1700_amd import ddps
    ddps.ddps_set_execution(S.h, 1, False, 1)
    n, _ = gemm_launches(S)
    line = '{\n  "gfx950/%s/t%d/p2/T3": {"streams": 1, "tile_policy": 3, "factor_ms": 1.000, "modes": "%s"}\n}\n'
    path.write_text(line % (dtype, t, digits * n))
    r = ddps.ddps_autotune(S.h, str(path))
    assert r["tile_policy"] == 3 and path.read_text() == line % (dtype, t, digits * n)
    return gemm_launches(S)[1]


def results(S, A, t):
    """Block solves of two vectors and both blocks' spikes."""
    from paper_1008_1700_amd import ddps
    torch = torch_cuda()
    y = np.random.default_rng(t).uniform(-1, 1, (2, A.n))
    g = torch.empty(2, A.n, dtype=torch.float64, device="cuda")
    ddps.ddps_block_solve(S.h, 2, torch.from_numpy(y).cuda(), g)
    G = []
    for i, n in enumerate((3 * t - 5, 2 * t + 1)):
        G.append(torch.empty(2 * t, n, dtype=torch.float64, device="cuda"))
        ddps.ddps_get_spikes(S.h, i, G[i])
    return y, host(g), [host(x).T for x in G]


@pytest.mark.parametrize("b", [50, 128, 190, 256, 320, 384, 448, 570, 700])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_128_tiles(b, dtype, tmp_path):
    from paper_1008_1700_amd import ddps
    d, t = system(b)
    A, part = d["A"], d["part_ptr"]
    S = ddps.Solver(A, part, dtype=dtype, max_rhs=2)
    try:
        ddps.ddps_set_execution(S.h, 1, False, 1)
        _, small = gemm_launches(S)
        large = recorded(S, dtype, t, "6", tmp_path / "tiles.json")
        assert large > small if t > 64 else large == small   # triangles in whole 128-wide tiles
        y, g, G = results(S, A, t)
        As = A.scipy().toarray()
        for i in range(2):
            lo, hi = int(part[i]), int(part[i + 1])
            Aii, x = As[lo:hi, lo:hi], g[:, lo:hi].T
            na = np.linalg.norm(Aii, np.inf)
            r = np.linalg.norm(Aii @ x - y[:, lo:hi].T) / (na * np.linalg.norm(x))
            R = np.zeros_like(G[i])
            if i == 1:
                R[:, :t] = As[lo:hi, lo - t:lo]
            else:
                R[:, t:] = As[lo:hi, hi:hi + t]
            rg = np.linalg.norm(Aii @ G[i] - R) / (na * np.linalg.norm(G[i]))
            print(f"b {b} {dtype} block {i}: solve {r:.2e}, spikes {rg:.2e}")
            assert r <= TOL[dtype] and rg <= TOL[dtype]
    finally:
        S.close()


@pytest.mark.parametrize("b", [50, 128, 190, 256, 320, 384, 448, 570, 700])
@pytest.mark.parametrize("dtype", ["bf16x3", "bf16"])
def test_bf16_tiles_give_the_same_bits(b, dtype, tmp_path):
    from paper_1008_1700_amd import ddps
    d, t = system(b)
    S = ddps.Solver(d["A"], d["part_ptr"], dtype=dtype, max_rhs=2)
    try:
        ddps.ddps_set_execution(S.h, 1, False, 1)
        _, small = gemm_launches(S)
        _, g, G = results(S, d["A"], t)
        # register-staged 128 x 128 and 256 x 128 (narrowed to what problems
        # fill); direct loads 128 x 128 and 256 x 256 on every launch
        for digit in "1289":
            flops = recorded(S, dtype, t, digit, tmp_path / f"tiles{digit}.json")
            assert flops > small if t >= 128 else flops >= small
            _, g1, G1 = results(S, d["A"], t)
            assert np.array_equal(g, g1) and all(np.array_equal(a, c) for a, c in zip(G, G1)), digit
    finally:
        S.close()


def test_recorded_tiles_are_the_ones_that_ran(tmp_path):
    """A recorded tile wider than a launch's problems is taken where it was
    recorded as run, and narrowed where it was recorded as asked for."""
    from paper_1008_1700_amd import ddps
    d, t = system(190)
    S = ddps.Solver(d["A"], d["part_ptr"], dtype="bf16x3", max_rhs=2)
    try:
        asked, narrow, ran = (recorded(S, "bf16x3", t, q, tmp_path / f"{q}.json") for q in "439")
        assert asked == narrow < ran
        # what the tuner records is what the recorded form runs again
        r = ddps.ddps_autotune(S.h, str(tmp_path / "own.json"), 20.0)
        again = ddps.ddps_autotune(S.h, str(tmp_path / "own.json"))
        assert (r["streams"], r["tile_policy"]) == (again["streams"], again["tile_policy"])
    finally:
        S.close()
