"""The learned guess's products at the edges of their tiles and chunks: sizes
below one tile, odd leading dimensions, one more and one less than a tile of
32, 64 and 128 and than a chunk of 64, 128 and 256, and layers large enough for
the 128-wide tiles.  Checked against the oracle with the same bf16 roundings, to
the 1e-2 that accumulation order and bf16 ties leave."""
import numpy as np
import pytest

from tests.gpu_util import host, relerr, torch_cuda
from tests.test_gpu_mlp import _net, _unpack

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_in,H,d_out,batch", [(9, 7, 5, 3), (33, 31, 32, 1), (255, 64, 129, 65), (257, 66, 258, 127),
                                                (130, 520, 1030, 600), (512, 100, 2050, 520), (40, 2100, 70, 4200)])
def test_products_at_tile_edges(d_in, H, d_out, batch):
    from oracle import mlp_oracle as M
    from paper_1008_1700_amd import ddps
    torch = torch_cuda()
    net, p = _net(d_in, H, d_out, batch, 7)
    try:
        rng = np.random.default_rng(8)
        X = rng.standard_normal((batch, d_in)).astype(np.float32)
        T = rng.standard_normal((batch, d_out)).astype(np.float32)
        Xd, Td = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
        P = _unpack(p, d_in, H, d_out)
        y, cache = M.forward(P, X.astype(np.float64), bf16=True)
        Yd = torch.empty(batch, d_out, dtype=torch.float32, device="cuda")
        ddps.ddps_mlp_forward(net, batch, Xd, Yd)
        torch.cuda.synchronize()
        assert relerr(host(Yd).astype(np.float64), y) <= 1e-2
        g, loss = ddps.ddps_mlp_gradients(net, batch, Xd, Td)
        assert abs(loss - M.mse(y, T)) <= 1e-3 * M.mse(y, T)
        for i, (a, b) in enumerate(zip(_unpack(g, d_in, H, d_out), M.backward(P, cache, y, T.astype(np.float64), bf16=True))):
            assert relerr(a, b) <= 1e-2, (i, relerr(a, b))
        # one step moves the parameters by the gradients just read, and returns their loss
        assert abs(ddps.ddps_mlp_train_step(net, batch, Xd, Td, 1e-3) - loss) <= 1e-12 * loss
    finally:
        ddps.ddps_mlp_destroy(net)
