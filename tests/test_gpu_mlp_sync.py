"""A call of the network that returns the loss waits for its stream."""
import ctypes

import pytest

from tests.gpu_util import torch_cuda

pytestmark = pytest.mark.gpu


def test_loss_waits_for_the_gradients():
    from paper_1008_1700_amd import ddps
    torch = torch_cuda()
    st = torch.cuda.Stream()
    # backward products of some milliseconds, all after the loss itself
    net = ddps.ddps_mlp_create(2048, 4096, 2048, 4096, seed=3, stream=st.cuda_stream)
    try:
        with torch.cuda.stream(st):
            X, T = torch.randn(4096, 2048, device="cuda"), torch.randn(4096, 2048, device="cuda")
        st.synchronize()
        for _ in range(3):
            loss = ctypes.c_double()
            rc = ddps.lib().ddps_mlp_gradients(net, 4096, ctypes.c_void_p(X.data_ptr()), ctypes.c_void_p(T.data_ptr()),
                                               None, ctypes.byref(loss))
            done = st.query()
            assert rc == 0 and loss.value > 0 and done
    finally:
        ddps.ddps_mlp_destroy(net)
