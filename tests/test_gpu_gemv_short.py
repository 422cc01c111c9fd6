"""Sweeps whose column ranges four or eight waves load at once (64 and 128
columns in FP64, 128 and 256 in FP32), one column more, and launches above the
count up to which eight waves take them; products of many right-hand sides on
launches where fewer loads per lane make fewer rounds of workgroups."""
import pytest

from tests import test_gpu_gemv_forms as forms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,t", [(3, 128), (5, 256), (4, 320), (140, 128), (257, 128), (150, 256)])
@pytest.mark.parametrize("dtype,k", [("f64", 1), ("f64", 2), ("f32", 1), ("f32", 2)])
def test_short_ranges(p, t, dtype, k):
    forms.test_products_at_dispatch_edges(p, t, dtype, k)


@pytest.mark.parametrize("p,t,k", [(129, 512, 8), (130, 512, 5), (150, 640, 4)])
def test_rounds_of_many_columns(p, t, k):
    forms.test_products_at_dispatch_edges(p, t, "f64", k)
