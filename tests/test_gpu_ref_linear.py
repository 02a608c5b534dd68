"""fp32 I/O, small calls: H = X A^T in the packing's launch and both branches of the forward in one.  Which calls take the form (and
that calls beyond it do not), and the products against the fp64 oracle at the edges of its 16x16 tiles, of the 64-index steps of the
codes and of the 16-index steps of the rank-r product (bound as for the fp64 products: one rounding to fp32)."""
import pytest

from launch_trace import kernels, trace
from test_gpu_ref import test_fp32_products_at_tile_edges as check_fp32

SHAPES = [(1, 32, 32, 8, None), (17, 96, 64, 8, None), (501, 2080, 512, 72, None), (75, 4096, 160, 24, 0.02), (1024, 288, 256, 16, None)]


@pytest.mark.parametrize("T,K,N,r,tau", SHAPES)
def test_shapes_take_the_form(T, K, N, r, tau):
    res = trace([dict(op="linear", tokens=T, d_in=K, d_out=N, hp_rank=r, io_dtype=0)])[0]
    assert res["rc"] == 0, res["error"]
    assert len(kernels(res, "ref_pack_kernel")) == 1 and len(kernels(res, "ref_linear_kernel")) == 1
    assert not kernels(res, "pack_sign_kernel")


@pytest.mark.parametrize("T,K,N,r", [(1040, 256, 256, 16), (64, 4128, 256, 16), (64, 256, 256, 0)])
def test_other_shapes_do_not(T, K, N, r):
    res = trace([dict(op="linear", tokens=T, d_in=K, d_out=N, hp_rank=r, io_dtype=0)])[0]
    assert res["rc"] == 0, res["error"]
    assert not kernels(res, "ref_linear_kernel")


@pytest.mark.gpu
@pytest.mark.parametrize("T,K,N,r,tau", SHAPES)
def test_against_the_oracle(T, K, N, r, tau):
    check_fp32(T, K, N, r, tau)
