"""Weight gradients on 192x256 tiles: rows and columns that end inside a tile, tokens that are whole and partial stages, fewer stages
than the ring holds, the clipping mask and the d beta sum in the epilogue, and two products in one launch; against the oracle."""
import pytest

from launch_trace import kernels, trace
from paper_2602_22592_amd import workloads as wl
from test_gpu_ffn import check_ffn
from test_gpu_tile import test_linear_at_tile_edges as check_linear

LINEARS = [(96, 2048, 4256, None), (33, 1312, 6400, None), (257, 2048, 4256, 0.02)]     # tokens, d_in, d_out, clipping
FFNS = [(64, 2048, 2100), (171, 1312, 3300)]                                            # tokens, d_model, d_ffn


@pytest.mark.parametrize("T,K,N,tau", LINEARS)
def test_linears_take_the_tiles(T, K, N, tau):
    res = trace([dict(op="linear", tokens=T, d_in=K, d_out=N)])[0]
    assert res["rc"] == 0, res["error"]
    assert [a for a, _ in kernels(res, "gemm_tn_192_kernel")] == [[int(T % 32 != 0), 0]], res["launches"]


@pytest.mark.parametrize("T,D,F", FFNS)
def test_ffns_take_the_tiles(T, D, F):
    res = trace([dict(op="ffn", tokens=T, d_model=D, d_ffn=F, hp_rank=8)])[0]
    assert res["rc"] == 0, res["error"]
    assert [int(T % 32 != 0), 1] in [a for a, _ in kernels(res, "gemm_tn_192_kernel")], res["launches"]


@pytest.mark.gpu
@pytest.mark.parametrize("T,K,N,tau", LINEARS)
def test_linear(T, K, N, tau):
    check_linear(T, K, N, 0, 1, 1, tau)


@pytest.mark.gpu
@pytest.mark.parametrize("T,D,F", FFNS)
def test_ffn_pair(T, D, F):
    print(f"ffn pair on 192x256 tiles T={T} d={D} F={F}", flush=True)
    check_ffn(wl.ffn_case(800 + T, T, D, F, 1, 8), top_k=1)
