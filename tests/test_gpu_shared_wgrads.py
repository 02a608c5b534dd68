"""The products behind dH in one launch: dW on 64x64 tiles, unsplit, with the branch's dB and dA and, where it takes such tiles too, dX;
sizes that end inside a tile or a contraction step, up to and beyond one workgroup per CU, with and without the clipping mask, bf16 and
INT8 branch; against the oracle, with the bar of the other linear tests."""
import pytest

from launch_trace import kernels, trace
from test_gpu_parity import test_linear_with_int8_high_precision_branch as check_int8_branch
from test_gpu_tile import test_linear_at_tile_edges as check_linear

# tokens, d_in, d_out, rank, clipping threshold, (ring of the shared launch, dX too), splits of dB and dA
CASES = [(1, 64, 96, 8, None, (4, 1), 1), (127, 224, 160, 72, 0.02, (4, 1), 1), (130, 768, 800, 40, None, (4, 1), 1), (600, 1056, 1088, 264, 0.02, (2, 1), 1),
         (1000, 2048, 1024, 64, None, (2, 1), 1), (1779, 2208, 800, 64, 0.02, (2, 0), 4)]
INT8_CASES = [(65, 192, 96, 32, (4, 1), 1), (333, 672, 1312, 96, (2, 1), 1)]


@pytest.mark.parametrize("T,K,N,r,i8,form,sp", [(*c[:4], 0, *c[5:]) for c in CASES] + [(*c[:4], 1, *c[4:]) for c in INT8_CASES])
def test_share_a_launch(T, K, N, r, i8, form, sp):
    res = trace([dict(op="linear", tokens=T, d_in=K, d_out=N, hp_rank=r, hp_kind=i8)])[0]
    assert res["rc"] == 0, res["error"]
    tiles = lambda m, n: -(-m // 64) * -(-n // 64)
    blocks = tiles(N, K) + sp * (tiles(N, r) + tiles(r, K)) + (tiles(T, K) if form[1] else 0)
    assert kernels(res, "tile64_grads_kernel") == [(list(form), [blocks, 1, 1])], res["launches"]


@pytest.mark.parametrize("T,K,N,r", [(300, 1024, 4096, 160), (8192, 256, 256, 16), (3032, 1504, 480, 16)])   # dW on 128x128 tiles; split; the pair split
def test_each_in_its_own_where_dw_takes_other_tiles(T, K, N, r):
    res = trace([dict(op="linear", tokens=T, d_in=K, d_out=N, hp_rank=r)])[0]
    assert res["rc"] == 0, res["error"]
    assert not kernels(res, "tile64_grads_kernel")


@pytest.mark.gpu
@pytest.mark.parametrize("T,K,N,r,tau", [c[:5] for c in CASES])
def test_against_the_oracle(T, K, N, r, tau):
    check_linear(T, K, N, r, 1, 1, tau)


@pytest.mark.gpu
@pytest.mark.parametrize("T,K,N,r", [c[:4] for c in INT8_CASES])
def test_int8_branch_against_the_oracle(T, K, N, r):
    check_int8_branch(T, K, N, r)
