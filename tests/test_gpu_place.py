"""Routed linears whose slots are ordered by several workgroups: more experts than a pass of the router counts at once, all of them chosen,
and more router workgroups than the ordering has of its own; against the oracle, with the bar of the other parity tests."""
import pytest

from launch_trace import kernels, trace
from test_gpu_tile import test_linear_at_tile_edges as check_linear

# tokens, d_in, d_out, rank, experts, active; workgroups that order the slots (the packing has one)
CASES = [(2100, 64, 96, 8, 64, 3, 512), (4200, 32, 64, 8, 16, 16, 512), (8300, 32, 32, 8, 8, 2, 512), (300, 32, 64, 8, 5, 5, 76), (3000, 64, 32, 16, 3, 1, 376),
         (9001, 32, 32, 8, 64, 2, 512)]


@pytest.mark.parametrize("T,K,N,r,E,k,groups", CASES)
def test_launch(T, K, N, r, E, k, groups):
    res = trace([dict(op="linear", tokens=T, d_in=K, d_out=N, hp_rank=r, n_experts=E, top_k=k)])[0]
    assert res["rc"] == 0, res["error"]
    (_, grid), = kernels(res, "pack_place_kernel")
    assert grid[0] == groups + -(-K // 512) * (N // 32)


@pytest.mark.gpu
@pytest.mark.parametrize("T,K,N,r,E,k,groups", CASES)
def test_against_the_oracle(T, K, N, r, E, k, groups):
    check_linear(T, K, N, r, E, k, None)
