"""Which kernel a call takes, where the choice depends on more than its sizes: host side only (launch_trace.py)."""
import os

import pytest

from fused_cases import CASES
from launch_trace import MFMA, kernels, trace
from paper_2602_22592_amd import binding as pq


@pytest.fixture(scope="module", autouse=True)
def built():
    if not os.path.exists(pq.LIB_PATH):
        from paper_2602_22592_amd.build import build
        build(verbose=False)


@pytest.mark.parametrize("int8", [False, True])
@pytest.mark.parametrize("batch,experts,layers,shared", [(8, 8, 16, True), (8, 16, 12, True), (8, 16, 16, False), (8, 32, 8, True), (8, 32, 12, False),
                                                         (16, 8, 12, True), (16, 8, 16, False), (16, 16, 8, True), (16, 16, 12, False),
                                                         (16, 32, 4, True), (16, 32, 6, False), (4, 4, 17, False)])
def test_small_batch_decode_shares_a_group_while_all_are_resident(batch, experts, layers, shared, int8):
    """4096 -> 4096: 64 groups a layer; a workgroup's LDS is 32 KB of codes and the hidden states of all experts."""
    r = trace([dict(op="decode", batch=batch, d_in=4096, d_out=4096, hp_rank=64, n_experts=experts, top_k=2, n_layers=layers, int8=int8)])[0]
    assert r["rc"] == 0, r["error"]
    (toks, i8, share), grid = kernels(r, "decode_gemm16_tiled_kernel")[0]
    assert (toks, i8, share) == (8 if batch <= 8 else 16, int(int8), int(shared))
    assert grid == [64 if shared else 16, layers, 1]


@pytest.mark.parametrize("T,K,N,r,hp_kind,paired", [(300, 1024, 4096, 160, 0, True), (2048, 2048, 2048, 64, 0, True), (7680, 256, 4608, 64, 0, True),
                                                    (2048, 2048, 2048, 256, 1, True), (16384, 1024, 4096, 160, 0, False),
                                                    (16384, 4096, 1024, 512, 0, False), (7680, 256, 4608, 672, 1, False)])
def test_factor_gradients_share_a_launch_only_where_small_tiles_serve_both(T, K, N, r, hp_kind, paired):
    """dB and dA on 64x64 tiles in one launch, or each with the tile of its own plan."""
    res = trace([dict(op="linear", tokens=T, d_in=K, d_out=N, hp_rank=r, hp_kind=hp_kind)])[0]
    assert res["rc"] == 0, res["error"]
    pairs = [grid for args, grid in kernels(res, "tile64_gemm_kernel") if args[2:4] == [1, 1] and grid[2] == 2]
    assert len(pairs) == (1 if paired else 0), res["launches"]


@pytest.mark.parametrize("batch,layers,kernel,early", [(16, 32, "decode_prep_kernel", True), (16, 33, "decode_prep_kernel", False),
                                                       (1, 60, "decode_prep_h_kernel", True), (1, 64, "decode_prep_h_kernel", False)])
def test_router_rows_are_requested_early_while_all_workgroups_are_resident(batch, layers, kernel, early):
    """Two workgroups a token; one token: one and, at 8 x 32 hidden rows, sixteen more a layer."""
    r = trace([dict(op="decode", batch=batch, d_in=4096, d_out=2048, hp_rank=32, n_experts=8, top_k=8 if batch == 1 else 2, n_layers=layers)])[0]
    assert r["rc"] == 0, r["error"]
    args, grid = kernels(r, kernel)[0]
    assert args[-1] == int(early) and (grid[0] <= 1024) == early


def fused_route(result, forward, contraction, rank):
    """The form of the 1-bit product with the branch in it (fused_cases.py), from the launches of a linear."""
    bits = 3 if forward else 4
    for name, a, grid in result["launches"]:
        if name == "mfma_gemm_kernel":
            d = dict(zip(MFMA, a))
            if d["b"] != bits:
                continue
            assert not d["whole_tiles"]
            steps = "partial" if d["partial_steps"] else "whole"
            if d["a2"] < 0:
                return 256, "unfused", steps
            n = -(-contraction // (128 if forward else 64))          # contraction steps; the ring has four stages
            return (256, "ring", steps, n % 4) if rank in (64, 128) and n >= 4 else (256, "registers", steps)
        if name in ("tile_gemm_kernel", "tile64_gemm_kernel") and a[-2] == bits:
            assert a[-1] >= 0, "not fused"
            return (128 if name == "tile_gemm_kernel" else 64), grid[1] > 1
    raise AssertionError(result["launches"])


def test_fused_cases_take_the_forms_they_stand_for():
    calls = [dict(op="linear", tokens=T, d_in=K, d_out=N, hp_rank=r, hp_kind=i8) for T, K, N, r, i8 in CASES]
    for (case, (fwd, dx)), res in zip(CASES.items(), trace(calls)):
        T, K, N, r, i8 = case
        assert res["rc"] == 0, (case, res["error"])
        if fwd is not None:
            assert fused_route(res, True, K, r) == fwd, case
        assert fused_route(res, False, N, r) == dx, case


@pytest.mark.parametrize("T,D,F,r", [(3904, 672, 36, 976), (7084, 448, 36, 776)])
def test_single_branch_of_large_rank_takes_split_256_tiles(T, D, F, r):
    res = trace([dict(op="ffn", tokens=T, d_model=D, d_ffn=F, hp_rank=r)])[0]
    (args, grid), = [k for k in kernels(res, "gemm_tn_w4_kernel") if k[0][2]]
    assert args == [int(T % 32 != 0), 0, 1] and grid[1] > 1
    assert [0, 1] in [a for a, _ in kernels(res, "splitk_reduce_kernel")]


@pytest.mark.parametrize("batch,d_in,experts,rank,layers,top_k,grouped", [(8, 2560, 8, 64, 16, 1, True), (4, 2560, 8, 64, 16, 1, False), (8, 2560, 8, 64, 8, 2, False),
                                                                          (8, 4096, 8, 64, 16, 1, True), (4, 4096, 8, 64, 16, 1, False), (16, 4096, 8, 64, 1, 2, False),
                                                                          (2, 1024, 8, 64, 64, 1, True), (8, 1024, 64, 64, 4, 1, False), (8, 3328, 4, 32, 64, 1, True),
                                                                          (16, 4224, 8, 64, 16, 2, False), (16, 1024, 8, 64, 4, 2, True),
                                                                          (16, 1152, 8, 64, 4, 2, False), (8, 1024, 8, 64, 4, 2, False)])
def test_decode_hidden_states_expert_by_expert_where_tokens_share_experts(batch, d_in, experts, rank, layers, top_k, grouped):
    """From 1024 workgroups of eight rows (rows of up to 1024 columns: 8192 workgroups times selections) and d_in / 4096 selections per
    expert on, whatever the width up to 4096."""
    r = trace([dict(op="decode", batch=batch, d_in=d_in, d_out=512, hp_rank=rank, n_experts=experts, top_k=top_k, n_layers=layers)])[0]
    assert r["rc"] == 0, r["error"]
    assert len(kernels(r, "decode_h_grouped_kernel")) == int(grouped) and len(kernels(r, "decode_h_kernel")) == int(not grouped)
