"""Independent products of a backward in one launch, in each form that the launch has on 64x64 and 128x128 tiles beside the all-small one of
test_gpu_ffn_sets.py: weight gradients on either tile with an input gradient (packed signs) or an expert's product on either; rows, columns
and contractions that end inside a tile or a step, split weight gradients; against the oracle, with the bar of the other tests."""
import pytest

from launch_trace import kernels, trace
from paper_2602_22592_amd import workloads as wl
from test_gpu_ffn import check_ffn
from test_gpu_tile import test_linear_at_tile_edges as check_linear

SIGNS, ROWS = 4, 1                                    # operand kinds: packed signs; rows along the contraction

# tokens, d_in, d_out, rank, experts, active -> [(tile of the weight gradients, tile of the other product, its operand, workgroups)], slab sums
LINEAR = {
    (3442, 640, 32, 0, 1, 1): ([(64, 128, SIGNS, 205)], 1),                                                # dW split 7 ways
    (664, 2976, 32, 8, 4, 1): ([(64, 128, SIGNS, 191), (64, 128, ROWS, 432)], 2),
    (378, 2528, 32, 8, 2, 2): ([(64, 64, SIGNS, 280), (64, 128, ROWS, 242)], 1),
    (1531, 1056, 3104, 24, 4, 2): ([(128, 64, SIGNS, 633), (64, 128, ROWS, 516)], 1),
    (1, 896, 2848, 0, 1, 1): ([(128, 64, SIGNS, 245)], 1),
    (3, 1152, 448, 672, 8, 2): ([(64, 64, SIGNS, 144), (128, 64, ROWS, 786)], 0),
    (393, 5216, 800, 0, 1, 1): ([(128, 128, SIGNS, 451)], 1),
    (194, 1440, 4256, 16, 8, 1): ([(128, 128, SIGNS, 624), (64, 64, ROWS, 996)], 3),
    (43, 5888, 1472, 368, 8, 2): ([(128, 128, ROWS, 1806)], 1),
}
# tokens, d_model, d_ffn, experts, rank, active, INT8 experts
FFN = {
    (714, 2176, 36, 8, 32, 1, False): ([(64, 64, ROWS, 134), (64, 128, ROWS, 850)], 3),
    (2, 1056, 60, 8, 384, 1, False): ([(64, 64, ROWS, 71), (128, 64, ROWS, 801)], 0),
    (304, 2368, 68, 8, 128, 2, False): ([(64, 64, ROWS, 254), (128, 128, ROWS, 703)], 2),
    (349, 3008, 128, 8, 160, 2, True): ([(64, 64, ROWS, 151), (128, 128, ROWS, 1296)], 1),
}


def sets(result):
    assert result["rc"] == 0, result["error"]
    return [(*args, grid[0]) for args, grid in kernels(result, "tile_set_kernel")], len(kernels(result, "splitk_reduce_kernel"))


@pytest.mark.parametrize("case", LINEAR)
def test_linear_takes_the_launches(case):
    T, K, N, r, E, k = case
    assert sets(trace([dict(op="linear", tokens=T, d_in=K, d_out=N, hp_rank=r, n_experts=E, top_k=k)])[0]) == LINEAR[case]


@pytest.mark.parametrize("case", FFN)
def test_ffn_takes_the_launches(case):
    T, D, F, E, r, k, i8 = case
    assert sets(trace([dict(op="ffn", tokens=T, d_model=D, d_ffn=F, n_experts=E, hp_rank=r, top_k=k, hp_kind=int(i8))])[0]) == FFN[case]


def test_every_form_has_a_case():
    forms = {s[:3] for launches, _ in [*LINEAR.values(), *FFN.values()] for s in launches}
    assert forms == {(w, x, b) for w in (64, 128) for x in (64, 128) for b in (SIGNS, ROWS)}


@pytest.mark.gpu
@pytest.mark.parametrize("T,K,N,r,E,k", LINEAR)
def test_linear_against_the_oracle(T, K, N, r, E, k):
    check_linear(T, K, N, r, E, k, None)


@pytest.mark.gpu
@pytest.mark.parametrize("T,D,F,E,r,k,i8", FFN)
def test_ffn_against_the_oracle(T, D, F, E, r, k, i8):
    print(f"ffn products together T={T} d={D} F={F} E={E} r={r} k={k} int8={i8}", flush=True)
    check_ffn(wl.ffn_case(1000 + T, T, D, F, E, r), top_k=k, experts="int8" if i8 else "bf16")
