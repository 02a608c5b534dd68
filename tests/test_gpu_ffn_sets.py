"""FFN backward on small tiles: dW_down in one launch with the experts' first product, all weight gradients (and what goes back through the
experts) in another; sizes that end inside a tile or a contraction step, padded hidden widths, one branch and routed ones, bf16 and INT8;
against the oracle, with the bar of the other FFN tests."""
import pytest

from launch_trace import kernels, trace
from paper_2602_22592_amd import workloads as wl
from test_gpu_ffn import check_ffn

# tokens, d_model, d_ffn, experts, rank, top_k, INT8 experts, products in the last shared launch
CASES = [(1, 64, 96, 1, 8, 1, False, 4), (65, 96, 164, 1, 96, 1, True, 4), (300, 512, 1020, 4, 24, 2, False, 5), (333, 224, 676, 8, 16, 1, False, 5),
         (1257, 320, 912, 1, 72, 1, False, 4)]


@pytest.mark.parametrize("T,D,F,E,r,k,i8,n", CASES)
def test_share_two_launches(T, D, F, E, r, k, i8, n):
    res = trace([dict(op="ffn", tokens=T, d_model=D, d_ffn=F, n_experts=E, hp_rank=r, top_k=k, hp_kind=int(i8))])[0]
    assert res["rc"] == 0, res["error"]
    tiles = lambda m, n: -(-m // 64) * -(-n // 64)
    Fp, S = -(-F // 32) * 32, T * k
    rows = lambda m: -(-m // 64) + (E if E > 1 else 0)       # row tiles of all experts at most
    sets = [g for _, g in kernels(res, "tile_set_kernel")]
    last = 2 * tiles(Fp, D) + E * (tiles(D, r) + tiles(2 * r, D)) + (rows(S) * -(-D // 64) if n == 5 else 0)
    assert sets[0] == [tiles(D, Fp) + rows(S) * -(-r // 64), 1, 1] and sets[-1] == [last, 1, 1], res["launches"]


@pytest.mark.gpu
@pytest.mark.parametrize("T,D,F,E,r,k,i8", [c[:7] for c in CASES])
def test_against_the_oracle(T, D, F, E, r, k, i8):
    print(f"ffn gradients together T={T} d={D} F={F} E={E} r={r} k={k} int8={i8}", flush=True)
    check_ffn(wl.ffn_case(950 + T, T, D, F, E, r), top_k=k, experts="int8" if i8 else "bf16")
