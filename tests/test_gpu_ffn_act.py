"""FFN backward whose hidden-state gradient goes through the gated unit inside the product: rows, columns and contractions that end inside a
tile or a step, padded hidden widths, one branch and routed ones; against the oracle, with the bar of the other FFN tests."""
import ctypes

import pytest

from launch_trace import kernels, trace
from paper_2602_22592_amd import binding as pq
from paper_2602_22592_amd import workloads as wl
from test_gpu_ffn import check_ffn

# tokens, d_model, d_ffn, experts, rank
CASES = [(1025, 256, 2052, 1, 8), (1400, 288, 1604, 4, 8), (1030, 512, 3072, 1, 32), (640, 224, 4100, 2, 16)]


@pytest.mark.parametrize("T,D,F,E,r", CASES)
def test_takes_the_product(T, D, F, E, r):
    res = trace([dict(op="ffn", tokens=T, d_model=D, d_ffn=F, n_experts=E, hp_rank=r)])[0]
    assert res["rc"] == 0, res["error"]
    assert not kernels(res, "swiglu_bwd_kernel")
    assert [a[6] for a, _ in kernels(res, "mfma_gemm_kernel") if a[-1] == 1] == [int(D % 64 != 0 or D % 128 != 0)], res["launches"]


@pytest.mark.parametrize("T,D,F", [(64, 256, 512), (300, 2048, 1024)])
def test_small_tiles_leave_it_apart(T, D, F):
    res = trace([dict(op="ffn", tokens=T, d_model=D, d_ffn=F, hp_rank=8)])[0]
    assert res["rc"] == 0, res["error"]
    assert len(kernels(res, "swiglu_bwd_kernel")) == 1


def test_no_memory_for_a_gradient_that_is_not_stored():
    """The workspace holds dU and dG [T][F], nothing of the size of dHd, and little else (8192 tokens: no split weight gradients)."""
    T, D, F = 8192, 2048, 5504
    desc = pq.FFNDesc(T, D, F, 8, 1, 1, pq.PQ_BF16, 2.0, 0.2, pq.PQ_HP_LOWRANK_BF16)
    assert 2 * (2 * T * F) < pq.lib().pq_ffn_workspace_bytes(ctypes.byref(desc)) < 2.5 * (2 * T * F)


@pytest.mark.gpu
@pytest.mark.parametrize("T,D,F,E,r", CASES)
def test_against_the_oracle(T, D, F, E, r):
    print(f"ffn gradient through the unit T={T} d={D} F={F} E={E} r={r}", flush=True)
    check_ffn(wl.ffn_case(900 + T, T, D, F, E, r), top_k=1)
