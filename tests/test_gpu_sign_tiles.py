"""Products with packed signs on 128x256 tiles at the edges they have: rows and columns that end inside a tile, contractions that end
inside a step or a packed chunk, a second contraction of less than a step, of more steps than the ring holds and behind a first
one that is shorter than the ring; against the oracle, with the bar of the other parity tests."""
import numpy as np
import pytest
import torch

from launch_trace import MFMA, kernels, trace
from oracle import pquant_oracle as po
from paper_2602_22592_amd import binding as pq
from test_gpu_tile import test_fused_products as check_fused_products

# tokens, d_in, d_out, rank, INT8 branch; both products of each case on 128x256 tiles (INT8: the input gradient)
CASES = [(2561, 2080, 2080, 8, 0), (2049, 1184, 1056, 136, 0), (2050, 1088, 1312, 328, 0), (1537, 2048, 2080, 72, 0), (4097, 1024, 1024, 128, 0),
         (5000, 1024, 288, 200, 0), (2600, 2080, 2080, 160, 1)]


@pytest.mark.parametrize("T,K,N,r,int8", CASES)
def test_cases_take_the_tiles(T, K, N, r, int8):
    res = trace([dict(op="linear", tokens=T, d_in=K, d_out=N, hp_rank=r, hp_kind=int8)])[0]
    assert res["rc"] == 0, res["error"]
    forms = {(d["b"], d["bm"], d["a2"] >= 0) for d in (dict(zip(MFMA, a)) for a, _ in kernels(res, "mfma_gemm_kernel")) if d["b"] in (3, 4)}
    assert (4, 128, True) in forms and (int8 or N < 1024 or (3, 128, True) in forms), res["launches"]


@pytest.mark.gpu
@pytest.mark.parametrize("T,K,N,r,int8", CASES)
def test_fused(T, K, N, r, int8):
    check_fused_products(T, K, N, r, int8)


@pytest.mark.gpu
@pytest.mark.parametrize("T,K,N", [(513, 512, 2056), (640, 1056, 4104), (1500, 416, 1288), (1024, 2080, 1024)])
def test_accumulators_exact(T, K, N):
    print(f"accumulators T={T} K={K} N={N}", flush=True)
    rng = np.random.default_rng(60 + T)
    q = rng.integers(-128, 128, (T, K)).astype(np.int8)
    S = np.where(rng.random((N, K)) < 0.5, 1, -1).astype(np.int8)
    acc = pq.onebit_acc(torch.from_numpy(q).cuda(), torch.from_numpy(po.pack_sign(S).view(np.int32)).cuda(), N)
    torch.cuda.synchronize()
    assert np.array_equal(acc.cpu().numpy().astype(np.int64), po.onebit_acc(q, S))
