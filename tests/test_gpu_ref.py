"""fp32 I/O (reference-precision products, fp64 sums on the matrix pipe): forward and backward of the dense linear against
the fp64 oracle at sizes where the wavefront tiles (64x64, 32x32, 16x16, with and without a shared contraction) and their
last contraction step end inside the matrix.  Bound: fp64 sums rounded once to fp32 differ from the oracle by half a unit
in the last place, 2**-24 of an element, and H and dH are themselves stored once in fp32 (twice that, averaged over the
rank); 1e-6 of the largest element leaves a factor of eight."""
import numpy as np
import pytest
import torch

from oracle import pquant_oracle as po
from paper_2602_22592_amd import binding as pq
from paper_2602_22592_amd import workloads as wl
from parity_metrics import relerr

pytestmark = pytest.mark.gpu
TOL = 1e-6


@pytest.mark.parametrize("T,K,N,r,tau", [(1, 32, 32, 8, None), (15, 64, 96, 24, None), (17, 32, 160, 8, 0.02), (67, 288, 352, 40, None),
                                         (131, 1056, 544, 72, None), (40, 2048, 2048, 8, None), (33, 4096, 2080, 16, 0.02),
                                         (1100, 224, 1312, 136, None), (129, 96, 64, 0, None)])
def test_fp32_products_at_tile_edges(T, K, N, r, tau):
    print(f"fp32 linear T={T} K={K} N={N} r={r} tau={tau}", flush=True)
    c = wl.linear_case(900 + T, T, K, N, hp_rank=r, bf16=False, outlier_count=2, outlier_scale=10.0)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    f32 = lambda *s: torch.full(s, float("nan"), dtype=torch.float32, device="cuda")
    desc = pq.make_desc(T, K, N, hp_rank=r, io_dtype=pq.PQ_F32, alpha=2.0, beta=0.2,
                        ste_mode=pq.PQ_STE_IDENTITY if tau is None else pq.PQ_STE_CLIP, ste_tau=tau or 0.0)
    bufs = pq.LinearBuffers(desc)
    X, W, dY = dev(c["X"]), dev(c["W"]), dev(c["dY"])
    A, B = (dev(c["A"]), dev(c["B"])) if r else (None, None)
    Y, dX, dW, dab = f32(T, N), f32(T, K), f32(N, K), f32(2)
    dA, dB = (f32(r, K), f32(N, r)) if r else (None, None)
    pq.linear_fwd(desc, X, W, Y, bufs, A=A, B=B)
    pq.linear_bwd(desc, dY, X, W, bufs, dX, dW, dab, A=A, B=B, dA=dA, dB=dB)
    torch.cuda.synchronize()
    f = po.linear_fwd(c["X"], c["W"], 2.0, 0.2, A=c.get("A"), B=c.get("B"))
    g = po.linear_bwd(c["dY"], c["X"], c["W"], 2.0, 0.2, f, A=c.get("A"), B=c.get("B"), ste_tau=np.inf if tau is None else tau)
    errs = {"Y": relerr(Y.cpu().numpy(), f["Y"]), "dX": relerr(dX.cpu().numpy(), g["dX"]), "dW": relerr(dW.cpu().numpy(), g["dW"])}
    if r:
        errs["dA"] = relerr(dA.cpu().numpy(), g["dA"]); errs["dB"] = relerr(dB.cpu().numpy(), g["dB"])
    dYd = c["dY"].astype(np.float64)
    errs["dbeta"] = abs(dab[1].item() - g["dbeta"]) / np.sqrt(((dYd * f["Y1_nobeta"]) ** 2).sum())
    if r:
        errs["dalpha"] = abs(dab[0].item() - g["dalpha"]) / np.sqrt(((dYd * f["Yhp"]) ** 2).sum())
    print("  errors: " + ", ".join(f"{k}={v:.1e}" for k, v in errs.items()), flush=True)
    assert max(errs.values()) <= TOL, errs
