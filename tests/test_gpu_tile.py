"""The 64x64, 128x128 and 256x256 streaming tiles at the edges they have: rows, columns and contractions that end inside a tile, a step
or a group of two steps, a second contraction longer than its first group, split contractions, expert segments shorter than a
tile; and the fused products in each of their forms on 128x128 and 256x256 tiles (fused_cases.py).  Accumulators are exact; bf16
results hold the 2e-2 bar of the other parity tests.  X and dY lie inside buffers of NaN, so that anything fetched past the last
token shows."""
import numpy as np
import pytest
import torch

from oracle import pquant_oracle as po
from paper_2602_22592_amd import binding as pq
from paper_2602_22592_amd import workloads as wl
from fused_cases import CASES
from parity_metrics import relerr
from test_gpu_ffn import check_ffn

pytestmark = pytest.mark.gpu
TOL = 2e-2


@pytest.mark.parametrize("T,K,N", [(1, 32, 8), (63, 96, 72), (64, 128, 64), (65, 160, 64), (128, 256, 128), (129, 288, 136), (300, 4096, 2056),
                                   (700, 2080, 3000),
                                   (4100, 1056, 2080), (4100, 96, 2056)])   # 256x256 tiles over contractions of partial steps
def test_accumulators_exact(T, K, N):
    print(f"accumulators T={T} K={K} N={N}", flush=True)
    rng = np.random.default_rng(40 + T)
    q = rng.integers(-128, 128, (T, K)).astype(np.int8)
    S = np.where(rng.random((N, K)) < 0.5, 1, -1).astype(np.int8)
    acc = pq.onebit_acc(torch.from_numpy(q).cuda(), torch.from_numpy(po.pack_sign(S).view(np.int32)).cuda(), N)
    torch.cuda.synchronize()
    assert np.array_equal(acc.cpu().numpy().astype(np.int64), po.onebit_acc(q, S))


def padded(x):
    """x on the device between rows of NaN."""
    t = torch.full((x.shape[0] + 70, x.shape[1]), float("nan"), dtype=torch.bfloat16, device="cuda")
    t[3:3 + x.shape[0]] = torch.from_numpy(x).cuda().to(torch.bfloat16)
    return t[3:3 + x.shape[0]]


@pytest.mark.parametrize("T,K,N,r,E,k,tau", [(1, 32, 32, 8, 1, 1, None), (31, 64, 96, 0, 1, 1, 0.02), (64, 128, 128, 136, 1, 1, None),
                                             (65, 160, 224, 264, 1, 1, None), (20, 4128, 672, 64, 1, 1, None), (513, 2048, 96, 24, 1, 1, None),
                                             (1100, 96, 64, 40, 1, 1, None), (777, 672, 1312, 72, 1, 1, 0.02), (1025, 1152, 1184, 128, 1, 1, None),
                                             (37, 64, 96, 8, 4, 1, None), (333, 1056, 224, 72, 8, 2, None), (600, 160, 1120, 136, 2, 1, None),
                                             (4101, 1056, 2080, 88, 1, 1, None), (4101, 2080, 1056, 0, 1, 1, 0.02)])   # 256x256 tiles, partial steps
def test_linear_at_tile_edges(T, K, N, r, E, k, tau):
    print(f"linear T={T} K={K} N={N} r={r} E={E} k={k} tau={tau}", flush=True)
    c = wl.linear_case(700 + T, T, K, N, hp_rank=r, n_experts=E, bf16=True, outlier_count=2, outlier_scale=10.0)
    to = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda().to(torch.bfloat16)
    nan = lambda *s, dt=torch.float32: torch.full(s, float("nan"), dtype=dt, device="cuda")
    desc = pq.make_desc(T, K, N, hp_rank=r, n_experts=E, top_k=k, io_dtype=pq.PQ_BF16, alpha=2.0, beta=0.2,
                        ste_mode=pq.PQ_STE_IDENTITY if tau is None else pq.PQ_STE_CLIP, ste_tau=tau or 0.0)
    bufs = pq.LinearBuffers(desc)
    X, dY, W = padded(c["X"]), padded(c["dY"]), to(c["W"])
    hp = {n: to(c[n]) for n in ("A", "B", "Wr") if c.get(n) is not None and (n != "Wr" or E > 1) and r}
    dhp = {"d" + n: nan(*t.shape) for n, t in hp.items()}
    Y, dX, dW, dab = nan(T, N, dt=torch.bfloat16), nan(T, K, dt=torch.bfloat16), nan(N, K), nan(2)
    pq.linear_fwd(desc, X, W, Y, bufs, **hp)
    pq.linear_bwd(desc, dY, X, W, bufs, dX, dW, dab, **hp, **dhp)
    torch.cuda.synchronize()
    kw = dict(A=c.get("A"), B=c.get("B")) if r else {}
    if E > 1:
        kw.update(Wr=c["Wr"])
    f = po.linear_fwd(c["X"], c["W"], 2.0, 0.2, top_k=k, **kw)
    g = po.linear_bwd(c["dY"], c["X"], c["W"], 2.0, 0.2, f, ste_tau=np.inf if tau is None else np.float32(tau), **kw)
    host = lambda t: t.float().cpu().numpy()
    errs = {"Y": relerr(host(Y), f["Y"]), "dX": relerr(host(dX), g["dX"]), "dW": relerr(host(dW), g["dW"])}
    for n, t in dhp.items():
        errs[n] = relerr(host(t), g[n])
    dYd = c["dY"].astype(np.float64)
    errs["dbeta"] = abs(dab[1].item() - g["dbeta"]) / np.sqrt(((dYd * f["Y1_nobeta"]) ** 2).sum())
    if r:
        errs["dalpha"] = abs(dab[0].item() - g["dalpha"]) / np.sqrt(((dYd * f["Yhp"]) ** 2).sum())
    else:
        assert dab[0].item() == 0.0
    print("  errors: " + ", ".join(f"{k}={v:.1e}" for k, v in errs.items()), flush=True)
    assert max(errs.values()) <= TOL, errs


@pytest.mark.parametrize("T,K,N,r,int8", CASES)
def test_fused_products(T, K, N, r, int8):
    """Y and dX of sampled tokens (each depends on its token alone): the first and last, both sides of tile edges, others at random."""
    print(f"fused products T={T} K={K} N={N} r={r} int8={int8}", flush=True)
    c = wl.linear_case(900 + T, T, K, N, hp_rank=r, bf16=True, outlier_count=2, outlier_scale=10.0)
    to = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda().to(torch.bfloat16)
    nan = lambda *s, dt=torch.float32: torch.full(s, float("nan"), dtype=dt, device="cuda")
    alpha, beta = 2.0, 0.2
    desc = pq.make_desc(T, K, N, hp_rank=r, alpha=alpha, beta=beta, hp_kind=pq.PQ_HP_LOWRANK_INT8 if int8 else pq.PQ_HP_LOWRANK_BF16)
    bufs = pq.LinearBuffers(desc)
    X, dY, W, A, B = padded(c["X"]), padded(c["dY"]), to(c["W"]), to(c["A"]), to(c["B"])
    Y, dX = nan(T, N, dt=torch.bfloat16), nan(T, K, dt=torch.bfloat16)
    pq.linear_fwd(desc, X, W, Y, bufs, A=A, B=B)
    pq.linear_bwd(desc, dY, X, W, bufs, dX, nan(N, K), nan(2), A=A, B=B, dA=nan(r, K), dB=nan(N, r))
    torch.cuda.synchronize()
    rng = np.random.default_rng(T)
    edges = [t for t in (0, 1, 63, 64, 127, 128, 255, 256, 257, T // 256 * 256 - 1, T // 256 * 256, T - 2, T - 1) if 0 <= t < T]
    tok = np.unique(np.concatenate([edges, rng.choice(T, min(T, 100), replace=False)])).astype(int)
    x, dy = c["X"][tok], c["dY"][tok]
    if int8:
        f = po.linear_fwd(x, c["W"], 0.0, beta)
        h = po.hp_int8_fwd(None, c["A"], c["B"], bf16=True, q_gamma=(f["q"], f["gamma"]))
        y = f["Y1"].astype(np.float64) + alpha * h["Yhp"].astype(np.float64)
        dx = po.linear_bwd(dy, x, c["W"], 0.0, beta, f)["dX"] + po.hp_int8_bwd(alpha * dy.astype(np.float64), h)["dX"]
    else:
        f = po.linear_fwd(x, c["W"], alpha, beta, A=c["A"], B=c["B"])
        y, dx = f["Y"], po.linear_bwd(dy, x, c["W"], alpha, beta, f, A=c["A"], B=c["B"])["dX"]
    sel = torch.from_numpy(tok).cuda()
    host = lambda t: t[sel].float().cpu().numpy()
    errs = {"Y": relerr(host(Y), y), "dX": relerr(host(dX), dx)}
    print("  errors: " + ", ".join(f"{k}={v:.1e}" for k, v in errs.items()), flush=True)
    assert max(errs.values()) <= TOL, errs
    assert torch.isfinite(Y).all() and torch.isfinite(dX).all()


@pytest.mark.parametrize("T,D,F,E,r,k", [(1300, 1056, 4116, 1, 64, 1),    # paired 256x256 products, partial steps, store limits
                                         (20, 4128, 160, 2, 8, 1),        # paired int8 product with a split contraction
                                         # paired weight gradients with a split contraction.  One branch: with two, dWr at these sizes is
                                         # a sum of 2100 terms of either sign, each good to a bf16 rounding (2**-8 at most), that cancels to
                                         # about sqrt(2100) of them: up to 2**-8 * sqrt(2100) / 6 = 3e-2 of its largest entry, whatever the products do
                                         (2100, 64, 100, 1, 8, 1)])
def test_ffn_paired_products(T, D, F, E, r, k):
    print(f"ffn paired products T={T} d={D} F={F} E={E} r={r} k={k}", flush=True)
    check_ffn(wl.ffn_case(300 + T, T, D, F, E, r), top_k=k)


@pytest.mark.parametrize("T,D,F,r", [(3904, 672, 36, 976), (7084, 448, 36, 776)])   # whole and partial steps
def test_ffn_single_branch_of_large_rank(T, D, F, r):
    """The gradient of [Up; Gate] on split 256x256 tiles, its rows' halves stored to two buffers by the slab sum."""
    print(f"ffn single branch T={T} d={D} F={F} r={r}", flush=True)
    check_ffn(wl.ffn_case(500 + T, T, D, F, 1, r), top_k=1)
