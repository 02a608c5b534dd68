"""fp32 I/O, calls large enough for the fixed-point form of dX and dW: against the fp64 oracle at sizes where rows, tokens and tiles end
inside their blocks (bound as for the fp64 products: one rounding to fp32), rows whose elements span the whole range of fp32 and
cancel (an fp64 sum's own rounding is the bound), and infinities and NaN, which must come out where plain arithmetic has them."""
import ctypes as C

import numpy as np
import pytest
import torch

from launch_trace import kernels, trace
from paper_2602_22592_amd import binding as pq
from paper_2602_22592_amd import workloads as wl
from test_gpu_ref import test_fp32_products_at_tile_edges as check_fp32

SHAPES = [(1037, 1056, 1120, 40, None), (517, 1568, 1504, 0, 0.02), (2049, 544, 1312, 8, None), (409, 2080, 2080, 16, None),
          (2050, 288, 2400, 16, None)]


@pytest.mark.parametrize("T,K,N,r,tau", SHAPES)
def test_shapes_take_the_form(T, K, N, r, tau):
    res = trace([dict(op="linear", tokens=T, d_in=K, d_out=N, hp_rank=r, io_dtype=0)])[0]
    assert res["rc"] == 0, res["error"]
    assert len(kernels(res, "fixed_rows_kernel")) == 1 and len(kernels(res, "fixed_cols_kernel")) == 1


@pytest.mark.parametrize("T,K,N", [(1037, 1056, 1120), (409, 2080, 2080), (2050, 288, 2400), (2048, 2048, 2048), (517, 1568, 1504)])
def test_both_products_are_one_launch_of_at_most_a_workgroup_per_cu(T, K, N):
    res = trace([dict(op="linear", tokens=T, d_in=K, d_out=N, io_dtype=0)])[0]
    assert res["rc"] == 0, res["error"]
    tiles = (-(-T // 64) + -(-N // 64)) * -(-K // 128)
    assert [grid for _, grid in kernels(res, "fixed_gemm_kernel")] == [[min(tiles, 256), 1, 1]]


# few tokens or narrow layers: the digits' traffic and launches outweigh the products (fp64 backward 144 / 349 / 171 / 168 / 861 us, digits 160 / 503 / 129 /
# 231 / 1086; 2048 tokens 8192 -> 128, where they do not, lies on the same side of the line, which counts every output more than it now costs)
@pytest.mark.parametrize("T,K,N", [(64, 4640, 4096), (64, 8192, 8192), (2048, 8192, 128), (2048, 128, 8192), (65536, 512, 256)])
def test_shapes_that_digits_would_slow_down_do_not(T, K, N):
    res = trace([dict(op="linear", tokens=T, d_in=K, d_out=N, io_dtype=0)])[0]
    assert res["rc"] == 0, res["error"]
    assert not kernels(res, "fixed_rows_kernel")


@pytest.mark.parametrize("T", [2048, 32768])
def test_column_maxima_are_reduced_once(T):
    """... in a launch of ceil(d_out / 64) workgroups whatever the tokens, not by every workgroup of the column pass."""
    res = trace([dict(op="linear", tokens=T, d_in=1024, d_out=1056, io_dtype=0)])[0]
    assert res["rc"] == 0, res["error"]
    assert [grid[0] for _, grid in kernels(res, "fixed_exps_kernel")] == [17]


def _workspace(kind, T, K, N, w_kind=pq.PQ_W_MASTER, r=16):
    return getattr(pq.lib(), kind + "_workspace_bytes")(C.byref(pq.make_desc(T, K, N, hp_rank=r, io_dtype=pq.PQ_F32, w_kind=w_kind)))


@pytest.mark.parametrize("op", ["linear", "linear_norm"])
def test_workspace_without_digits_is_accepted(op):
    """The digits are a region behind everything else: forward and backward take a workspace that ends in front of it (the size of the
    packed descriptor, which cannot have a backward), and the backward then runs fp64 products."""
    T, K, N, r = 1037, 1056, 1120, 16
    small, full = (_workspace("pq_" + op, T, K, N, w) for w in (pq.PQ_W_PACKED, pq.PQ_W_MASTER))
    assert 0 < full - small - (14 * T * N + 28 * N * K) < 4 << 20
    calls = [dict(op=op, tokens=T, d_in=K, d_out=N, hp_rank=r, io_dtype=0, workspace_bytes=n) for n in (full, full - 1, small, small - 1)]
    res = trace(calls)
    assert [x["rc"] for x in res] == [0, 0, 0, -4], [x["error"] for x in res]      # PQ_ERR_WORKSPACE
    assert [len(kernels(x, "fixed_rows_kernel")) for x in res] == [1, 0, 0, 0]
    assert not res[3]["launches"]


@pytest.mark.parametrize("T,K,N", [(65536, 8192, 8192), (8192, 4096, 11008), (4096, 2048, 2040)])
def test_workspace_of_digits_is_bounded(T, K, N):
    """Beyond 2 GiB, and for d_out that no backward takes, there are no digits."""
    assert _workspace("pq_linear", T, K, N) == _workspace("pq_linear", T, K, N, pq.PQ_W_PACKED) < 1 << 30


@pytest.mark.gpu
def test_workspace_without_digits_gives_the_same_gradients():
    T, K, N, r = 517, 1568, 1504, 24
    c = wl.linear_case(9, T, K, N, hp_rank=r, bf16=False, outlier_count=2, outlier_scale=10.0)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    t = {k: dev(c[k]) for k in ("X", "W", "dY", "A", "B")}
    desc = pq.make_desc(T, K, N, hp_rank=r, io_dtype=pq.PQ_F32)
    out = []
    for ws in (None, torch.empty(_workspace("pq_linear", T, K, N, pq.PQ_W_PACKED, r), dtype=torch.uint8, device="cuda")):
        bufs = pq.LinearBuffers(desc, ws=ws)
        Y, dX, dW, dA, dB, dab = (torch.empty(s, device="cuda") for s in ((T, N), (T, K), (N, K), (r, K), (N, r), (2,)))
        pq.linear_fwd(desc, t["X"], t["W"], Y, bufs, A=t["A"], B=t["B"])
        pq.linear_bwd(desc, t["dY"], t["X"], t["W"], bufs, dX, dW, dab, A=t["A"], B=t["B"], dA=dA, dB=dB)
        torch.cuda.synchronize()
        out.append([x.cpu().numpy().astype(np.float64) for x in (Y, dX, dW, dA, dB, dab)])
    for a, b in zip(*out):                            # sums that agree to fp64, each rounded to fp32
        assert np.abs(a - b).max() <= 2.0**-23 * np.abs(a).max()


@pytest.mark.gpu
@pytest.mark.parametrize("T,K,N,r,tau", SHAPES)
def test_against_the_oracle(T, K, N, r, tau):
    check_fp32(T, K, N, r, tau)


def run(dY, T, K, N, X=None):
    c = wl.linear_case(7, T, K, N, hp_rank=0, bf16=False, outlier_count=2, outlier_scale=10.0)
    if X is not None:
        c["X"] = X
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    desc = pq.make_desc(T, K, N, hp_rank=0, io_dtype=pq.PQ_F32, alpha=2.0, beta=0.5)
    bufs = pq.LinearBuffers(desc)
    X, W, g = dev(c["X"]), dev(c["W"]), dev(dY)
    Y, dX, dW, dab = (torch.empty(s, dtype=torch.float32, device="cuda") for s in ((T, N), (T, K), (N, K), (2,)))
    pq.linear_fwd(desc, X, W, Y, bufs)
    pq.linear_bwd(desc, g, X, W, bufs, dX, dW, dab)
    torch.cuda.synchronize()
    w, x = c["W"].astype(np.float64), c["X"]
    mu, lam = np.float32(w.mean()), np.float32(np.abs(w).mean())
    S = np.where(c["W"] >= mu, 1.0, -1.0)
    gam = np.float32(128.0) / np.maximum(np.abs(x).max(1), np.float32(1e-5)).astype(np.float32)
    q = np.clip(np.rint(x * gam[:, None]), -128, 127).astype(np.float64)
    return dX.cpu().numpy(), dW.cpu().numpy(), dab.cpu().numpy(), S, q, gam.astype(np.float64), np.float64(np.float32(0.5) * lam)


@pytest.mark.gpu
def test_wide_ranges_and_cancellation():
    T, K, N = 1030, 1056, 1120
    rng = np.random.default_rng(5)
    dY = (rng.standard_normal((T, N)) * np.exp(rng.uniform(-40, 40, (T, N)))).astype(np.float32)
    dY[:, 1::2] -= dY[:, 0::2]                        # pairs that nearly cancel where their signs agree
    dX, dW, _, S, q, gam, bl = run(dY, T, K, N)
    rows, cols = rng.choice(T, 24, replace=False), rng.choice(N, 24, replace=False)
    L = np.longdouble
    ref = (dY[rows].astype(L) @ S.astype(L)) * bl
    # one rounding to fp32, and what N additions in fp64 may lose against the row's largest element
    bound = 2.0**-24 * np.abs(ref) + bl * N * 2.0**-53 * np.abs(dY[rows]).max(1, keepdims=True)
    assert (np.abs(dX[rows] - ref) <= bound).all()
    E = dY[:, cols].astype(L) / gam[:, None]
    ref = (E.T @ q.astype(L)) * 0.5
    # ... and what T additions in fp64, or the digits of sums that may be taken from them, lose against the elements that enter
    assert (np.abs(dW[cols] - ref) <= 2.0**-24 * np.abs(ref) + 2.0**-28 * 0.5 * (np.abs(E).T @ np.abs(q).astype(L))).all()


@pytest.mark.gpu
@pytest.mark.parametrize("big", [1e3, 1e6, 1e9, 1e10, 1e12, 1e16, 1e30])
def test_tokens_that_dominate_but_have_zero_codes(big):
    """The largest elements of dY's columns belong to tokens whose codes are zero in a third of the channels: they set the unit of the digits
    and take no part in those sums, which must keep the precision of sums without them."""
    T, K, N = 1030, 1056, 1120
    rng = np.random.default_rng(8)
    dY = rng.standard_normal((T, N)).astype(np.float32)
    dY[[77, 500]] *= np.float32(big)
    X = wl.linear_case(7, T, K, N, hp_rank=0, bf16=False, outlier_count=2, outlier_scale=10.0)["X"]
    X[77, ::3] = 0.0
    X[500, ::3] = 0.0
    X[:, 5] = 0.0                                     # a channel of zeros
    X[:, 7] = np.where(rng.random(T) < 0.9, np.float32(0), X[:, 7])
    dY[:, 3] = 0.0                                    # a column of zeros
    dY[200:800, 11] = 0.0                             # masked tokens
    _, dW, _, _, q, gam, _ = run(dY, T, K, N, X)
    L = np.longdouble
    cols = np.arange(48)
    E = dY[:, cols].astype(L) / gam[:, None].astype(L)
    ref = (E.T @ q.astype(L)) * L(0.5)
    assert (np.abs(dW[cols] - ref) <= 2.0**-24 * np.abs(ref) + 2.0**-28 * 0.5 * (np.abs(E).T @ np.abs(q).astype(L))).all()
    out = np.zeros(K, bool)
    out[::3] = True
    err = np.linalg.norm((dW[cols][:, out] - ref[:, out]).astype(np.float64)) / np.linalg.norm(ref[:, out].astype(np.float64))
    print(f"  dominating tokens x {big:g}: relative error of the sums without them {err:.2e}", flush=True)
    assert err <= 2.0**-24                            # one rounding to fp32 is 2.5e-8 in the 2-norm


@pytest.mark.gpu
def test_infinities_and_nan():
    T, K, N = 1030, 1056, 1120
    rng = np.random.default_rng(6)
    dY = rng.standard_normal((T, N)).astype(np.float32)
    dY[3, 17] = np.inf
    dY[700, [5, 900]] = np.inf, -np.inf
    dY[1029, 1119] = np.nan
    dX, dW, dab, S, q, gam, bl = run(dY, T, K, N)
    with np.errstate(invalid="ignore"):
        for got, ref in ((dX, (dY.astype(np.float64) @ S) * bl), (dW, 0.5 * (dY.astype(np.float64).T @ (q / gam[:, None])))):
            assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
            assert np.array_equal(np.sign(got[np.isinf(ref)]), np.sign(ref[np.isinf(ref)]))
            ok = np.isfinite(ref)
            assert np.abs(got[ok] - ref[ok]).max() <= 1e-6 * np.abs(ref[ok]).max()
    assert np.isnan(dab[1])


@pytest.mark.gpu
def test_infinities_and_nan_cost_what_fp64_products_cost():
    """A tile with rows that have no digits is formed as an fp64 product.  One infinite activation marks every row of dW, i.e. the digits
    and the whole fp64 product: a training loop that skips overflowing steps meets it.  Element by element it took 23 times a finite
    backward; now 2.9 times (bar: 5)."""
    T = K = N = 2048
    g = torch.Generator(device="cuda").manual_seed(3)
    X, W, dY = (torch.randn(s, generator=g, device="cuda") for s in ((T, K), (N, K), (T, N)))
    desc = pq.make_desc(T, K, N, io_dtype=pq.PQ_F32)
    bufs = pq.LinearBuffers(desc)
    Y, dX, dW, dab = (torch.empty(s, device="cuda") for s in ((T, N), (T, K), (N, K), (2,)))

    def ms():
        times = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            pq.linear_fwd(desc, X, W, Y, bufs)
            a.record()
            pq.linear_bwd(desc, dY, X, W, bufs, dX, dW, dab)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        return sorted(times)[2]

    finite = ms()
    dY[100, 200] = float("nan")
    marked_row = ms()
    dY[100, 200] = 0.0
    X[100, 200] = float("inf")
    all_rows = ms()
    print(f"  backward: finite {finite:.3f} ms, one NaN in dY {marked_row:.3f}, one infinity in X {all_rows:.3f}", flush=True)
    assert marked_row <= 5 * finite and all_rows <= 5 * finite
