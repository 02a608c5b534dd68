"""The workloads this library is timed on, each one pass through its public entry points.

Shapes are those of the paper's 1.3B model (d = 2048, hidden width 5504 or 5076, branches of width 32 to 384, sequences
of 2048 tokens), of the packed decode product (4096 -> 11008) and of the small parity case; `draw` gives sizes around
them, odd ones included.  Inputs follow the paper's statistics: latent weights N(0, 0.02), activations N(0, 1) with one
input channel in a hundred twenty times larger, output gradients N(0, 1).
"""
import math

import torch

from paper_2602_22592_amd import binding as pq
from paper_2602_22592_amd import workloads as wl
from paper_2602_22592_amd.stack import Stack

ALPHA, BETA = 2.0, 0.2          # the paper's initial feature scales


def listed():
    return [
        # the smallest training call: 64 tokens through a 256 x 256 linear in full precision, where launches count
        dict(name="linear_small_fp32", kind="linear", tokens=64, d_in=256, d_out=256, rank=16, experts=1, top_k=1,
             dtype="f32", hp="bf16"),
        # a training step of a 1.3B-shaped projection with its dense high-precision branch (four sequences)
        dict(name="linear_projection", kind="linear", tokens=8192, d_in=2048, d_out=2048, rank=128, experts=1, top_k=1,
             dtype="bf16", hp="bf16"),
        # a ragged batch through a linear with routed experts: no size is a whole number of tiles
        dict(name="linear_routed_ragged", kind="linear", tokens=1531, d_in=1056, d_out=3104, rank=24, experts=4, top_k=2,
             dtype="bf16", hp="bf16"),
        # full-precision training of one sequence (fp32 activations, weights and gradients)
        dict(name="linear_fp32", kind="linear", tokens=2048, d_in=2048, d_out=2048, rank=128, experts=1, top_k=1,
             dtype="f32", hp="bf16"),
        # normalisation, 1-bit linear and INT8 branch, two sequences
        dict(name="linear_norm_int8", kind="linear_norm", tokens=4096, d_in=2048, d_out=2048, rank=128, experts=1,
             top_k=1, dtype="bf16", hp="int8"),
        # prefill of a 512-token prompt on packed weights, nothing kept for a backward
        dict(name="linear_prefill", kind="prefill", tokens=512, d_in=4096, d_out=11008, rank=64),
        # a training step of the 1.3B-shaped feed-forward block with eight routed experts
        dict(name="ffn_routed", kind="ffn", tokens=8192, d_model=2048, d_ffn=5504, rank=32, experts=8, top_k=1, hp="bf16"),
        # the paper's default block: one INT8 branch of width 384 beside 5076 one-bit hidden units, one sequence
        dict(name="ffn_single_int8", kind="ffn", tokens=2048, d_model=2048, d_ffn=5076, rank=384, experts=1, top_k=1,
             hp="int8"),
        # token-by-token generation: one token through one packed linear with two of eight experts
        dict(name="decode_linear_one", kind="decode_linear", batch=1, layers=1, d_in=4096, d_out=11008, rank=64, experts=8,
             top_k=2, hp="bf16"),
        # eight sequences decoded together, INT8 experts, every layer of a model in one call
        dict(name="decode_linear_batch", kind="decode_linear", batch=8, layers=64, d_in=4096, d_out=11008, rank=64,
             experts=8, top_k=2, hp="int8"),
        # token-by-token generation through the packed feed-forward blocks of a 32-layer model
        dict(name="decode_ffn", kind="decode_ffn", batch=1, layers=32, d_model=4096, d_ffn=11008, rank=64, experts=8,
             top_k=2),
        # the linears of a whole training step at 16384 tokens, two layers deep (the largest)
        dict(name="stack", kind="stack", tokens=16384, layers=2, d_model=2048, d_ffn=5504, rank=32, experts=8, top_k=1),
    ]


# ---------------------------------------------------------------------------------------------------------------------
# more cases of the same ranges
# ---------------------------------------------------------------------------------------------------------------------
def _spread(rng, lo, hi, step=1):
    """A multiple of `step` in [lo, hi], even over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(max(int(round(v / step)) * step, lo), hi)


def draw(rng):
    """Training calls of 64 to 16384 tokens, prefill of 16 to 4096, decoding of 1 to 16 sequences through 1 to 64 layers."""
    limit = work(listed()[-1])["flops"] / 3      # drawn shapes are less regular than the largest listed one
    while True:
        kind = rng.choice(["linear", "linear", "linear", "linear_norm", "prefill", "ffn", "ffn", "decode_linear",
                           "decode_linear", "decode_ffn", "decode_ffn", "stack"])
        if kind in ("linear", "linear_norm"):
            form = rng.choice(["bf16", "bf16", "none", "routed", "int8", "f32"])
            f32 = form == "f32"
            c = dict(kind=kind, tokens=_spread(rng, 64, 2048 if f32 else 16384), d_in=_spread(rng, 256, 2048 if f32 else 4096, 32),
                     d_out=_spread(rng, 256, 2048 if f32 else 8192, 32), rank=_spread(rng, 8, 256, 8), experts=1, top_k=1,
                     dtype="f32" if f32 else "bf16", hp="int8" if form == "int8" else "bf16")
            if form == "none":
                c["rank"] = 0
            elif form == "int8":
                c["rank"] = _spread(rng, 32, 256, 32)
            elif form == "routed":
                c["rank"] = _spread(rng, 8, 64, 8)
                c["experts"] = rng.choice([2, 4, 8])
                c["top_k"] = rng.choice([1, 2])
        elif kind == "prefill":
            c = dict(kind=kind, tokens=_spread(rng, 16, 4096), d_in=_spread(rng, 512, 8192, 32), d_out=_spread(rng, 512, 11008, 32),
                     rank=rng.choice([0, 32, 64, 128]))
        elif kind == "ffn":
            c = dict(kind=kind, tokens=_spread(rng, 64, 8192), d_model=_spread(rng, 256, 4096, 32), d_ffn=_spread(rng, 512, 8192, 4),
                     rank=32, experts=1, top_k=1, hp=rng.choice(["bf16", "bf16", "int8"]))
            if rng.random() < 0.5:
                c["rank"] = rng.choice([128, 256, 384])
            else:
                c["experts"] = rng.choice([2, 4, 8])
                c["top_k"] = rng.choice([1, 1, 2])
        elif kind == "decode_linear":
            c = dict(kind=kind, batch=rng.choice([1, 1, 2, 4, 8, 13, 16]), layers=_spread(rng, 1, 64), d_in=_spread(rng, 1024, 8192, 128),
                     d_out=_spread(rng, 1024, 11008, 4), rank=64, experts=rng.choice([4, 8]), top_k=rng.choice([1, 2]),
                     hp=rng.choice(["bf16", "int8"]))
        elif kind == "decode_ffn":
            c = dict(kind=kind, batch=rng.choice([1, 1, 3, 5, 8, 16]), layers=_spread(rng, 1, 32), d_model=_spread(rng, 1024, 4096, 128),
                     d_ffn=_spread(rng, 2048, 11008, 128), rank=rng.choice([32, 64]), experts=rng.choice([4, 8]),
                     top_k=rng.choice([1, 2]))
        else:
            c = dict(kind=kind, tokens=_spread(rng, 256, 8192), layers=rng.choice([1, 2]), d_model=_spread(rng, 256, 2048, 32),
                     d_ffn=_spread(rng, 512, 5504, 32), rank=rng.choice([16, 32]), experts=rng.choice([2, 4, 8]), top_k=1)
        scale = 8.0 if c.get("dtype") == "f32" else 1.0     # fp64 products run at a fraction of the 16-bit rate
        if work(c)["flops"] * scale <= limit:
            return c


# ---------------------------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------------------------
def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(g, shape, std=1.0, dtype=torch.bfloat16):
    t = torch.randn(shape, generator=g, device="cuda")
    return t.mul_(std).to(dtype)


def _activations(g, tokens, d, dtype=torch.bfloat16):
    """N(0, 1) with one channel in a hundred twenty times larger (the outlier channels of trained models)."""
    t = torch.randn((tokens, d), generator=g, device="cuda")
    ch = torch.randperm(d, generator=g, device="cuda")[: max(1, d // 100)]
    t[:, ch] *= 20.0
    return t.to(dtype)


def _empty(*shape, dtype=torch.float32):
    return torch.empty(shape, dtype=dtype, device="cuda")


def _tiled_bits(g, layers, n, k):
    """Packed sign rows in the row-interleaved order of the decode calls, one set per layer."""
    rows = torch.randint(-2**31, 2**31 - 1, (layers, n, k // 32), dtype=torch.int32, device="cuda", generator=g)
    return torch.stack([pq.pack_retile64(rows[l], k) for l in range(layers)]).contiguous()


def _scales(shape, value):
    """fp16 bits of one stored scale per packed matrix."""
    return torch.full(shape, value, dtype=torch.float16, device="cuda").view(torch.int16)


_W_LAMBDA = 0.02 * math.sqrt(2.0 / math.pi)      # mean |W| of N(0, 0.02)


def _prepare_linear(c, g):
    T, K, N, r, E = c["tokens"], c["d_in"], c["d_out"], c["rank"], c["experts"]
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    io = pq.PQ_F32 if c["dtype"] == "f32" else pq.PQ_BF16
    kind = pq.PQ_HP_LOWRANK_INT8 if c["hp"] == "int8" else pq.PQ_HP_LOWRANK_BF16
    desc = pq.make_desc(T, K, N, hp_rank=r, n_experts=E, top_k=c["top_k"], io_dtype=io, alpha=ALPHA, beta=BETA, hp_kind=kind)
    lead = (E,) if E > 1 else ()
    s = dict(c=c, desc=desc, X=_activations(g, T, K, dt), W=_normal(g, (N, K), 0.02, dt), dY=_normal(g, (T, N), 1.0, dt),
             Y=_empty(T, N, dtype=dt), dX=_empty(T, K, dtype=dt), dW=_empty(N, K), dab=_empty(2))
    s["hp"] = dict(A=None, B=None, Wr=None)
    s["dhp"] = dict(dA=None, dB=None, dWr=None)
    if r:
        s["hp"].update(A=_normal(g, lead + (r, K), 0.02, dt), B=_normal(g, lead + (N, r), 0.02, dt))
        s["dhp"].update(dA=_empty(*lead, r, K), dB=_empty(*lead, N, r))
        if E > 1:
            s["hp"]["Wr"] = _normal(g, (E, K), 0.02, dt)
            s["dhp"]["dWr"] = _empty(E, K)
    if c["kind"] == "linear_norm":
        s.update(gain=(1.0 + 0.1 * torch.randn((K,), generator=g, device="cuda")).to(dt), dgain=_empty(K),
                 bufs=pq.LinearNormBuffers(desc))
    else:
        s["bufs"] = pq.LinearBuffers(desc)
    return s


def _prepare_prefill(c, g):
    T, K, N, r = c["tokens"], c["d_in"], c["d_out"], c["rank"]
    desc = pq.make_desc(T, K, N, hp_rank=r, w_kind=pq.PQ_W_PACKED, alpha=ALPHA, beta=BETA)
    bits = torch.randint(-2**31, 2**31 - 1, (N, K // 32), dtype=torch.int32, device="cuda", generator=g)
    return dict(c=c, desc=desc, bufs=pq.LinearBuffers(desc), X=_activations(g, T, K), P=bits,
                mu_lambda=torch.tensor([0.0, _W_LAMBDA], dtype=torch.float32, device="cuda"),
                A=_normal(g, (r, K), 0.02) if r else None, B=_normal(g, (N, r), 0.02) if r else None,
                Y=_empty(T, N, dtype=torch.bfloat16))


def _ffn_weights(g, D, F, E, r):
    return dict(W_up=_normal(g, (F, D), 0.02), W_gate=_normal(g, (F, D), 0.02), W_down=_normal(g, (D, F), 0.02),
                Up=_normal(g, (E, r, D), 0.02), Gate=_normal(g, (E, r, D), 0.02), Down=_normal(g, (E, D, r), 0.02),
                Wr=_normal(g, (E, D), 0.02))


def _prepare_ffn(c, g):
    T, D, F, E, r = c["tokens"], c["d_model"], c["d_ffn"], c["experts"], c["rank"]
    kind = pq.PQ_HP_LOWRANK_INT8 if c["hp"] == "int8" else pq.PQ_HP_LOWRANK_BF16
    desc = pq.FFNDesc(T, D, F, r, E, c["top_k"], pq.PQ_BF16, ALPHA, BETA, kind)
    w = _ffn_weights(g, D, F, E, r)
    return dict(c=c, desc=desc, bufs=pq.FFNBuffers(desc), X=_activations(g, T, D), dY=_normal(g, (T, D)), w=w,
                Y=_empty(T, D, dtype=torch.bfloat16), dX=_empty(T, D, dtype=torch.bfloat16),
                g={n: _empty(*t.shape) for n, t in w.items()}, dab=_empty(2))


def _prepare_decode_linear(c, g):
    L, B, K, N, E, r = c["layers"], c["batch"], c["d_in"], c["d_out"], c["experts"], c["rank"]
    desc = pq.DecodeDesc(B, K, N, r, E, c["top_k"], L, pq.PQ_PACKED_TILED64, ALPHA)
    s = dict(c=c, desc=desc, ws=pq.decode_workspace(desc), P=_tiled_bits(g, L, N, K), scale=_scales((L,), BETA * _W_LAMBDA),
             X=_activations(g, L * B, K).view(L, B, K), A=_normal(g, (L, E, r, K), 0.02), B=_normal(g, (L, E, N, r), 0.02),
             Wr=_normal(g, (L, E, K), 0.02), Y=_empty(L, B, N, dtype=torch.bfloat16))
    if c["hp"] == "int8":       # quantised once, when the weights are loaded
        s["Aq"], s["gA"] = pq.quant_rows(s.pop("A"))
        s["Bq"], s["gB"] = pq.quant_rows(s.pop("B"))
    return s


def _prepare_decode_ffn(c, g):
    L, B, D, F, E, r = c["layers"], c["batch"], c["d_model"], c["d_ffn"], c["experts"], c["rank"]
    desc = pq.DecodeFFNDesc(D, F, r, E, c["top_k"], L, ALPHA, B)
    return dict(c=c, desc=desc, ws=pq.decode_ffn_workspace(desc), X=_activations(g, L * B, D).view(L, B, D),
                Pug=_tiled_bits(g, 2 * L, F, D), Pd=_tiled_bits(g, L, D, F), sug=_scales((L, 2), _W_LAMBDA),
                sd=_scales((L,), BETA * _W_LAMBDA), UpGate=_normal(g, (L, E, 2 * r, D), 0.02),
                Down=_normal(g, (L, E, D, r), 0.02), Wr=_normal(g, (L, E, D), 0.02), Y=_empty(L, B, D, dtype=torch.bfloat16))


def _prepare_stack(c, g):
    T, L, D, F, E, r = c["tokens"], c["layers"], c["d_model"], c["d_ffn"], c["experts"], c["rank"]
    ws = []
    for _ in range(L):
        w = {n: _normal(g, (D, D), 0.02) for n in ("Wq", "Wk", "Wv", "Wo")}
        w.update(_ffn_weights(g, D, F, E, r))
        ws.append(w)
    st = Stack(L, T, D, F, E, r, c["top_k"], [wl.TRAINED_ALPHA[l % 16] for l in range(L)], [wl.TRAINED_BETA[l % 16] for l in range(L)])
    return dict(c=c, st=st, w=ws, h0=_normal(g, (T, D)), dY=_normal(g, (T, D)),
                g=[dict({n: _empty(*t.shape) for n, t in w.items()}, dab=_empty(2)) for w in ws])


_PREPARE = dict(linear=_prepare_linear, linear_norm=_prepare_linear, prefill=_prepare_prefill, ffn=_prepare_ffn,
                decode_linear=_prepare_decode_linear, decode_ffn=_prepare_decode_ffn, stack=_prepare_stack)


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, _generator(seed))


# ---------------------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------------------
def run(s):
    kind = s["c"]["kind"]
    if kind == "linear":                    # forward and straight-through backward
        pq.linear_fwd(s["desc"], s["X"], s["W"], s["Y"], s["bufs"], **s["hp"])
        pq.linear_bwd(s["desc"], s["dY"], s["X"], s["W"], s["bufs"], s["dX"], s["dW"], s["dab"], **s["hp"], **s["dhp"])
        return dict(Y=s["Y"], dX=s["dX"], dW=s["dW"], dab=s["dab"], **s["dhp"])
    if kind == "linear_norm":
        pq.linear_norm_fwd(s["desc"], s["X"], s["gain"], 1e-6, s["W"], s["Y"], s["bufs"], **s["hp"])
        pq.linear_norm_bwd(s["desc"], s["dY"], s["X"], s["gain"], s["W"], s["bufs"], s["dX"], s["dgain"], s["dW"], s["dab"],
                           **s["hp"], **s["dhp"])
        return dict(Y=s["Y"], dX=s["dX"], dgain=s["dgain"], dW=s["dW"], dab=s["dab"], **s["dhp"])
    if kind == "prefill":
        pq.linear_fwd(s["desc"], s["X"], s["P"], s["Y"], s["bufs"], A=s["A"], B=s["B"], mu_lambda=s["mu_lambda"], save=False)
        return s["Y"]
    if kind == "ffn":
        w, g = s["w"], s["g"]
        pq.ffn_fwd(s["desc"], s["X"], w["W_up"], w["W_gate"], w["W_down"], w["Up"], w["Gate"], w["Down"], w["Wr"], s["Y"], s["bufs"])
        pq.ffn_bwd(s["desc"], s["dY"], s["X"], w["Up"], w["Gate"], w["Down"], w["Wr"], s["bufs"], s["dX"], g["W_up"], g["W_gate"],
                   g["W_down"], g["Up"], g["Gate"], g["Down"], g["Wr"], s["dab"])
        return dict(Y=s["Y"], dX=s["dX"], dab=s["dab"], **g)
    if kind == "decode_linear":
        if s["c"]["hp"] == "int8":
            return pq.decode_gemv_int8(s["desc"], s["X"], s["P"], s["scale"], s["Y"], s["ws"], s["Aq"], s["gA"], s["Bq"], s["gB"], s["Wr"])
        return pq.decode_gemv(s["desc"], s["X"], s["P"], s["scale"], s["Y"], s["ws"], A=s["A"], B=s["B"], Wr=s["Wr"])
    if kind == "decode_ffn":
        return pq.decode_ffn(s["desc"], s["X"], s["Pug"], s["sug"], s["Pd"], s["sd"], s["UpGate"], s["Down"], s["Wr"], s["Y"], s["ws"])
    out = s["st"].forward(s["h0"], s["w"])
    dh = s["st"].backward(s["dY"], s["w"], s["g"])
    return dict(out=out, dh=dh, grads=s["g"])


# ---------------------------------------------------------------------------------------------------------------------
# what a pass cannot do without: every input read once, every output written once, every product formed once
# ---------------------------------------------------------------------------------------------------------------------
def _linear_work(T, K, N, r, E, k, es, norm=False):
    b = es * (2 * T * K + 2 * T * N + N * K) + 4 * N * K + (es * K + 4 * K if norm else 0)
    f = 6.0 * T * K * N
    if r:
        b += (es + 4) * E * r * (K + N) + ((es + 4) * E * K if E > 1 else 0)
        f += 6.0 * T * k * r * (K + N) + (6.0 * T * K * E if E > 1 else 0)
    return b, f


def _ffn_work(T, D, F, r, E, k):
    w = 3 * D * F + 3 * E * r * D + E * D
    return 2 * 4 * T * D + (2 + 4) * w, 18.0 * T * D * F + 18.0 * T * k * r * D + (6.0 * T * D * E if E > 1 else 0)


def work(case):
    c = case
    kind = c["kind"]
    if kind in ("linear", "linear_norm"):
        b, f = _linear_work(c["tokens"], c["d_in"], c["d_out"], c["rank"], c["experts"], c["top_k"], 4 if c["dtype"] == "f32" else 2,
                            kind == "linear_norm")
    elif kind == "prefill":
        T, K, N, r = c["tokens"], c["d_in"], c["d_out"], c["rank"]
        b, f = 2 * T * (K + N) + N * K // 8 + 2 * r * (K + N), 2.0 * T * K * N + 2.0 * T * r * (K + N)
    elif kind == "ffn":
        b, f = _ffn_work(c["tokens"], c["d_model"], c["d_ffn"], c["rank"], c["experts"], c["top_k"])
    elif kind == "decode_linear":
        L, B, K, N, E, r, k = c["layers"], c["batch"], c["d_in"], c["d_out"], c["experts"], c["rank"], c["top_k"]
        sel = E * (1.0 - (1.0 - k / E) ** B)     # distinct experts that B independent tokens choose
        b = L * (N * K / 8 + 2 * B * (K + N) + 2 * E * K + sel * r * (K + N) * (1 if c["hp"] == "int8" else 2))
        f = L * B * (2.0 * K * N + 2.0 * k * r * (K + N) + 2.0 * E * K)
    elif kind == "decode_ffn":
        L, B, D, F, E, r, k = c["layers"], c["batch"], c["d_model"], c["d_ffn"], c["experts"], c["rank"], c["top_k"]
        sel = E * (1.0 - (1.0 - k / E) ** B)
        b = L * (3 * D * F / 8 + 4 * B * D + 2 * E * D + sel * 3 * r * D * 2)
        f = L * B * (6.0 * D * F + 6.0 * k * r * D + 2.0 * E * D)
    else:
        T, D = c["tokens"], c["d_model"]
        lb, lf = _linear_work(T, D, D, 0, 1, 1, 2)
        fb, ff = _ffn_work(T, D, c["d_ffn"], c["rank"], c["experts"], c["top_k"])
        b, f = c["layers"] * (4 * lb + fb), c["layers"] * (4 * lf + ff)
    return {"bytes": float(b), "flops": float(f)}


# ---------------------------------------------------------------------------------------------------------------------
# how far another correct implementation of the same precision may be off
# Four times what the calls were measured to differ by from an fp64 evaluation of the same formulas that rounds nothing
# between the quantisers (300 to 512 tokens of the shapes above, scaled down); "max" is 40 times "rel" unless stated.
# ---------------------------------------------------------------------------------------------------------------------
def tolerance(case):
    kind = case["kind"]
    if case.get("dtype") == "f32":      # fp64 sums rounded once: 8e-8 (2-norm) and 7e-7 (largest) seen
        return {"rel": 4e-7, "max": 3e-6}
    if kind in ("decode_linear", "decode_ffn", "prefill"):      # bf16 outputs: 2.2e-3 seen
        return {"rel": 9e-3}
    if kind == "stack":     # a chain of quantisers: a bf16 rounding moves codes of the next layer; 8.2e-3 seen
        return {"rel": 3e-2}
    # bf16 tensors 2e-3 to 4.2e-3; the two scale gradients are sums of tokens * d_out terms of either sign, where what is
    # left carries up to 1.9e-2: another rounding of an intermediate may show as much as that once
    return {"rel": 2e-2}
