"""Every split contraction of a library call leaves its slabs inside the section that the call's workspace query reserved for it
(the launches compare the two and refuse with PQ_ERR_WORKSPACE): whole training and prefill calls, run on the host alone, over
random sizes of everything the descriptors accept, far beyond the sizes the workloads use."""
import ctypes
import math
import os
import random

import pytest

from launch_trace import trace
from paper_2602_22592_amd import binding as pq


@pytest.fixture(scope="module", autouse=True)
def built():
    if not os.path.exists(pq.LIB_PATH):
        from paper_2602_22592_amd.build import build
        build(verbose=False)


def _spread(rng, lo, hi, step):
    return max(step, int(math.exp(rng.uniform(math.log(lo), math.log(hi)))) // step * step)


def _linear(rng, kind):
    c = dict(op="prefill" if kind == "prefill" else "linear", tokens=_spread(rng, 1, 20000, 1), d_in=_spread(rng, 32, 9000, 32),
             d_out=_spread(rng, 32, 12000, 32))
    if kind == "int8_large":       # where the branch's share of dX is most often a launch of its own
        c.update(tokens=_spread(rng, 256, 1000, 1), d_in=_spread(rng, 3000, 7000, 32), d_out=_spread(rng, 3000, 7000, 32), hp_kind=1,
                 hp_rank=_spread(rng, 2000, 4096, 32))
    elif kind == "int8":
        c.update(hp_kind=1, hp_rank=_spread(rng, 32, 4096, 32))
    elif kind == "routed":
        c.update(n_experts=rng.choice([2, 3, 8, 16, 64]), hp_rank=_spread(rng, 8, 4096, 8))
        c["top_k"] = rng.choice([1, 2, min(8, c["n_experts"])])
    elif kind != "none":
        c.update(hp_rank=_spread(rng, 8, 4096, 8))
    if kind == "norm":
        c.update(op="linear_norm", d_in=min(c["d_in"], 4096), hp_kind=rng.choice([0, 1]), hp_rank=_spread(rng, 32, 4096, 32))
    if kind == "f32":
        c["io_dtype"] = 0
    return c


def _ffn(rng):
    E = rng.choice([1, 1, 2, 8, 64])
    return dict(op="ffn", tokens=_spread(rng, 1, 20000, 1), d_model=_spread(rng, 32, 8000, 32), d_ffn=_spread(rng, 32, 12000, 4), n_experts=E,
                top_k=rng.choice([1, min(2, E), min(8, E)]), hp_kind=rng.choice([0, 1]), hp_rank=_spread(rng, 32, 2048, 32))


def draw(rng):
    kind = rng.choice(["dense", "none", "int8", "int8_large", "routed", "norm", "prefill", "f32", "ffn", "ffn", "hp_int8"])
    if kind == "ffn":
        return _ffn(rng)
    if kind == "hp_int8":
        return dict(op="hp_int8", tokens=_spread(rng, 1, 20000, 1), d_in=_spread(rng, 32, 9000, 32), d_out=_spread(rng, 32, 12000, 32),
                    hp_rank=_spread(rng, 32, 4096, 32))
    return _linear(rng, kind)


# INT8 branch of a large rank behind a split 256x256 input-gradient product: the branch's share of dX is a launch of its own
# whose plan has more splits than the first one's
LARGE_RANK = [(658, 3712, 4000, 2560), (389, 5376, 6368, 2752), (452, 4768, 4640, 2592), (601, 3712, 4032, 2432)]


def test_large_rank_int8_branch():
    calls = [dict(op=op, tokens=T, d_in=min(K, 4096) if op == "linear_norm" else K, d_out=N, hp_rank=r, hp_kind=1)
             for T, K, N, r in LARGE_RANK for op in ("linear", "linear_norm")]
    for c, r in zip(calls, trace(calls)):
        assert r["rc"] == 0, (c, r["error"])


@pytest.mark.parametrize("seed", range(4))
def test_random_calls(seed):
    rng = random.Random(seed)
    calls = [draw(rng) for _ in range(500)]
    for c, r in zip(calls, trace(calls)):
        assert r["rc"] == 0, (c, r["error"])


# bytes that these calls have taken since before the router counted its experts for the ordering of the slots; a workspace allocated once for
# a model's layers is kept over versions of the library
LINEAR_BYTES = {(1, 32, 32, 8, 64, 1): 27136, (9, 64, 32, 8, 64, 1): 41472, (105, 5152, 32, 64, 64, 8): 16403712, (1531, 1056, 3104, 24, 4, 2): 30470400,
                (2100, 64, 96, 8, 16, 3): 4332032}
FFN_BYTES = {(1, 32, 36, 8, 64, 1, 0): 60928, (64, 256, 512, 128, 1, 1, 0): 837376, (2048, 2048, 5076, 384, 1, 1, 1): 119200768,
             (300, 512, 1020, 24, 4, 2, 0): 4249856, (35, 64, 164, 32, 64, 8, 1): 850688}


def test_routed_calls_take_no_larger_workspace():
    sizes = {}
    for T, K, N, r, E, k in LINEAR_BYTES:
        sizes[T, K, N, r, E, k] = pq.lib().pq_linear_workspace_bytes(ctypes.byref(pq.make_desc(T, K, N, hp_rank=r, n_experts=E, top_k=k)))
    assert all(n <= LINEAR_BYTES[c] for c, n in sizes.items()), sizes
    sizes = {}
    for T, D, F, r, E, k, i8 in FFN_BYTES:
        sizes[T, D, F, r, E, k, i8] = pq.lib().pq_ffn_workspace_bytes(ctypes.byref(pq.FFNDesc(T, D, F, r, E, k, pq.PQ_BF16, 2.0, 0.2, i8)))
    assert all(n <= FFN_BYTES[c] for c, n in sizes.items()), sizes
    calls = [dict(op="linear", tokens=T, d_in=K, d_out=N, hp_rank=r, n_experts=E, top_k=k, workspace_bytes=n)
             for (T, K, N, r, E, k), n in LINEAR_BYTES.items()]
    calls += [dict(op="ffn", tokens=T, d_model=D, d_ffn=F, hp_rank=r, n_experts=E, top_k=k, hp_kind=i8) for T, D, F, r, E, k, i8 in FFN_BYTES]
    for c, r in zip(calls, trace(calls)):
        assert r["rc"] == 0, (c, r["error"])
