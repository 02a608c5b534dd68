"""Every split contraction of a library call leaves its slabs inside the section that the call's workspace query reserved for it
(the launches compare the two and refuse with PQ_ERR_WORKSPACE): whole training and prefill calls, run on the host alone, over
random sizes of everything the descriptors accept, far beyond the sizes the workloads use."""
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
