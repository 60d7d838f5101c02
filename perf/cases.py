"""Performance cases of the OptCC schedule executor on one MI355X.

A case is one AllReduce of p logical ranks' buffers through the package's
entry points: the profile (ranks, slow NICs, GPUs per server), the vector
length, the segment count, the element type, how the caller holds the buffers
and which of the three calls it makes.  ``listed()`` names twelve of them,
from a launch-bound message to the largest workload; ``draw()`` gives more of
the same ranges.

Keys of a case:
  p, g        ranks, GPUs per server (1: one rank per server)
  slow        bandwidths of the slow ranks (of the slow server when g > 1),
              "rank:bandwidth" joined by commas; every other NIC has 1.0
  n, k        elements per rank, segments (per part when g > 1)
  dtype       "f32", "bf16", "f16" or "i32"
  values      value recipe, see _rank_values
  layout      "rows": one contiguous [p, n] tensor, so that an odd n leaves
              most rows aligned to the element only; "list" (up to 64 ranks):
              p tensors of their own, each aligned by the allocator
  call        "fused" (optcc_allreduce_emulate), "staged" (one launch per
              stage slot) or "noalloc" (optcc_allreduce_emulate_noalloc)
"""
import math

import torch

from paper_2606_01680_amd import optcc

_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16, "i32": torch.int32}
_ESIZE = {"f32": 4, "bf16": 2, "f16": 2, "i32": 4}
_MAX_STATE = 8 << 30  # bytes of rank buffers of the largest case


def _case(name, p, slow, n, k, dtype, values="normal", g=1, layout="rows", call="fused"):
    return {"name": name, "p": p, "g": g, "slow": slow, "n": n, "k": k, "dtype": dtype,
            "values": values, "layout": layout, "call": call}


def listed():
    return [
        # the smallest message: four ranks, 256 KiB each, bound by launch and host
        _case("tiny_p4_f32", 4, "3:0.5", 1 << 16, 8, "f32"),
        # a small bucket over many ranks: one long serial chain per element
        _case("small_p128_f32", 128, "124:0.875,125:0.75,126:0.5,127:0.5", 1 << 16, 256, "f32",
              "student_t3_1e-3"),
        # an ordinary gradient bucket (8 MiB per rank), one of eight NICs lost
        _case("bucket_p8_f32", 8, "7:0.875", 1 << 21, 64, "f32"),
        # an odd-length integer vector in one [p, n] tensor: rows aligned to 4 bytes
        _case("odd_p8_i32", 8, "7:0.875", 5_000_011, 64, "i32", "uniform_2p20"),
        # an odd-length fp16 vector in one [p, n] tensor: rows aligned to 2 bytes
        _case("odd_p16_f16", 16, "15:0.5", 3_000_017, 128, "f16", "normal_1e-2"),
        # the p = 8 workload at full size (256 MiB per rank)
        _case("full_p8_f32", 8, "7:0.875", 1 << 26, 64, "f32"),
        # the p = 16 workload at full size, bf16 gradients
        _case("full_p16_bf16", 16, "15:0.5", 1 << 26, 128, "bf16", "normal_1e-2"),
        # two stragglers among 64 ranks at full size
        _case("full_p64_f32", 64, "62:0.75,63:0.5", 1 << 24, 128, "f32", "normal_zeros1pct"),
        # the largest workload: four stragglers among 128 ranks (8 GiB of buffers)
        _case("full_p128_f32", 128, "124:0.875,125:0.75,126:0.5,127:0.5", 1 << 24, 256, "f32",
              "student_t3_1e-3"),
        # four servers of four GPUs, a ragged bf16 bucket in tensors of their own
        _case("bucket_q4g4_bf16", 16, "0:0.5", 4_200_005, 128, "bf16", "normal_1e-2", g=4,
              layout="list"),
        # sixteen servers of four GPUs at full size
        _case("full_q16g4_f32", 64, "15:0.5", 1 << 24, 128, "f32", g=4),
        # the AllReduce one stage slot at a time (stage-by-stage study)
        _case("staged_p8_f32", 8, "7:0.875", 1 << 22, 64, "f32", call="staged"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    dtype = rng.choice(["f32", "f32", "bf16", "f16", "i32"])
    es = _ESIZE[dtype]
    servers = rng.random() < 0.25
    if servers:
        g = rng.choice([2, 4, 4, 8])
        q = _log_uniform(rng, 3, 128 // g)
        p = q * g
        slow = f"{rng.randrange(q)}:{rng.choice([0.5, 0.75, 0.875])}"
        k = 8 * rng.randint(3, 16)
    else:
        g = 1
        p = _log_uniform(rng, 3, 256)
        m = min(rng.choice([0, 1, 1, 1, 2, 4]), p - 2)
        ranks = rng.sample(range(p), m)
        slow = ",".join(f"{r}:{rng.choice([0.25, 0.5, 0.75, 0.875])}" for r in ranks)
        k = 4 * rng.randint(2, 64)
    layout = rng.choice(["rows", "list"]) if p <= 64 else "rows"
    call = rng.choice(["fused", "fused", "fused", "fused", "staged", "noalloc"])
    odd = rng.random() < 0.5
    # what moves more than the bare AllReduce stays below a quarter of the largest size
    cap = _MAX_STATE if call == "fused" and not (odd and layout == "rows") else _MAX_STATE // 4
    n = _log_uniform(rng, 1 << 12, min(1 << 26, cap // (p * es) - 64))
    n = n | 1 if odd else max(n - n % 64, 64)
    values = "uniform_2p20" if dtype == "i32" else ("normal" if dtype == "f32" else "normal_1e-2")
    c = _case(None, p, slow, n, k, dtype, values, g, layout, call)
    del c["name"]
    return c


def _bandwidths(case):
    b = [1.0] * (case["p"] // case["g"])
    for item in case["slow"].split(","):
        if item:
            r, v = item.split(":")
            b[int(r)] = float(v)
    return b


def _rank_values(case, seed, r):
    """Rank r's input: gradient-like values, made on the GPU from the seed."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed((seed * 1009 + r * 7919 + 2606) % (1 << 62))
    n, values = case["n"], case["values"]
    if values == "uniform_2p20":
        return torch.randint(-(1 << 20), (1 << 20) + 1, (n,), generator=gen, device="cuda",
                             dtype=torch.int32)
    x = torch.randn(n, generator=gen, device="cuda")
    if values == "normal_1e-2":
        x *= 1e-2
    elif values == "normal_zeros1pct":
        x *= torch.rand(n, generator=gen, device="cuda") >= 0.01
    elif values == "student_t3_1e-3":
        c = torch.randn((3, n), generator=gen, device="cuda").pow_(2).sum(0)
        x = x / torch.sqrt(c / 3.0) * 1e-3
    elif values != "normal":
        raise ValueError(f"unknown value recipe {values!r}")
    return x.to(_TORCH[case["dtype"]])


def prepare(case, seed):
    """The rank buffers and the plan, as a training program holds them."""
    p, n, g = case["p"], case["n"], case["g"]
    if case["layout"] == "rows":
        bufs = torch.empty((p, n), dtype=_TORCH[case["dtype"]], device="cuda")
        for r in range(p):
            bufs[r].copy_(_rank_values(case, seed, r))
    else:
        bufs = [_rank_values(case, seed, r) for r in range(p)]
    bw = _bandwidths(case)
    if g > 1:
        plan = optcc.optcc_plan_servers(p // g, g, bw, n, case["k"])
    else:
        plan = optcc.optcc_plan(p, bw, n, case["k"])
    return {"case": case, "bufs": bufs, "plan": plan}


def run(state):
    """One AllReduce in place; every rank's buffer is an output."""
    c, bufs, plan = state["case"], state["bufs"], state["plan"]
    if c["call"] == "staged":
        optcc.optcc_allreduce_emulate_slots(bufs, c["p"], c["n"], c["dtype"], plan, 0,
                                            plan.num_slots, launches=0)
    elif c["call"] == "noalloc":
        optcc.optcc_allreduce_emulate_noalloc(bufs, c["p"], c["n"], c["dtype"], plan)
    else:
        optcc.optcc_allreduce_emulate(bufs, c["p"], c["n"], c["dtype"], plan)
    return bufs


def work(case):
    """Every rank's input read once and its result written once; one addition
    per rank and element beyond the first."""
    p, n = case["p"], case["n"]
    return {"bytes": 2 * p * n * _ESIZE[case["dtype"]], "flops": (p - 1) * n}


def tolerance(case):
    """The schedule fixes the order of every element's additions and the
    rounding of each step, so results are the same bit for bit."""
    return "exact"


def exact(case, seed):
    """The sum over ranks in 64 bits, once per rank as the AllReduce leaves it."""
    p, n = case["p"], case["n"]
    integer = case["dtype"] == "i32"
    s = torch.zeros(n, dtype=torch.int64 if integer else torch.float64, device="cuda")
    for r in range(p):
        s += _rank_values(case, seed, r)
    if integer:  # additions modulo 2^32
        s = ((s + (1 << 31)) % (1 << 32) - (1 << 31)).to(torch.int32)
    return s.expand(p, n) if case["layout"] == "rows" else [s] * p
