"""GPU parity: the HIP executor against the oracle, through the C ABI.

Every case compares every element of every rank bit for bit with the
oracle's serial execution (fp32, bf16 and int32 alike: the schedule fixes the
reduction order; fp16 likewise), from small ragged cases to the full-size workloads.  Slot
prefixes check that every step is materialised in its destination buffer,
stage by stage.  Full-size runs also check properties that hold at any size
(all ranks identical, exact int32 sums, the fp error bound) and sampled
coordinates through the oracle's per-coordinate executor.
"""
import sys

import numpy as np
import pytest
import torch

import oracle
from gpu_util import (bits_equal, call_choice, int_view, rand_inputs, run_slots, to_device,
                      to_host)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def o():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_01680_amd import optcc
    return optcc


def _bw(p, slow):
    b = [1.0] * p
    for r, v in slow.items():
        b[r] = v
    return b


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


PROFILES = [
    (3, {}), (3, {2: 0.5}), (4, {3: 0.5}), (5, {0: 0.5}), (5, {2: 0.75}), (8, {7: 0.875}),
    (8, {3: 0.25}), (6, {0: 0.5, 5: 0.75}), (9, {0: 0.875, 3: 0.75, 8: 0.5}), (16, {15: 0.5}),
    (12, {}), (20, {1: 0.5, 2: 0.5, 19: 0.9}), (40, {5: 0.6}),
    # degenerate profiles: two healthy ranks, slowdown barely above 1, just
    # under and exactly at l = 2
    (4, {0: 0.5, 1: 0.75}), (5, {1: 0.5, 2: 0.5, 3: 0.5}), (8, {2: 0.9999999}),
    (6, {5: 0.50000001}), (6, {5: 0.5}),
]
# sizes span several tiles (at these sizes 1024 elements for 4-byte types,
# 2048 for 2-byte types), ragged tails, empty sections
SIZES = [(1, 4), (37, 4), (64, 4), (1000, 8), (2048 * 3 + 64 * 5 + 3, 8), (40000, 12)]


def _run_both(o, p, slow, n, k, dtype, seed, kind="normal", slot_end=6, launches=1):
    bw = _bw(p, slow)
    x = rand_inputs(dtype, p, n, seed, kind)
    ref = oracle.run(oracle.Schedule(p, bw, n, k), dtype, x.copy(), 0, slot_end)
    pl = o.optcc_plan(p, bw, n, k)
    d = to_device(x, dtype)
    o.optcc_allreduce_emulate_slots(d, p, n, dtype, pl, 0, slot_end, launches)
    torch.cuda.synchronize()
    return x, ref, to_host(d, dtype)


@pytest.mark.parametrize("dtype", ["f32", "bf16", "i32", "f16"])
@pytest.mark.parametrize("p,slow", PROFILES)
@pytest.mark.parametrize("n,k", SIZES)
def test_small_bit_exact(o, dtype, p, slow, n, k):
    _say(f"case dtype={dtype} p={p} slow={slow} n={n} k={k}")
    x, ref, got = _run_both(o, p, slow, n, k, dtype, seed=p * 1000 + n)
    assert bits_equal(got, ref)
    if n:
        assert (got == got[0][None, :]).all()


@pytest.mark.parametrize("dtype,p,slow,n,k", [
    # 2048-element tiles (two vectors per lane) with a sub-vector tail, and
    # just below the size where they start (1024-element tiles)
    ("f32", 8, {7: 0.875}, (1 << 21) + 2048 * 3 + 64 * 5 + 3, 64),
    ("i32", 8, {7: 0.875}, (1 << 21) + 2048 * 3 + 64 * 5 + 3, 64),
    ("f32", 8, {7: 0.875}, (1 << 21) - 64 * 3 + 1, 64),
    # 4096-element tiles (fp32 p = 4; fp16 p = 6) and 8192 (bf16 p = 3)
    ("f32", 4, {3: 0.5}, (1 << 22) + 5, 8),
    ("f16", 6, {5: 0.5}, (1 << 22) + 2048 + 9, 16),
    ("bf16", 3, {2: 0.5}, (1 << 23) + 77, 8),
])
def test_tile_lengths_bit_exact(o, dtype, p, slow, n, k):
    """Every tile length the launch picks (1024 to 8192 elements: longer for
    plans that move little per element, shorter for small messages), each
    with ragged tiles at segment ends, bit for bit against the oracle."""
    _say(f"case tiles dtype={dtype} p={p} slow={slow} n={n} k={k}")
    x, ref, got = _run_both(o, p, slow, n, k, dtype, seed=5 * p + n % 97)
    assert bits_equal(got, ref)


@pytest.mark.parametrize("dtype", ["f32", "i32"])
@pytest.mark.parametrize("p,slow,n,k", [
    (8, {7: 0.875}, (1 << 20) + 12345, 64),   # 5 to 7 healthy: 1024-element tiles
    (6, {0: 0.5}, (1 << 21) + 77, 16),
    (7, {}, (1 << 20) + 3, 8),                  # no straggler: the ring
    (4, {3: 0.5}, (1 << 22) + 999, 8),          # 3 healthy: the plan's own tile length
    (9, {0: 0.875, 3: 0.75, 8: 0.5}, (1 << 20) + 64 * 5 + 1, 12),
])
def test_mid_size_short_chains_bit_exact(o, dtype, p, slow, n, k):
    """Short chains of 32-bit elements whose rank buffers total 16 MiB to
    2 GiB run one vector per lane in the identity tile order on the general
    kernel: as two slot ranges, and the whole AllReduce on the chain kernel,
    every element of every rank bit for bit against the oracle, ragged tails
    included."""
    _say(f"case mid-size short chain dtype={dtype} p={p} slow={slow} n={n} k={k}")
    x, ref, got = _run_both(o, p, slow, n, k, dtype, seed=61 + p)
    assert bits_equal(got, ref)
    pl = o.optcc_plan(p, _bw(p, slow), n, k)
    d = to_device(x, dtype)
    run_slots(o, d, p, n, dtype, pl, (5,), two=0, xcd_runs=0)
    torch.cuda.synchronize()
    assert bits_equal(to_host(d, dtype), ref)


@pytest.mark.parametrize("dtype", ["f32", "i32"])
@pytest.mark.parametrize("p,n", [(20, (16 << 20) // 80 + 1), (20, (1 << 20) + 7), (22, (1 << 18) + 2),
                                 (24, (16 << 20) // 96 + 3), (24, (1 << 22) + 64 * 5 + 1),
                                 (24, 20_000_003)])
def test_pipelined_ring_tiles(o, dtype, p, n):
    """Whole AllReduces of 3 to 7 healthy ranks and 17 stragglers, 16 MiB to
    1.8 GiB of buffers, in tiles that carry a vector's allgather stores into the
    next vector's chain: ragged tiles, rows aligned to the element only, every
    rest past the last vector, bit for bit against the oracle."""
    slow, k = {i: 0.5 if i % 3 else 0.25 for i in range(17)}, 12
    bw = _bw(p, slow)
    pl = o.optcc_plan(p, bw, n, k)
    c = call_choice(o, pl, dtype)
    assert c.kernel == "general" and c.pipe == 1
    _say(f"case pipelined tiles dtype={dtype} p={p} n={n}")
    x, ref, got = _run_both(o, p, slow, n, k, dtype, seed=p + n % 89)
    assert bits_equal(got, ref)


@pytest.mark.parametrize("p,n", [(40, 1 << 17), (64, 1 << 18), (64, (1 << 19) + 4097),
                                 # 62 healthy ranks keep the runs up to 4,096 tiles
                                 (64, 1024 * 4000 + 3)])
def test_long_chains_one_round_of_tiles(o, p, n):
    """Long chains whose tiles fit in one round of resident workgroups take
    the identity tile order, more tiles the per-XCD runs: both bit for bit as
    slot ranges, and the whole AllReduce on the chain kernel."""
    slow = {p - 1: 0.5, p - 2: 0.75}
    _say(f"case long chain p={p} n={n}")
    x, ref, got = _run_both(o, p, slow, n, 16, "f32", seed=7 + p)
    assert bits_equal(got, ref)
    d = to_device(x, "f32")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    run_slots(o, d, p, n, "f32", o.optcc_plan(p, _bw(p, slow), n, 16), (5,),
              xcd_runs=int(n > 1024 * cus), steal=0, per_cu=1)
    torch.cuda.synchronize()
    assert bits_equal(to_host(d, "f32"), ref)


@pytest.mark.parametrize("dtype", ["f32", "bf16", "i32", "f16"])
@pytest.mark.parametrize("p,slow", [(5, {0: 0.5}), (8, {7: 0.875}), (9, {0: 0.875, 3: 0.75, 8: 0.5}),
                                    (7, {}), (6, {1: 0.25, 2: 0.5})])
@pytest.mark.parametrize("launches", [1, 0])
def test_stage_snapshots(o, dtype, p, slow, launches):
    """After the first s slots (s = 1..6), in one fused launch or one launch
    per slot, every buffer equals the oracle's state after the same slots:
    every step's destination write is materialised."""
    n, k = 2048 * 2 + 64 * 7 + 5, 8
    for s in range(1, 7):
        _say(f"case snapshot dtype={dtype} p={p} slots=[0,{s}) launches={launches}")
        x, ref, got = _run_both(o, p, slow, n, k, dtype, seed=17 + s, slot_end=s, launches=launches)
        assert bits_equal(got, ref), f"slots [0,{s})"


@pytest.mark.parametrize("dtype,kind", [(d, k) for d in ("f32", "bf16", "f16")
                                         for k in ("denormal", "wide")] + [("f16", "overflow")])
def test_special_values(o, dtype, kind):
    """Subnormal inputs (no flush to zero on either side), values spread over
    the format's binades (heavy cancellation) and, for fp16, partial sums
    beyond the largest finite half (rounded to infinity on both sides) stay
    bit-exact."""
    for p, slow in [(5, {0: 0.5}), (8, {7: 0.875}), (9, {0: 0.875, 3: 0.75, 8: 0.5})]:
        _say(f"case special {kind} dtype={dtype} p={p}")
        x, ref, got = _run_both(o, p, slow, 5000, 8, dtype, seed=3, kind=kind)
        assert bits_equal(got, ref)
        if kind == "overflow":
            assert np.isinf(oracle.f16_to_f64(got)).any()


def _put_specials(x, dtype, share, rng):
    """Overwrite a share of x's elements with NaNs of random sign and payload
    (quiet and signalling) and, three in ten, infinities."""
    man = {"f32": 23, "bf16": 7, "f16": 10}[dtype]
    u = x.view(np.uint32) if dtype == "f32" else x
    hit = rng.random(u.shape) < share
    m = int(hit.sum())
    payload = rng.integers(0, 1 << man, m) * (rng.random(m) >= 0.3)
    bits = 8 * u.itemsize
    expo = ((1 << (bits - 1 - man)) - 1) << man
    u[hit] = (expo | payload | rng.integers(0, 2, m) << (bits - 1)).astype(u.dtype)


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("p,g,slow", [
    (4, 1, {3: 0.5}), (8, 1, {7: 0.875}), (9, 1, {0: 0.875, 3: 0.75, 8: 0.5}), (9, 1, {0: 0.875}),
    (13, 1, {}), (17, 1, {2: 0.75}), (24, 1, {i: 0.5 for i in range(9)}), (33, 1, {32: 0.875}),
    (40, 1, {3: 0.5}), (100, 1, {0: 0.75, 9: 0.5}), (6, 2, {1: 0.5}), (16, 4, {0: 0.5}),
    (40, 8, {4: 0.75})])
def test_nan_and_infinity(o, dtype, p, g, slow):
    """NaNs of any payload and infinities: the whole AllReduce bit for bit, so
    that a step whose operands are both NaN keeps its destination's (a step is
    own value + received value), and one launch per slot the same up to the
    payload of such a NaN, whose choice IEEE 754 leaves open."""
    q, k, n = p // g, 24, 64 * 400 + 7
    bw = _bw(q, slow)
    if g > 1:
        sch, pl = oracle.Schedule.servers(q, g, bw, n, k), o.optcc_plan_servers(q, g, bw, n, k)
    else:
        sch, pl = oracle.Schedule(p, bw, n, k), o.optcc_plan(p, bw, n, k)
    rng = np.random.default_rng(5 * p + g)
    for share in (0.2 / p, 0.3):
        _say(f"case nan and infinity dtype={dtype} p={p} g={g} share={share:.3f}")
        x = rand_inputs(dtype, p, n, 3 * p).copy()
        _put_specials(x, dtype, share, rng)
        ref = oracle.run(sch, dtype, x.copy())
        d, d2 = to_device(x, dtype), to_device(x, dtype)
        o.optcc_allreduce_emulate(d, p, n, dtype, pl)
        o.optcc_allreduce_emulate_slots(d2, p, n, dtype, pl, 0, pl.num_slots, 0)
        torch.cuda.synchronize()
        nan = torch.isnan(to_device(ref, dtype))
        assert bool(nan.any())
        assert bits_equal(to_host(d, dtype), ref)
        assert torch.equal(torch.isnan(d2), nan)
        assert torch.equal(int_view(d2)[~nan], int_view(d)[~nan])


@pytest.mark.parametrize("dtype", ["f32", "bf16", "i32", "f16"])
def test_unaligned_buffers(o, dtype):
    """Rank buffers that are only element-aligned."""
    p, n, k = 8, 3000, 8
    bw = _bw(p, {7: 0.875})
    x = rand_inputs(dtype, p, n, 5)
    ref = oracle.run(oracle.Schedule(p, bw, n, k), dtype, x.copy())
    pl = o.optcc_plan(p, bw, n, k)
    stride = n + 1  # rank r starts at 1 + r*(n+1) elements: not 16-byte aligned
    flat = torch.zeros(p * stride + 8, dtype=to_device(x[:1, :1], dtype).dtype, device="cuda:0")
    for r in range(p):
        flat[1 + r * stride: 1 + r * stride + n].copy_(to_device(x[r:r + 1], dtype)[0])
    views = [flat[1 + r * stride: 1 + r * stride + n] for r in range(p)]
    _say(f"case unaligned dtype={dtype}")
    o.optcc_allreduce_emulate(views, p, n, dtype, pl)
    torch.cuda.synchronize()
    got = np.stack([to_host(v, dtype) for v in views])
    assert bits_equal(got, ref)


# healthy ranks on both sides of every register bucket of the chain kernel, and
# more stragglers than its short pointer table holds
CHAIN_EDGES = [(9, {8: 0.5}), (10, {8: 0.5}), (17, {0: 0.875}), (18, {0: 0.875}), (32, {}),
               (33, {}), (66, {3: 0.5, 65: 0.75}), (67, {3: 0.5, 65: 0.75}), (128, {}),
               (129, {1: 0.75}), (30, {i: 0.5 for i in range(9, 29)}), (70, {i: 0.25 for i in range(68)})]


@pytest.mark.parametrize("dtype", ["f32", "bf16", "i32", "f16"])
@pytest.mark.parametrize("p,slow", CHAIN_EDGES)
def test_chain_buckets_bit_exact(o, dtype, p, slow):
    """Chains held in registers: one-quantum sections (waves that straddle many),
    a tail shorter than a lane's vector, and rows of one [p, n] tensor with odd
    n (aligned to the element only), bit for bit against the oracle."""
    n, k = 64 * 301 + 13, 8
    _say(f"case chain bucket dtype={dtype} p={p} n={n}")
    x, ref, got = _run_both(o, p, slow, n, k, dtype, seed=11 * p)
    assert bits_equal(got, ref)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("p,slow,n,k", [
    (3, {2: 0.5}, (1 << 25) + 21, 8),             # up to 448 MiB, then beyond
    (3, {2: 0.5}, (1 << 26) + 21, 8),
    (7, {0: 0.875}, (1 << 24) + 64 * 9 + 3, 16),
    (12, {11: 0.75}, 7_000_001, 64),
    (9, {}, (1 << 24) + 7, 8),
    (24, {5: 0.5, 6: 0.25}, 3_500_003, 16),
    (40, {}, (1 << 21) + 1, 64),
    (60, {59: 0.5}, (1 << 21) + 65, 64),
    (100, {0: 0.875}, (1 << 20) + 129, 64),
    (126, {7: 0.5, 9: 0.75}, (1 << 20) + 3, 64),
])
def test_chain_shapes_equal_noalloc_and_sum(o, dtype, p, slow, n, k):
    """Launch shapes above the memory-side cache's size, on rows that begin on a
    line and on rows aligned to the element only (which the no-allocation entry
    point runs on the chain kernel too): sampled coordinates bit for bit against
    the oracle, every rank equal, and the no-allocation entry point gives the same
    bits."""
    for n in (n, n // 64 * 64):
        _chain_shape(o, dtype, p, slow, n, k)


def _chain_shape(o, dtype, p, slow, n, k):
    _say(f"case chain shape dtype={dtype} p={p} n={n}")
    bw = _bw(p, slow)
    from paper_2606_01680_amd.workloads import make_rank
    x = torch.stack([make_rank("normal", dtype, n, 31 * p + r, "cuda:0") for r in range(p)])
    x0 = x.clone()
    pl = o.optcc_plan(p, bw, n, k)
    assert call_choice(o, pl, dtype).kernel == "chain"
    assert call_choice(o, pl, dtype, noalloc=True, align=2).kernel == "chain"
    o.optcc_allreduce_emulate(x, p, n, dtype, pl)
    torch.cuda.synchronize()
    rng = np.random.default_rng(p)
    coords = _sample_coords(pl, n, rng)
    idx = torch.from_numpy(coords).to("cuda:0")
    cols = to_host(x0[:, idx], dtype).copy()
    oracle.run_sampled(oracle.Schedule(p, bw, n, k), dtype, cols, coords)
    assert bits_equal(to_host(x[:, idx], dtype), cols)
    iv = int_view(x)
    for r in range(1, p):
        assert torch.equal(iv[r], iv[0]), r
    o.optcc_allreduce_emulate_noalloc(x0, p, n, dtype, pl)
    torch.cuda.synchronize()
    assert torch.equal(int_view(x0), iv)


@pytest.mark.parametrize("n,k", [(64 * 33000, 131076), (64 * 40, 400), (64 * 1000 + 1, 996)])
def test_chain_many_segments(o, n, k):
    """More segments than 32-bit segment arithmetic takes (quanta times segments
    of 2^32 or more), more segments than quanta, and about one quantum each."""
    p, slow = 6, {5: 0.75}
    _say(f"case many segments n={n} k={k}")
    x, ref, got = _run_both(o, p, slow, n, k, "f32", seed=k)
    assert bits_equal(got, ref)


# healthy servers on both sides of every register bucket, for each g that has one
SERVER_EDGES = [(3, 2), (8, 2), (9, 2), (16, 2), (17, 2), (25, 2), (32, 2), (33, 2), (64, 2),
                (3, 4), (4, 4), (5, 4), (8, 4), (9, 4), (13, 4), (16, 4), (17, 4), (32, 4),
                (3, 8), (4, 8), (5, 8), (7, 8), (8, 8), (9, 8), (16, 8), (4, 3)]


@pytest.mark.parametrize("dtype", ["f32", "bf16", "i32", "f16"])
@pytest.mark.parametrize("q,g", SERVER_EDGES)
def test_server_chain_buckets_bit_exact(o, dtype, q, g):
    """Server chains held in registers: parts and segments of two lengths,
    one-quantum sections, a tail shorter than a lane's vector and rows aligned
    to the element only, bit for bit against the oracle, for a first, middle or
    last straggler server; fewer quanta than parts takes the general kernel."""
    bw = [1.0] * q
    bw[(q * g) % q if g == 2 else (0 if g == 4 else q // 2)] = 0.625
    p, k = q * g, 24
    for n in (64 * 211 + 37, 64 * (g - 1)):
        _say(f"case server bucket dtype={dtype} q={q} g={g} n={n}")
        x = rand_inputs(dtype, p, n, 13 * p + g)
        ref = oracle.run(oracle.Schedule.servers(q, g, bw, n, k), dtype, x.copy())
        pl = o.optcc_plan_servers(q, g, bw, n, k)
        d = to_device(x, dtype)
        o.optcc_allreduce_emulate(d, p, n, dtype, pl)
        d2 = to_device(x, dtype)
        o.optcc_allreduce_emulate_noalloc(d2, p, n, dtype, pl)
        torch.cuda.synchronize()
        assert bits_equal(to_host(d, dtype), ref)
        assert bits_equal(to_host(d2, dtype), ref)


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("q,g,n", [(3, 2, 8_000_001), (4, 2, 1 << 24), (5, 4, 2_500_003),
                                   (6, 4, 6_000_001), (6, 8, 5_000_003), (16, 4, 1_000_001),
                                   (8, 8, 4_000_001), (32, 4, 1 << 18), (64, 2, 2_000_003),
                                   (16, 8, 5_000_001)])
def test_server_chain_shapes(o, dtype, q, g, n):
    """Launch shapes above 80, 448 and 1000 MiB of rank buffers, on rows that
    begin on a line and on rows aligned to the element only (which the
    no-allocation entry point runs on the chain kernel too): sampled coordinates
    bit for bit against the oracle, every rank equal, and the no-allocation entry
    point gives the same bits."""
    for n in (n, n // 64 * 64):
        _server_chain_shape(o, dtype, q, g, n)


def _server_chain_shape(o, dtype, q, g, n):
    _say(f"case server shape dtype={dtype} q={q} g={g} n={n}")
    from paper_2606_01680_amd.workloads import make_rank
    p, k = q * g, 64
    bw = [1.0] * (q - 1) + [0.5]
    x = torch.stack([make_rank("normal", dtype, n, 17 * p + r, "cuda:0") for r in range(p)])
    pl = o.optcc_plan_servers(q, g, bw, n, k)
    coords = _sample_coords(pl, n, np.random.default_rng(p))
    idx = torch.from_numpy(coords).to("cuda:0")
    cols = to_host(x[:, idx], dtype).copy()
    x0 = x.clone()
    assert call_choice(o, pl, dtype).kernel == "server chain"
    assert call_choice(o, pl, dtype, noalloc=True, align=2).kernel == "server chain"
    o.optcc_allreduce_emulate_noalloc(x0, p, n, dtype, pl)
    o.optcc_allreduce_emulate(x, p, n, dtype, pl)
    torch.cuda.synchronize()
    assert torch.equal(int_view(x0), int_view(x))
    del x0
    oracle.run_sampled(oracle.Schedule.servers(q, g, bw, n, k), dtype, cols, coords)
    assert bits_equal(to_host(x[:, idx], dtype), cols)
    iv = int_view(x)
    for r in range(1, p):
        assert torch.equal(iv[r], iv[0]), r


def test_deterministic_and_stream(o):
    """Same inputs, same bits, on the default stream and a side stream."""
    p, n, k = 9, 50000, 8
    bw = _bw(p, {0: 0.875, 3: 0.75, 8: 0.5})
    x = rand_inputs("f32", p, n, 9)
    pl = o.optcc_plan(p, bw, n, k)
    a = to_device(x, "f32")
    b = to_device(x, "f32")
    o.optcc_allreduce_emulate(a, p, n, "f32", pl)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        o.optcc_allreduce_emulate(b, p, n, "f32", pl, stream=s)
    torch.cuda.synchronize()
    assert torch.equal(a.view(torch.int32), b.view(torch.int32))


# ----------------------------------------------------------- full workloads
def _sample_coords(plan, n, rng, count=4096):
    """Random coordinates plus every segment's first and last element, both
    sides of each P2P chunk boundary and the vector's ends."""
    off, ln, p2p = plan.segments()
    picks = set(rng.integers(0, n, size=count).tolist())
    for g in range(len(off)):
        b, e = int(off[g]), int(off[g] + ln[g])
        for c in (b, e - 1, e - int(p2p[g]), e - int(p2p[g]) - 1):
            if 0 <= c < n:
                picks.add(c)
    picks.update([0, n - 1])
    return np.array(sorted(picks), dtype=np.int64)


WORKLOADS = ["p4_f32", "p8_f32", "p8_i32", "p16_bf16", "p16_f16", "p64_f32", "p128_f32"]
UNIT = {"f32": 2.0 ** -24, "f16": 2.0 ** -11, "bf16": 2.0 ** -8}  # unit roundoff


@pytest.mark.parametrize("name", WORKLOADS)
def test_workload_full_size(o, name):
    from paper_2606_01680_amd.workloads import WORKLOADS as W, make_inputs
    w = W[name]
    _say(f"case workload {name} p={w.p} N={w.n} dtype={w.dtype} k={w.k}")
    x = make_inputs(w, device="cuda:0")
    x0 = x.clone()
    pl = o.optcc_plan(w.p, w.bandwidths, w.n, w.k)
    o.optcc_allreduce_emulate(x, w.p, w.n, w.dtype, pl)
    torch.cuda.synchronize()
    iv = int_view(x)
    for r in range(1, w.p):  # every rank holds the same bits
        assert torch.equal(iv[r], iv[0]), r
    rng = np.random.default_rng(1234)
    coords = _sample_coords(pl, w.n, rng)
    idx = torch.from_numpy(coords).to("cuda:0")
    cols = to_host(x0[:, idx], w.dtype).copy()
    sched = oracle.Schedule(w.p, w.bandwidths, w.n, w.k)
    oracle.run_sampled(sched, w.dtype, cols, coords)
    got = to_host(x[:, idx], w.dtype)
    assert bits_equal(got, cols)
    # properties over every coordinate, chunked
    step = max(1 << 16, (1 << 28) // w.p)
    for c0 in range(0, w.n, step):
        c1 = min(w.n, c0 + step)
        if w.dtype == "i32":
            want = x0[:, c0:c1].to(torch.int64).sum(0)
            want = ((want + 2**31) % 2**32 - 2**31).to(torch.int32)
            assert torch.equal(x[0, c0:c1], want)
        else:
            xs = x0[:, c0:c1].to(torch.float64)
            err = (x[0, c0:c1].to(torch.float64) - xs.sum(0)).abs()
            assert bool((err <= w.p * UNIT[w.dtype] * xs.abs().sum(0)).all())
    # and every element of every rank against the oracle's full serial run
    _say(f"case workload {name}: full oracle run")
    full = oracle.run(sched, w.dtype, to_host(x0, w.dtype).copy())
    del x0
    got_all = to_host(x, w.dtype)
    assert bits_equal(got_all, full)


@pytest.mark.parametrize("dtype", ["i32", "f32"])
def test_replanning_between_calls(o, dtype):
    """Re-planning online (Sec. 4.3, schedule generation: closed-form rules,
    cheap enough to run when a failure is detected): a sequence of NIC-loss
    profiles on p=8 (PXN pooling: losing c of 8 NICs leaves bandwidth
    (8-c)/8, Sec. 2), one fresh plan per call on the same buffers, each
    result bit-exact against the oracle."""
    p, n, k = 8, 300000, 16
    seq = [{}, {3: 7 / 8}, {3: 6 / 8, 6: 7 / 8}, {3: 4 / 8}, {3: 2 / 8, 5: 4 / 8, 6: 6 / 8},
           {0: 7 / 8, 1: 7 / 8, 2: 7 / 8, 4: 7 / 8}, {}]
    x = rand_inputs(dtype, p, n, 77)
    d = to_device(x, dtype)
    d0 = d.clone()
    prev = None
    for slow in seq:
        bw = _bw(p, slow)
        _say(f"case replan dtype={dtype} slow={slow}")
        pl = o.optcc_plan(p, bw, n, k)
        d.copy_(d0)
        o.optcc_allreduce_emulate(d, p, n, dtype, pl)
        torch.cuda.synchronize()
        ref = oracle.run(oracle.Schedule(p, bw, n, k), dtype, x.copy())
        assert bits_equal(to_host(d, dtype), ref)
        if prev is not None:
            o.optcc_plan_free(prev)  # the previous plan's device tables go with it
        prev = pl


def test_largest_rank_count(o):
    """p = OPTCC_MAX_EMULATE_RANKS (256): every rank pointer in the kernel
    arguments; one past the limit is rejected before any launch."""
    p, n, k = o.OPTCC_MAX_EMULATE_RANKS, 20000, 8
    for dtype in ("i32", "f32"):
        _say(f"case p=256 dtype={dtype}")
        x, ref, got = _run_both(o, p, {0: 0.5, 100: 0.875, 255: 0.75}, n, k, dtype, seed=256)
        assert bits_equal(got, ref)
    big = o.optcc_plan(p + 1, [1.0] * (p + 1), 128, 4)
    d = torch.zeros((p + 1, 128), dtype=torch.float32, device="cuda:0")
    with pytest.raises(o.OptccError) as e:
        o.optcc_allreduce_emulate(d, p + 1, 128, "f32", big)
    assert e.value.status == o.OPTCC_EUNSUPPORTED


def test_empty_vector(o):
    """N = 0: a valid plan with empty segments; emulation is a no-op."""
    pl = o.optcc_plan(5, [1, 1, 0.5, 1, 1], 0, 8)
    d = torch.zeros((5, 0), dtype=torch.float32, device="cuda:0")
    o.optcc_allreduce_emulate(d, 5, 0, "f32", pl)
    torch.cuda.synchronize()


def test_first_call_inside_capture_is_refused(o):
    """A plan's first call on a device uploads its tables, so it cannot be
    captured: made during a capture it raises OPTCC_EINVAL before touching
    the device, the capture stays valid (the work around it replays), the
    buffers are untouched, and an eager call afterwards gives the oracle's
    result bit for bit."""
    p, n, k = 8, 50000, 8
    bw = _bw(p, {7: 0.875})
    dtype = "f32"
    x = rand_inputs(dtype, p, n, 41)
    ref = oracle.run(oracle.Schedule(p, bw, n, k), dtype, x.copy())
    pl = o.optcc_plan(p, bw, n, k)
    d = to_device(x, dtype)
    d0 = d.clone()
    side = torch.zeros(64, device="cuda:0")
    torch.cuda.synchronize()
    _say("case first call inside a capture")
    g = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            side.add_(1.0)
            with pytest.raises(o.OptccError) as e:
                o.optcc_allreduce_emulate(d, p, n, dtype, pl)
            side.add_(2.0)
    assert e.value.status == o.OPTCC_EINVAL
    assert "captured" in str(e.value)
    torch.cuda.synchronize()
    g.replay()
    torch.cuda.synchronize()
    assert (side == 3.0).all()
    assert torch.equal(int_view(d), int_view(d0))
    del g
    o.optcc_allreduce_emulate(d, p, n, dtype, pl)
    torch.cuda.synchronize()
    assert bits_equal(to_host(d, dtype), ref)


def test_graph_capture_replays(o):
    """After its first call on a device (which uploads the plan tables) an
    AllReduce is one kernel launch, so it can be captured in a HIP graph.
    Each replay, with eager restores and synchronisations in between, equals
    the eager result bit for bit."""
    p, n, k = 8, 200000, 16
    bw = _bw(p, {7: 0.875})
    pl = o.optcc_plan(p, bw, n, k)
    for dtype in ("f32", "bf16", "i32", "f16"):
        x = rand_inputs(dtype, p, n, 31)
        d = to_device(x, dtype)
        d0 = d.clone()
        o.optcc_allreduce_emulate(d, p, n, dtype, pl)  # first use: table upload
        torch.cuda.synchronize()
        eager = d.clone()
        ref = oracle.run(oracle.Schedule(p, bw, n, k), dtype, x.copy())
        assert bits_equal(to_host(eager, dtype), ref)
        g = torch.cuda.CUDAGraph()
        d.copy_(d0)
        torch.cuda.synchronize()
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            with torch.cuda.graph(g, stream=s):
                o.optcc_allreduce_emulate(d, p, n, dtype, pl)
        torch.cuda.synchronize()
        for rep in range(4):
            _say(f"case graph replay dtype={dtype} rep={rep}")
            d.copy_(d0)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(int_view(d), int_view(eager))
        del g


def test_captured_plan_outlives_its_python_reference(o):
    """A plan whose call was captured into a graph stays alive when the
    caller drops it (its device tables are still in the graph): replays
    after garbage collection give the eager result; freeing it explicitly is
    refused until release_captured_plans()."""
    import gc
    p, n, k = 8, 100000, 8
    bw = _bw(p, {7: 0.875})
    dtype = "f32"
    x = rand_inputs(dtype, p, n, 47)
    ref = oracle.run(oracle.Schedule(p, bw, n, k), dtype, x.copy())
    d = to_device(x, dtype)
    d0 = d.clone()
    pl = o.optcc_plan(p, bw, n, k)
    o.optcc_allreduce_emulate(d, p, n, dtype, pl)  # first use: table upload
    torch.cuda.synchronize()
    assert bits_equal(to_host(d, dtype), ref)
    g = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            o.optcc_allreduce_emulate(d, p, n, dtype, pl)
    torch.cuda.synchronize()
    with pytest.raises(RuntimeError):
        o.optcc_plan_free(pl)
    del pl
    gc.collect()
    for rep in range(3):
        _say(f"case captured plan after its reference is dropped rep={rep}")
        d.copy_(d0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert bits_equal(to_host(d, dtype), ref)
    del g
    torch.cuda.synchronize()
    o.release_captured_plans()
    gc.collect()


def test_every_small_length(o):
    """Every length from 0 to 200 and around each tile and quantum boundary up
    to three tiles, for one straggler (bubble filling), several stragglers
    and a server plan: bit for bit against the oracle."""
    lengths = sorted(set(range(0, 201)) | {b + d for b in (1984, 2048, 4096, 6144)
                                           for d in (-65, -64, -63, -1, 0, 1, 63, 64, 65)})
    profiles = [("one", 8, {7: 0.875}, None), ("multi", 9, {0: 0.875, 3: 0.75, 8: 0.5}, None),
                ("servers", 6, None, (3, 2, [1.0, 1.0, 0.5]))]
    for name, p, slow, srv in profiles:
        _say(f"case every small length {name}")
        for n in lengths:
            x = rand_inputs("i32", p, n, 7 + n)
            if srv is None:
                bw = _bw(p, slow)
                pl, sched = o.optcc_plan(p, bw, n, 8), oracle.Schedule(p, bw, n, 8)
            else:
                q, g, sbw = srv
                pl = o.optcc_plan_servers(q, g, sbw, n, 24)
                sched = oracle.Schedule.servers(q, g, sbw, n, 24)
            ref = oracle.run(sched, "i32", x.copy())
            d = to_device(x, "i32")
            o.optcc_allreduce_emulate(d, p, n, "i32", pl)
            torch.cuda.synchronize()
            assert bits_equal(to_host(d, "i32"), ref), (name, n)


def test_more_than_2g_elements_per_rank(o):
    """N = 2^31 + 4099 elements per rank (three ranks, 25.8 GB): element
    offsets beyond 32 bits.  All ranks identical, the exact wrapped int32
    sum everywhere, and sampled coordinates (segment and section ends, the
    last elements) bit for bit against the oracle."""
    p, n, k = 3, (1 << 31) + 4099, 4
    bw = [1.0, 1.0, 0.5]
    _say(f"case p=3 N={n} i32")
    g = torch.Generator(device="cuda:0")
    g.manual_seed(2606)
    x0 = torch.randint(-(1 << 30), 1 << 30, (p, n), generator=g, device="cuda:0", dtype=torch.int32)
    x = x0.clone()
    pl = o.optcc_plan(p, bw, n, k)
    o.optcc_allreduce_emulate(x, p, n, "i32", pl)
    torch.cuda.synchronize()
    for r in range(1, p):
        assert torch.equal(x[r], x[0]), r
    step = 1 << 28
    for c0 in range(0, n, step):
        c1 = min(n, c0 + step)
        want = x0[:, c0:c1].to(torch.int64).sum(0)
        want = ((want + 2**31) % 2**32 - 2**31).to(torch.int32)
        assert torch.equal(x[0, c0:c1], want), c0
    rng = np.random.default_rng(31)
    coords = _sample_coords(pl, n, rng, count=2048)
    coords = np.unique(np.concatenate([coords, np.arange(n - 300, n)]))
    idx = torch.from_numpy(coords).to("cuda:0")
    cols = to_host(x0[:, idx], "i32").copy()
    oracle.run_sampled(oracle.Schedule(p, bw, n, k), "i32", cols, coords)
    assert bits_equal(to_host(x[:, idx], "i32"), cols)


@pytest.mark.parametrize("n", [(1 << 32) - 512, (1 << 32) + 4099])
def test_rank_vectors_at_the_launch_limit(o, n):
    """Six ranks of 2^32 - 512 elements, the longest the chain kernel takes with
    one element per lane, and of 2^32 + 4099, which run the general kernel (96
    GiB of buffers): the exact wrapped int32 sum in every element of every rank,
    inputs made again chunk by chunk."""
    p, k, step = 6, 8, 1 << 28
    if torch.cuda.mem_get_info()[0] < p * n * 4 + (24 << 30):
        pytest.skip("needs 120 GiB of free device memory")
    _say(f"case launch limit p={p} n={n}")

    def chunk(r, c0, c1):
        g = torch.Generator(device="cuda:0")
        g.manual_seed(c0 // step * p + r)
        return torch.randint(-(1 << 31), 1 << 31, (c1 - c0,), generator=g, device="cuda:0",
                             dtype=torch.int32)

    x = torch.empty((p, n), dtype=torch.int32, device="cuda:0")
    spans = [(c0, min(n, c0 + step)) for c0 in range(0, n, step)]
    for c0, c1 in spans:
        for r in range(p):
            x[r, c0:c1] = chunk(r, c0, c1)
    pl = o.optcc_plan(p, _bw(p, {5: 0.75}), n, k)
    o.optcc_allreduce_emulate(x, p, n, "i32", pl)
    torch.cuda.synchronize()
    for c0, c1 in spans:
        want = chunk(0, c0, c1)
        for r in range(1, p):
            want += chunk(r, c0, c1)
        for r in range(p):
            assert torch.equal(x[r, c0:c1], want), (r, c0)
    del x
    torch.cuda.empty_cache()


@pytest.mark.parametrize("dtype", ["f32", "bf16", "i32", "f16"])
def test_fused_ranges_from_the_middle(o, dtype):
    """Any slot range [a, b), fused into one launch and started from the
    state after [0, a) (computed by the oracle), ends in the oracle's state
    after [0, b): the executor's lanes pick up mid-way state from memory
    exactly where the earlier slots left it.  One straggler with bubble
    filling, several stragglers, no straggler, and two server plans (with
    the local ring fixed at compile time, g = 2, and general, g = 3)."""
    n = 2048 * 2 + 64 * 7 + 5
    cases = [("one", 8, _bw(8, {7: 0.875}), None, 8, 6),
             ("multi", 9, _bw(9, {0: 0.875, 3: 0.75, 8: 0.5}), None, 8, 6),
             ("ring", 5, _bw(5, {}), None, 8, 6),
             ("servers g=2", 8, [1.0, 0.5, 1.0, 1.0], (4, 2), 24, 12),
             ("servers g=3", 9, [1.0, 1.0, 0.75], (3, 3), 24, 12)]
    for name, p, bw, srv, k, ns in cases:
        if srv is None:
            pl, sched = o.optcc_plan(p, bw, n, k), oracle.Schedule(p, bw, n, k)
        else:
            pl = o.optcc_plan_servers(srv[0], srv[1], bw, n, k)
            sched = oracle.Schedule.servers(srv[0], srv[1], bw, n, k)
        x = rand_inputs(dtype, p, n, 23 + p)
        for a in range(1, ns):
            start = oracle.run(sched, dtype, x.copy(), 0, a)
            for b in range(a + 1, ns + 1):
                _say(f"case fused range {name} dtype={dtype} [{a},{b})")
                want = oracle.run(sched, dtype, start.copy(), a, b)
                d = to_device(start, dtype)
                o.optcc_allreduce_emulate_slots(d, p, n, dtype, pl, a, b, 1)
                torch.cuda.synchronize()
                assert bits_equal(to_host(d, dtype), want), (name, a, b)


def test_binding_rejects_mismatched_tensors(o):
    """The binding refuses tensors whose element size or length disagrees
    with dtype and N before any pointer reaches the library: the library
    reads and writes N elements of dtype at every rank address and cannot
    see allocation sizes."""
    p, n, k = 5, 1000, 8
    pl = o.optcc_plan(p, [1, 1, 0.5, 1, 1], n, k)
    bf = torch.zeros((p, n), dtype=torch.bfloat16, device="cuda:0")
    with pytest.raises(ValueError, match="element"):
        o.optcc_allreduce_emulate(bf, p, n, "f32", pl)
    with pytest.raises(ValueError, match="element"):
        o.optcc_allreduce_emulate([bf[r] for r in range(p)], p, n, "i32", pl)
    short = [torch.zeros(n - 1, device="cuda:0") for _ in range(p)]
    with pytest.raises(ValueError, match="elements per rank"):
        o.optcc_allreduce_emulate(short, p, n, "f32", pl)
    with pytest.raises(ValueError, match="dtype"):
        o.optcc_allreduce_emulate(torch.zeros((p, n), device="cuda:0"), p, n, "f64", pl)
    torch.cuda.synchronize()


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_narrowing_every_fp32_pattern(o, dtype):
    """The executor's per-step rounding of an fp32 sum to bf16 / fp16 (round
    to nearest even; fp16 subnormals and overflow to infinity), through the
    library's optcc_narrow_f32, equals the oracle's C rule on all 2^32 fp32
    bit patterns.  NaN inputs: bf16 bit for bit (both sides keep the top
    payload bits and quieten), fp16 NaN for NaN (IEEE 754 leaves the payload
    of a narrowed NaN open)."""
    chunk = 1 << 27
    round_ref = oracle.bf16_round if dtype == "bf16" else oracle.f16_round
    out = torch.empty(chunk, dtype=torch.int16, device="cuda:0")
    for c in range((1 << 32) // chunk):
        if c % 8 == 0:
            _say(f"case narrow {dtype} patterns from {c * chunk:#x}")
        bits = np.arange(c * chunk, (c + 1) * chunk, dtype=np.int64).astype(np.uint32)
        x = bits.view(np.float32)
        want = round_ref(x)
        d = torch.from_numpy(x).to("cuda:0")
        o.optcc_narrow_f32(d, out, dtype)
        torch.cuda.synchronize()
        got = out.cpu().numpy().view(np.uint16)
        nan_in = (bits & 0x7fffffff) > 0x7f800000
        if dtype == "bf16":
            assert np.array_equal(got, want), c
        else:
            assert np.array_equal(got[~nan_in], want[~nan_in]), c
            g = got[nan_in]
            assert bool((((g & 0x7c00) == 0x7c00) & ((g & 0x3ff) != 0)).all()), c
    # odd lengths: the last element goes through the single-value form
    bits = np.array([0x7fa00001, 0xffc12345, 0x3f808000, 0x3f818000, 0x00000001,
                     0x7f7fffff, 0xc0490fdb], dtype=np.uint32)
    for n in (1, 3, 7):
        x = bits[:n].view(np.float32)
        want = round_ref(x)
        d = torch.from_numpy(x.copy()).to("cuda:0")
        o.optcc_narrow_f32(d, out[:n], dtype)
        torch.cuda.synchronize()
        got = out[:n].cpu().numpy().view(np.uint16)
        nan_in = (bits[:n] & 0x7fffffff) > 0x7f800000
        if dtype == "bf16":
            assert np.array_equal(got, want), n
        else:
            assert np.array_equal(got[~nan_in], want[~nan_in]), n


def test_threads_share_one_plan(o):
    """A plan is shared read-only across host threads and streams: four
    threads call a fresh plan at once (its device tables are uploaded on
    first use under the plan's lock), each on its own stream and buffers,
    and every result is bit-exact against the oracle."""
    import threading
    p, n, k = 9, 70000, 8
    bw = _bw(p, {0: 0.875, 3: 0.75, 8: 0.5})
    pl = o.optcc_plan(p, bw, n, k)
    dts = ["f32", "bf16", "i32", "f16"]
    xs = {dt: rand_inputs(dt, p, n, 300 + i) for i, dt in enumerate(dts)}
    devs = {dt: to_device(xs[dt], dt) for dt in dts}
    streams = {dt: torch.cuda.Stream() for dt in dts}
    torch.cuda.synchronize()
    errors = []
    start = threading.Barrier(len(dts))

    def work(dt):
        try:
            start.wait()
            for it in range(3):  # repeated calls reuse the uploaded tables
                with torch.cuda.stream(streams[dt]):
                    d = devs[dt]
                    o.optcc_allreduce_emulate(d, p, n, dt, pl, stream=streams[dt])
                    streams[dt].synchronize()
                    if it == 0:
                        first = d.clone()
                    d.copy_(to_device(xs[dt], dt))
                    streams[dt].synchronize()
            devs[dt] = first
        except Exception as e:  # reported by the main thread
            errors.append((dt, e))

    _say("case threads sharing one plan")
    ts = [threading.Thread(target=work, args=(dt,)) for dt in dts]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    sched = oracle.Schedule(p, bw, n, k)
    for dt in dts:
        ref = oracle.run(sched, dt, xs[dt].copy())
        assert bits_equal(to_host(devs[dt], dt), ref), dt


# Long chains on the general kernel (more than 32 healthy ranks, one workgroup
# per CU, tiles of one vector per lane) whose tiles outnumber the per-XCD-run
# limit (2,048; 4,096 below 90 healthy ranks) run as a persistent grid that takes
# tiles from a device counter (work stealing), every element type: slot ranges,
# and whole AllReduces of more than 128 healthy ranks.  Sizes above the limit,
# ragged, two just above it; 2-byte types have half the tiles.
STEAL = [(40, {5: 0.6}, 2048 * 2100 + 77, 8), (70, {3: 0.875}, 2048 * 2200 + 130, 16),
         (36, {}, 2048 * 2300 + 3, 4), (100, {7: 0.5, 60: 0.75}, 1024 * 2049 + 5, 8),
         (64, {63: 0.5, 62: 0.75}, 1024 * 4100 + 5, 16),
         # 98 healthy ranks, 2,101 tiles of 2048 2-byte elements: bf16 and fp16 steal too
         (100, {7: 0.5, 60: 0.75}, 2048 * 2100 + 9, 8),
         (140, {7: 0.5, 60: 0.75}, 1024 * 2049 + 5, 8)]


@pytest.mark.parametrize("p,slow,n,k", STEAL)
def test_work_stealing_launches(o, p, slow, n, k):
    """A work-stealing plan three times in a row (the counters reset
    themselves at the end of each launch), fp32, int32, fp16 and bf16, as two
    slot ranges and as the whole AllReduce: the first result equals the oracle
    on every element, the others equal the first."""
    cuts = () if p > 130 else (5,)
    limit = 1024 * (2048 if p >= 95 else 4096)
    bw = _bw(p, slow)
    pl = o.optcc_plan(p, bw, n, k)
    sched = oracle.Schedule(p, bw, n, k)
    for dtype in ("f32", "i32", "f16", "bf16"):
        _say(f"case work stealing p={p} n={n} k={k} dtype={dtype}")
        x = rand_inputs(dtype, p, n, 90 + p)
        d = to_device(x, dtype)
        d0 = d.clone()
        steal = int(n > limit * (4 // d.element_size()))
        assert steal or d.element_size() == 2
        first = None
        for rep in range(3):
            d.copy_(d0)
            run_slots(o, d, p, n, dtype, pl, cuts, steal=steal)
            torch.cuda.synchronize()
            if first is None:
                first = d.clone()
            else:
                assert torch.equal(int_view(d), int_view(first)), rep
        d.copy_(d0)
        o.optcc_allreduce_emulate(d, p, n, dtype, pl)
        torch.cuda.synchronize()
        assert torch.equal(int_view(d), int_view(first))
        del d, d0
        ref = oracle.run(sched, dtype, x)
        assert bits_equal(to_host(first, dtype), ref), dtype
        del first
        torch.cuda.empty_cache()


def test_work_stealing_equals_static_order(o):
    """Work stealing changes only which workgroup runs which tile: the same
    AllReduce through the no-allocation entry point and inside a captured
    HIP graph (both keep the static tile order) gives the same bits."""
    p, n, k = 140, 1024 * 2300 + 77, 8
    bw = _bw(p, {5: 0.6})
    pl = o.optcc_plan(p, bw, n, k)
    assert call_choice(o, pl, "f32").steal == 1
    c = call_choice(o, pl, "f32", noalloc=True)
    assert c.kernel == "general" and c.steal == 0
    x = rand_inputs("f32", p, n, 4242)
    d0 = to_device(x, "f32")
    d = d0.clone()
    o.optcc_allreduce_emulate(d, p, n, "f32", pl)
    torch.cuda.synchronize()
    steal = d.clone()
    d.copy_(d0)
    o.optcc_allreduce_emulate_noalloc(d, p, n, "f32", pl)
    torch.cuda.synchronize()
    assert torch.equal(int_view(d), int_view(steal))
    g = torch.cuda.CUDAGraph()
    d.copy_(d0)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            o.optcc_allreduce_emulate(d, p, n, "f32", pl)
            captured = call_choice(o, pl, "f32", stream=s.cuda_stream)
    assert captured.kernel == "general" and captured.steal == 0
    torch.cuda.synchronize()
    for rep in range(3):
        _say(f"case work stealing against a captured graph, replay {rep}")
        d.copy_(d0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(int_view(d), int_view(steal)), rep
    del g


def test_work_stealing_slot_ranges(o):
    """A work-stealing plan run as two slot ranges in a row, and as one
    launch per slot (each launch takes the same counter block after the one
    before has set it back to zero), equals the fused call bit for bit, and
    the oracle's stage prefix after the first range."""
    p, n, k = 40, 2048 * 2100 + 77, 8
    bw = _bw(p, {5: 0.6})
    pl = o.optcc_plan(p, bw, n, k)
    x = rand_inputs("f32", p, n, 777)
    d0 = to_device(x, "f32")
    d = d0.clone()
    o.optcc_allreduce_emulate(d, p, n, "f32", pl)
    torch.cuda.synchronize()
    fused = d.clone()
    d.copy_(d0)
    assert call_choice(o, pl, "f32", (0, 2)).steal == 1
    o.optcc_allreduce_emulate_slots(d, p, n, "f32", pl, 0, 2, 1)
    torch.cuda.synchronize()
    ref = oracle.run(oracle.Schedule(p, bw, n, k), "f32", x.copy(), 0, 2)
    assert bits_equal(to_host(d, "f32"), ref)
    o.optcc_allreduce_emulate_slots(d, p, n, "f32", pl, 2, 6, 1)
    torch.cuda.synchronize()
    assert torch.equal(int_view(d), int_view(fused))
    d.copy_(d0)
    o.optcc_allreduce_emulate_slots(d, p, n, "f32", pl, 0, 6, 0)
    torch.cuda.synchronize()
    assert torch.equal(int_view(d), int_view(fused))


def test_work_stealing_threads_share_one_plan(o):
    """Four host threads, each on its own stream and buffers, run one
    work-stealing plan at once, three times each, in two slot ranges: concurrent
    launches take different counter blocks, and every result equals the
    oracle."""
    import threading
    p, n, k = 40, 2048 * 4200 + 77, 8
    bw = _bw(p, {5: 0.6})
    pl = o.optcc_plan(p, bw, n, k)
    names = ["a", "b", "c", "d"]
    dts = {"a": "f32", "b": "i32", "c": "f32", "d": "f16"}
    xs = {nm: rand_inputs(dts[nm], p, n, 500 + i) for i, nm in enumerate(names)}
    devs = {nm: to_device(xs[nm], dts[nm]) for nm in names}
    orig = {nm: devs[nm].clone() for nm in names}
    streams = {nm: torch.cuda.Stream() for nm in names}
    o.optcc_allreduce_emulate(devs["a"].clone(), p, n, "f32", pl)  # tables uploaded first
    torch.cuda.synchronize()
    errors, out = [], {}
    start = threading.Barrier(len(names))

    def work(nm):
        try:
            start.wait()
            with torch.cuda.stream(streams[nm]):
                for it in range(3):
                    d = devs[nm]
                    d.copy_(orig[nm])
                    for b, e in ((0, 2), (2, 6)):
                        o.optcc_allreduce_emulate_slots(d, p, n, dts[nm], pl, b, e, 1,
                                                        stream=streams[nm])
                    if it == 0:
                        out[nm] = d.clone()
                    elif not torch.equal(int_view(d), int_view(out[nm])):
                        errors.append((nm, it, "differs from the first call"))
                streams[nm].synchronize()
        except Exception as e:  # reported by the main thread
            errors.append((nm, e))

    for nm in names:
        assert call_choice(o, pl, dts[nm], (0, 2)).steal == 1
        assert call_choice(o, pl, dts[nm], (2, 6)).steal == 1
    _say("case threads sharing one work-stealing plan")
    ts = [threading.Thread(target=work, args=(nm,)) for nm in names]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    sched = oracle.Schedule(p, bw, n, k)
    for nm in names:
        ref = oracle.run(sched, dts[nm], xs[nm].copy())
        assert bits_equal(to_host(out[nm], dts[nm]), ref), nm


def _random_case(rng):
    """One random plan: ranks, stragglers and their bandwidths (NIC losses of
    eighths or any fraction), N, k, element type; a fifth are server plans."""
    dtype = ["f32", "bf16", "i32", "f16"][int(rng.integers(4))]
    n = int(np.exp(rng.uniform(0.0, np.log(300000))))
    def bandwidth():
        return float(rng.integers(1, 8)) / 8 if rng.random() < 0.5 else float(rng.uniform(0.2, 0.999))
    if rng.random() < 0.2:
        q, g = int(rng.integers(3, 13)), int(rng.integers(2, 10))
        bw = [1.0] * q
        bw[int(rng.integers(q))] = bandwidth()
        return dict(servers=(q, g), p=q * g, bw=bw, n=n, k=8 * int(rng.integers(3, 9)), dtype=dtype)
    p = int(rng.integers(3, 73))
    m = min(int(rng.choice([0, 1, 1, 1, 2, 3, 5])), p - 2)
    bw = [1.0] * p
    for r in rng.choice(p, size=m, replace=False):
        bw[int(r)] = bandwidth()
    return dict(servers=None, p=p, bw=bw, n=n, k=4 * int(rng.integers(1, 17)), dtype=dtype)


def test_random_plans_bit_exact(o):
    """200 seeded random plans of every kind, each bit for bit against the
    oracle on every element of every rank."""
    rng = np.random.default_rng(26060168)
    for i in range(200):
        c = _random_case(rng)
        _say(f"case random #{i}: {c}")
        if c["servers"] is None:
            pl = o.optcc_plan(c["p"], c["bw"], c["n"], c["k"])
            sched = oracle.Schedule(c["p"], c["bw"], c["n"], c["k"])
        else:
            q, g = c["servers"]
            pl = o.optcc_plan_servers(q, g, c["bw"], c["n"], c["k"])
            sched = oracle.Schedule.servers(q, g, c["bw"], c["n"], c["k"])
        x = rand_inputs(c["dtype"], c["p"], c["n"], 1000 + i)
        ref = oracle.run(sched, c["dtype"], x.copy())
        d = to_device(x, c["dtype"])
        o.optcc_allreduce_emulate(d, c["p"], c["n"], c["dtype"], pl)
        torch.cuda.synchronize()
        assert bits_equal(to_host(d, c["dtype"]), ref), i


def _random_rule_case(rng, i):
    """A random plan at the sizes where the launch rules change: short
    chains (3-8 healthy ranks) with 16 MiB to 512 MiB of rank buffers; long
    chains (33-200 ranks) with more tiles than one round of resident workgroups
    of the general kernel; server plans of the same sizes."""
    def bandwidth():
        return float(rng.integers(1, 8)) / 8 if rng.random() < 0.5 else float(rng.uniform(0.2, 0.999))
    kind = ("short", "long", "servers")[i % 3]
    if kind == "servers":
        q, g = int(rng.integers(3, 17)), int(rng.choice([2, 4, 8]))
        bw = [1.0] * q
        bw[int(rng.integers(q))] = bandwidth()
        n = int(rng.integers(1 << 19, (1 << 28) // (q * g)))
        dtype = ["f32", "bf16", "i32"][int(rng.integers(3))]
        return dict(servers=(q, g), p=q * g, bw=bw, n=n, k=8 * int(rng.integers(3, 9)), dtype=dtype)
    if kind == "short":
        p = int(rng.integers(4, 10))
        m = min(int(rng.choice([0, 1, 1, 2])), p - 3)
        n = int(rng.integers((4 << 20) // p, (128 << 20) // p))
        dtype = ["f32", "i32", "f32", "bf16"][int(rng.integers(4))]
    else:
        p = int(rng.integers(33, 201))
        m = int(rng.choice([0, 1, 2, 3]))
        n = int(rng.integers(600_000, (1 << 28) // p))
        dtype = ["f32", "i32", "bf16"][int(rng.integers(3))]
    bw = [1.0] * p
    for r in rng.choice(p, size=m, replace=False):
        bw[int(r)] = bandwidth()
    return dict(servers=None, p=p, bw=bw, n=n, k=4 * int(rng.integers(2, 33)), dtype=dtype)


def test_random_plans_at_rule_sizes(o):
    """18 seeded random plans at mid and large sizes (up to 2^28 elements in
    all), each bit for bit against the oracle's full serial run on every
    element of every rank."""
    rng = np.random.default_rng(1680)
    for i in range(18):
        c = _random_rule_case(rng, i)
        _say(f"case rule-size random #{i}: p={c['p']} n={c['n']} k={c['k']} "
             f"dtype={c['dtype']} servers={c['servers']} bw={sorted(set(c['bw']))}")
        if c["servers"] is None:
            pl = o.optcc_plan(c["p"], c["bw"], c["n"], c["k"])
            sched = oracle.Schedule(c["p"], c["bw"], c["n"], c["k"])
        else:
            q, g = c["servers"]
            pl = o.optcc_plan_servers(q, g, c["bw"], c["n"], c["k"])
            sched = oracle.Schedule.servers(q, g, c["bw"], c["n"], c["k"])
        x = rand_inputs(c["dtype"], c["p"], c["n"], 7000 + i)
        d = to_device(x, c["dtype"])
        o.optcc_allreduce_emulate(d, c["p"], c["n"], c["dtype"], pl)
        torch.cuda.synchronize()
        got = to_host(d, c["dtype"])
        del d
        ref = oracle.run(sched, c["dtype"], x)
        assert bits_equal(got, ref), i
        del x, got, ref
        torch.cuda.empty_cache()


THREE_PER_CU_CASES = [
    # (..., workgroups per CU as a slot range, 0: as many as fit)
    # 6-7 healthy ranks at the 512 MiB edge of the three-workgroups-per-CU
    # launch: just above, just below, and rows aligned to the element only
    ("p=8 at 0.875, fp32, 512 MiB", 8, {7: 0.875}, 1 << 24, "f32", 3),
    ("p=8 at 0.875, fp32, 512 MiB - 128 B", 8, {7: 0.875}, (1 << 24) - 4, "f32", 0),
    ("p=7 at 0.5, int32, 512 MiB + 80 B", 7, {6: 0.5}, 19173964, "i32", 3),
    ("p=9, two stragglers, fp32, odd N", 9, {7: 0.5, 8: 0.5}, (1 << 24) + 1, "f32", 3),
    # bf16 chains of 13-32 healthy ranks (three per CU at any size) and
    # just outside that range
    ("p=14 at 0.5, bf16, 13 healthy", 14, {13: 0.5}, 3 << 20, "bf16", 3),
    ("p=13 at 0.5, bf16, 12 healthy", 13, {12: 0.5}, 3 << 20, "bf16", 0),
    ("p=33 at 0.75, bf16, 32 healthy", 33, {0: 0.75}, (1 << 20) + 8, "bf16", 3),
    ("p=16 at 0.5, bf16, odd N", 16, {15: 0.5}, (1 << 21) + 3, "bf16", 3),
    # fp32/int32 chains of 11-32 healthy ranks from 1 GiB of buffers run one
    # workgroup per CU; 10 healthy ranks and smaller buffers keep two
    ("p=12 at 0.5, fp32, 11 healthy, 1 GiB", 12, {11: 0.5}, 22369624, "f32", 1),
    ("p=11 at 0.5, int32, 10 healthy, 1 GiB", 11, {10: 0.5}, 24403352, "i32", 0),
    ("p=16 at 0.875, fp32, 1 GiB - 256 B", 16, {15: 0.875}, (1 << 24) - 4, "f32", 0),
    ("p=33 at 0.5, int32, 32 healthy, 1 GiB + 7 KiB", 33, {32: 0.5}, 8134464, "i32", 1),
    ("p=16 at 0.5, fp32, odd N, 1 GiB + 64 B", 16, {15: 0.5}, (1 << 24) + 1, "f32", 1),
    ("p=16, three stragglers, fp32, 1 GiB (two per CU)", 16, {0: 0.5, 1: 0.75, 15: 0.875},
     1 << 24, "f32", 0),
    ("p=16 ring, int32, 1 GiB", 16, {}, 1 << 24, "i32", 1),
]


@pytest.mark.parametrize("case", THREE_PER_CU_CASES, ids=[c[0] for c in THREE_PER_CU_CASES])
def test_three_workgroups_per_cu_edges(o, case):
    """Plans on both sides of the launch rules that change the workgroups
    per CU (three: short fp32/int32 chains from 512 MiB of rank buffers and
    bf16 chains of 13-32 healthy ranks; one: fp32/int32 chains of 11-32
    healthy ranks from 1 GiB), as two slot ranges on the general kernel and as
    the whole AllReduce: every element of every rank bit for bit against the
    oracle's full serial run."""
    label, p, strag, n, dtype, per_cu = case
    _say(f"case three-per-CU edge: {label}: p={p} n={n} dtype={dtype}")
    bw = _bw(p, strag)
    pl = o.optcc_plan(p, bw, n, 64)
    x = rand_inputs(dtype, p, n, 4242 + p)
    d = to_device(x, dtype)
    d2 = d.clone()
    run_slots(o, d, p, n, dtype, pl, (5,), per_cu=per_cu)
    o.optcc_allreduce_emulate(d2, p, n, dtype, pl)
    torch.cuda.synchronize()
    assert torch.equal(int_view(d2), int_view(d))
    got = to_host(d, dtype)
    del d, d2
    ref = oracle.run(oracle.Schedule(p, bw, n, 64), dtype, x)
    assert bits_equal(got, ref), label
    del x, got, ref
    torch.cuda.empty_cache()


WIDE_WINDOW_CASES = [
    # (..., 1: 24 hop loads in flight as a slot range, 0: 16)
    # 32-bit chains of more than 32 healthy ranks keep 24 hop loads in flight
    # from 2^23 elements per rank, also on rows aligned to the element only;
    # just below and for bf16 they keep 16
    ("p=34 at 0.5, fp32, 2^23", 34, {33: 0.5}, 1 << 23, "f32", 1),
    ("p=34 at 0.5, int32, 2^23 - 4", 34, {33: 0.5}, (1 << 23) - 4, "i32", 0),
    ("p=40, two stragglers, int32, 2^23 + 4", 40, {38: 0.5, 39: 0.75},
     (1 << 23) + 4, "i32", 1),
    ("p=34 at 0.5, fp32, odd N", 34, {33: 0.5}, (1 << 23) + 1, "f32", 1),
    ("p=64 at 0.875 (P2P chunks), fp32, 2^23", 64, {63: 0.875}, 1 << 23, "f32", 1),
    ("p=34 at 0.5, bf16, 2^23", 34, {33: 0.5}, 1 << 23, "bf16", 0),
]


@pytest.mark.parametrize("case", WIDE_WINDOW_CASES, ids=[c[0] for c in WIDE_WINDOW_CASES])
def test_wide_hop_window_edges(o, case):
    """Long chains on both sides of the launch rule that selects the kernel
    with the deeper hop-load window (32-bit elements, at least 2^23 per
    rank), as two slot ranges and as the whole AllReduce: every element of every
    rank bit for bit against the oracle's full serial run."""
    label, p, strag, n, dtype, wide = case
    _say(f"case wide hop window edge: {label}: p={p} n={n} dtype={dtype}")
    bw = _bw(p, strag)
    pl = o.optcc_plan(p, bw, n, 64)
    x = rand_inputs(dtype, p, n, 2424 + p)
    d = to_device(x, dtype)
    d2 = d.clone()
    run_slots(o, d, p, n, dtype, pl, (5,), wide_window=wide)
    o.optcc_allreduce_emulate(d2, p, n, dtype, pl)
    torch.cuda.synchronize()
    assert torch.equal(int_view(d2), int_view(d))
    got = to_host(d, dtype)
    del d, d2
    ref = oracle.run(oracle.Schedule(p, bw, n, 64), dtype, x)
    assert bits_equal(got, ref), label
    del x, got, ref
    torch.cuda.empty_cache()


def test_random_large_short_chains(o):
    """Four seeded random plans of 6-8 healthy ranks with 480 MiB to 1.9 GiB
    of rank buffers (the range where the general kernel launches 6-7 healthy
    ranks at three workgroups per CU and 8 with two vectors per lane), fp32 and
    int32, one or two stragglers, as two slot ranges and as the whole AllReduce:
    every element of every rank bit for bit against the oracle's full serial
    run."""
    rng = np.random.default_rng(2606)
    for i in range(4):
        p = int(rng.integers(7, 10))
        m = 1 if p < 9 else int(rng.integers(1, 3))
        bw = [1.0] * p
        for r in rng.choice(p, size=m, replace=False):
            bw[int(r)] = float(rng.integers(1, 8)) / 8
        dtype = ("f32", "i32")[i % 2]
        lo, hi = (480 << 20) // (4 * p), (1900 << 20) // (4 * p)
        n = int(rng.integers(lo, hi)) // 4 * 4 + int(rng.integers(0, 4))
        k = 4 * int(rng.integers(4, 33))
        _say(f"case large short chain #{i}: p={p} n={n} k={k} dtype={dtype} bw={sorted(set(bw))}")
        pl = o.optcc_plan(p, bw, n, k)
        x = rand_inputs(dtype, p, n, 9100 + i)
        d = to_device(x, dtype)
        d2 = d.clone()
        run_slots(o, d, p, n, dtype, pl, (5,))
        o.optcc_allreduce_emulate(d2, p, n, dtype, pl)
        torch.cuda.synchronize()
        assert torch.equal(int_view(d2), int_view(d))
        got = to_host(d, dtype)
        del d, d2
        ref = oracle.run(oracle.Schedule(p, bw, n, k), dtype, x)
        assert bits_equal(got, ref), i
        del x, got, ref
        torch.cuda.empty_cache()


def test_one_graph_of_several_allreduces(o):
    """Several AllReduces with different plans and element types (bubble
    filling, several stragglers, a 40-rank chain launched at one workgroup
    per CU, a server plan, fp16) captured in one HIP graph, as a training
    step would capture its gradient buckets.  Every replay, with eager
    restores and synchronisations in between, equals the oracle bit for bit."""
    specs = [("one", 8, _bw(8, {7: 0.875}), None, 60000, 16, "f32"),
             ("multi", 9, _bw(9, {0: 0.875, 3: 0.75, 8: 0.5}), None, 30000, 8, "bf16"),
             ("long", 40, _bw(40, {5: 0.6}), None, 50000, 8, "f32"),
             ("servers", 6, [1.0, 1.0, 0.5], (3, 2), 40000, 24, "i32"),
             ("fp16", 5, _bw(5, {0: 0.5}), None, 20000, 8, "f16")]
    cases = []
    for name, p, bw, srv, n, k, dt in specs:
        if srv is None:
            pl, sched = o.optcc_plan(p, bw, n, k), oracle.Schedule(p, bw, n, k)
        else:
            pl = o.optcc_plan_servers(srv[0], srv[1], bw, n, k)
            sched = oracle.Schedule.servers(srv[0], srv[1], bw, n, k)
        x = rand_inputs(dt, p, n, 500 + p)
        d = to_device(x, dt)
        cases.append((name, p, n, dt, pl, oracle.run(sched, dt, x.copy()), d, d.clone()))
    for name, p, n, dt, pl, ref, d, d0 in cases:  # first use: table upload
        o.optcc_allreduce_emulate(d, p, n, dt, pl)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    for c in cases:
        c[6].copy_(c[7])
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            for name, p, n, dt, pl, ref, d, d0 in cases:
                o.optcc_allreduce_emulate(d, p, n, dt, pl)
    torch.cuda.synchronize()
    for rep in range(3):
        _say(f"case one graph of several AllReduces rep={rep}")
        for c in cases:
            c[6].copy_(c[7])
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for name, p, n, dt, pl, ref, d, d0 in cases:
            assert bits_equal(to_host(d, dt), ref), (name, rep)
    del g


@pytest.mark.parametrize("dtype", ["f32", "bf16", "i32", "f16"])
@pytest.mark.parametrize("p,g,slow", [(5, 1, {4: 0.75}), (40, 1, {0: 0.5, 9: 0.75}), (150, 1, {3: 0.5}),
                                      (9, 3, {1: 0.5}), (25, 5, {0: 0.5}), (16, 4, {3: 0.5}),
                                      (36, 12, {2: 0.5}), (133, 7, {4: 0.5})])
def test_general_kernel_element_aligned(o, dtype, p, g, slow):
    """The general kernel on rows of one [p, n] tensor that are aligned to the
    element only, with every length of the rest past the last whole vector (and
    one shorter than a vector): one launch per slot and, where no chain kernel
    takes it, the whole AllReduce, bit for bit against the oracle."""
    q, k = p // g, 24
    bw = _bw(q, slow)
    for n in [3] + [64 * 37 + r for r in (0, 1, 2, 3, 5, 7)] + [64 * 400 + 62]:
        _say(f"case element aligned dtype={dtype} p={p} g={g} n={n}")
        if g > 1:
            sch, pl = oracle.Schedule.servers(q, g, bw, n, k), o.optcc_plan_servers(q, g, bw, n, k)
        else:
            sch, pl = oracle.Schedule(p, bw, n, k), o.optcc_plan(p, bw, n, k)
        x = rand_inputs(dtype, p, n, 7 * p + n)
        ref = oracle.run(sch, dtype, x.copy())
        d, d2 = to_device(x, dtype), to_device(x, dtype)
        o.optcc_allreduce_emulate_slots(d, p, n, dtype, pl, 0, pl.num_slots, 0)
        o.optcc_allreduce_emulate(d2, p, n, dtype, pl)
        torch.cuda.synchronize()
        assert bits_equal(to_host(d, dtype), ref), n
        assert bits_equal(to_host(d2, dtype), ref), n


@pytest.mark.parametrize("dtype", ["f32", "bf16", "i32", "f16"])
@pytest.mark.parametrize("p,slow,mib", [(6, {5: 0.75}, 79), (6, {5: 0.75}, 81), (40, {0: 0.5}, 79),
                                        (40, {0: 0.5}, 81), (150, {3: 0.5}, 255), (150, {3: 0.5}, 257)])
def test_cache_hints_by_size(o, dtype, p, slow, mib):
    """The general kernel on both sides of the buffer sizes up to which its
    accesses are ordinary ones: the whole AllReduce and one launch per slot give
    the same bits, sampled coordinates those of the oracle."""
    from paper_2606_01680_amd.workloads import make_rank
    es = 4 if dtype in ("f32", "i32") else 2
    n, k = (mib << 20) // (p * es) - 1, 16
    _say(f"case cache hints dtype={dtype} p={p} n={n}")
    bw = _bw(p, slow)
    x = torch.stack([make_rank("uniform_2p20" if dtype == "i32" else "normal", dtype, n, 5 * p + r,
                               "cuda:0") for r in range(p)])
    d = x.clone()
    pl = o.optcc_plan(p, bw, n, k)
    coords = _sample_coords(pl, n, np.random.default_rng(p))
    idx = torch.from_numpy(coords).to("cuda:0")
    cols = to_host(x[:, idx], dtype).copy()
    oracle.run_sampled(oracle.Schedule(p, bw, n, k), dtype, cols, coords)
    o.optcc_allreduce_emulate(x, p, n, dtype, pl)
    o.optcc_allreduce_emulate_slots(d, p, n, dtype, pl, 0, pl.num_slots, 0)
    torch.cuda.synchronize()
    assert torch.equal(int_view(x), int_view(d))
    assert bits_equal(to_host(x[:, idx], dtype), cols)
