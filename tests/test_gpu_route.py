"""GPU parity of moe_route: indices, counts and offsets bit-exact against the
oracle; gates to fp32 rounding."""
import ctypes

import numpy as np
import pytest
import torch

import moe_synth
import oracle
from helpers import gpu_routing_as_np, say

pytestmark = pytest.mark.gpu


def run_route(cfg, logits_np):
    import paper_2604_19241_amd as moe
    shape = moe.make_shape(**cfg.shape_dict())
    r = moe.moe_route(shape, torch.from_numpy(logits_np).cuda())
    torch.cuda.synchronize()
    return gpu_routing_as_np(r)


def check(cfg, logits_np, tag):
    say(f"[route] {tag} {cfg.shape_dict()}")
    want = oracle.route(cfg.shape_dict(), logits_np)
    got = run_route(cfg, logits_np)
    for key in ("topk_idx", "counts", "offsets", "perm", "inv_perm"):
        assert np.array_equal(got[key], want[key]), (tag, key)
    assert np.allclose(got["topk_w"], want["topk_w"], rtol=2e-6, atol=1e-7), tag
    return got


CASES = [
    dict(T=256, d=64, E=8, k=2, I=64),
    dict(T=1000, d=64, E=128, k=8, I=64),
    dict(T=777, d=64, E=256, k=8, I=64, e_start=32, e_count=32),
    dict(T=333, d=64, E=64, k=6, I=64),
    dict(T=129, d=64, E=512, k=10, I=64),
    dict(T=65, d=64, E=1024, k=16, I=64, e_start=1000, e_count=24),
    dict(T=50, d=64, E=5, k=5, I=64),
    dict(T=1, d=64, E=3, k=1, I=64),
    dict(T=2049, d=64, E=16, k=4, I=64, e_start=3, e_count=9),
]


@pytest.mark.parametrize("kw", CASES)
def test_route_matches_oracle(kw):
    cfg = moe_synth.small_config(**kw)
    rng = np.random.default_rng(kw["T"] + kw["E"])
    logits = rng.standard_normal((cfg.T, cfg.E)).astype(np.float32)
    check(cfg, logits, "random")


def test_route_ties_and_skew():
    cfg = moe_synth.small_config(T=600, d=64, E=48, k=4, I=64)
    rng = np.random.default_rng(7)
    logits = rng.integers(0, 3, (cfg.T, cfg.E)).astype(np.float32)   # many exact ties
    logits[0] = 1.0                                                   # all equal
    check(cfg, logits, "ties")
    bias = -3.0 * np.log(rng.permutation(cfg.E) + 1.0)
    logits = (rng.standard_normal((cfg.T, cfg.E)) * 0.3 + bias).astype(np.float32)
    got = check(cfg, logits, "skew")
    assert (got["counts"] == 0).any()
    one = np.zeros((cfg.T, cfg.E), np.float32)
    one[:, 17] = 5.0
    check(moe_synth.small_config(T=600, d=64, E=48, k=1, I=64), one, "one-expert")


def test_route_is_bitwise_repeatable():
    cfg = moe_synth.CONFIGS[4]
    inp = moe_synth.make_inputs(cfg, with_weights=False, with_dy=False)
    logits = inp["logits"].numpy()
    say(f"[route] repeat {cfg.name}")
    first = run_route(cfg, logits)
    for _ in range(9):
        again = run_route(cfg, logits)
        for key in first:
            assert np.array_equal(first[key], again[key]), key


@pytest.mark.parametrize("cid", [2, 3, 4])
def test_route_full_size_configs(cid):
    cfg = moe_synth.CONFIGS[cid]
    inp = moe_synth.make_inputs(cfg, with_weights=False, with_dy=False)
    got = check(cfg, inp["logits"].numpy(), cfg.name)
    say(f"[route] {cfg.name} histogram {moe_synth.histogram_summary(got['counts'])}")


def test_route_empty_batch():
    import paper_2604_19241_amd as moe
    shape = moe.make_shape(T=0, d=64, E=8, k=2, I=64)
    r = moe.moe_route(shape, torch.empty((0, 8), dtype=torch.float32, device="cuda"))
    torch.cuda.synchronize()
    assert r.counts.cpu().tolist() == [0] * 8
    assert r.offsets.cpu().tolist() == [0] * 9


@pytest.mark.parametrize("kw", [
    dict(T=300, d=64, E=128, k=8, I=64),
    dict(T=65, d=64, E=1024, k=16, I=64),
    dict(T=129, d=64, E=5, k=5, I=64),
    dict(T=40, d=64, E=7, k=1, I=64),
    dict(T=33, d=64, E=300, k=2, I=64), dict(T=33, d=64, E=65, k=3, I=64), dict(T=33, d=64, E=64, k=4, I=64),
    dict(T=5, d=64, E=129, k=9, I=64),
])
def test_route_backward_matches_oracle(kw):
    """dlogits from the gate gradients: parity with the oracle (fp32 arithmetic on the GPU, the
    gates themselves are fp32: rtol 1e-5), exact zeros for unselected experts."""
    import paper_2604_19241_amd as moe
    cfg = moe_synth.small_config(**kw)
    say(f"[route-bwd] {cfg.shape_dict()}")
    rng = np.random.default_rng(17)
    logits = rng.normal(0, 1.5, (cfg.T, cfg.E)).astype(np.float32)
    g = rng.normal(0, 1, (cfg.T, cfg.k)).astype(np.float32)
    want_r = oracle.route(cfg.shape_dict(), logits)
    want = oracle.route_backward(cfg.shape_dict(), logits, want_r["topk_idx"], g)
    shape = moe.make_shape(**cfg.shape_dict())
    routing = moe.moe_route(shape, torch.from_numpy(logits).cuda())
    got = moe.moe_route_backward(shape, routing, torch.from_numpy(g).cuda())
    torch.cuda.synchronize()
    got = got.cpu().numpy().astype(np.float64)
    assert np.array_equal(routing.topk_idx.cpu().numpy(), want_r["topk_idx"])
    mask = np.zeros((cfg.T, cfg.E), bool)
    np.put_along_axis(mask, want_r["topk_idx"].astype(np.int64), True, axis=1)
    assert (got[~mask] == 0).all()
    assert np.allclose(got, want, rtol=1e-5, atol=2e-7), np.abs(got - want).max()


# T k = 256, 257.. slots: one chunk of whole tokens / two; 64 / 65 chunks (the workgroups add the
# chunks themselves / a scan does); a chunk of more than 256 slots; more chunks than one scan round
@pytest.mark.parametrize("kw", [
    dict(T=32, E=128, k=8), dict(T=33, E=128, k=8), dict(T=2048, E=40, k=8), dict(T=2049, E=40, k=8),
    dict(T=18, E=1024, k=15), dict(T=18 * 65 + 7, E=65, k=15), dict(T=40000, E=24, k=4, e_start=5, e_count=17),
    dict(T=16, E=64, k=16), dict(T=256, E=1, k=1),
])
def test_route_chunk_edges(kw):
    cfg = moe_synth.small_config(d=64, I=64, **kw)
    rng = np.random.default_rng(kw["T"] + kw["k"])
    check(cfg, rng.integers(-4, 5, (cfg.T, cfg.E)).astype(np.float32) * np.float32(0.25), "chunk edge")


# From 1024 chunks of 256 slots on the chunks are longer: the last one short, the last size and the first, chunks of fewer than
# 1024 slots (k = 3, 10), one slot a token, experts here and elsewhere, ties in every token; one token more than one, two and
# three rounds of 256 chunks hold.
@pytest.mark.parametrize("kw", [
    dict(T=32736, E=40, k=8), dict(T=32768, E=200, k=8, e_start=7, e_count=90), dict(T=100003, E=33, k=3), dict(T=262200, E=65, k=1),
    dict(T=27001, E=260, k=10, e_start=250, e_count=10), dict(T=16500, E=600, k=16),
    dict(T=32769, E=40, k=8), dict(T=26113, E=40, k=10), dict(T=65537, E=90, k=8), dict(T=78337, E=40, k=10, e_start=3, e_count=30),
])
def test_route_long_chunks(kw):
    cfg = moe_synth.small_config(d=64, I=64, **kw)
    rng = np.random.default_rng(kw["T"])
    logits = rng.standard_normal((cfg.T, cfg.E), np.float32)
    logits[::3] = np.round(logits[::3] * 4)
    check(cfg, logits, "long chunks")


@pytest.mark.parametrize("T", [20, 500])
def test_route_special_values(T):
    """-inf loses to every number and ties by id, both zeros and equal denormals tie by id, a NaN is
    never selected: the order of a plain float comparison."""
    cfg = moe_synth.small_config(T=T, d=64, E=80, k=6, I=64)
    rng = np.random.default_rng(T)
    pool = np.array([0.0, -0.0, -np.inf, 1e-42, -1e-42, 3e38, -3e38, 1.5, -1.5, np.nan], np.float32)
    logits = pool[rng.integers(0, len(pool), (T, cfg.E))]
    logits[0] = -np.inf
    say(f"[route] special values {cfg.shape_dict()}")
    got = run_route(cfg, logits)
    # stable descending order with NaN behind everything; adding 0 makes the zeros one value
    key = np.where(np.isnan(logits), -np.inf, logits).astype(np.float64) + 0.0
    order = np.lexsort((np.broadcast_to(np.arange(cfg.E), key.shape), -key, np.isnan(logits)), axis=1)
    assert np.array_equal(got["topk_idx"], order[:, :cfg.k])


# Up to 256 experts four tokens share a wave, 16 lanes each with 2, 4, 8 or 16 keys: the first and last number of experts of each,
# one, eight, nine and sixteen selected, tokens that are no multiple of four, logits that are not aligned to 16 bytes.
@pytest.mark.parametrize("E,k", [(1, 1), (3, 2), (16, 4), (17, 16), (32, 8), (33, 8), (64, 9), (65, 16), (128, 8), (128, 1), (129, 8), (129, 9),
                                 (255, 7), (256, 8), (256, 16), (257, 8)])
@pytest.mark.parametrize("T", [3, 67, 301])
def test_route_order_of_special_values(T, E, k):
    import paper_2604_19241_amd as moe
    say(f"[route] special values, {T} tokens, {E} experts, {k} selected")
    rng = np.random.default_rng(1000 * E + k)
    pool = np.array([0.0, -0.0, -np.inf, np.inf, 1e-30, -1e-30, 3e38, -3e38, 1.5, 1.5000001, -1.5, np.nan], np.float32)
    logits = pool[rng.integers(0, len(pool), (T, E))]
    logits[1::3] = rng.standard_normal((len(logits[1::3]), E))
    buffer = torch.empty(T * E + 1, dtype=torch.float32, device="cuda")
    buffer[1:] = torch.from_numpy(logits).cuda().flatten()
    r = moe.moe_route(moe.make_shape(T=T, d=64, E=E, k=k, I=64), buffer[1:].view(T, E))
    value = np.where(np.isnan(logits), -np.inf, logits).astype(np.float64) + 0.0
    order = np.lexsort((np.broadcast_to(np.arange(E), value.shape), -value, np.isnan(logits)), axis=1)[:, :k]
    picked = np.take_along_axis(logits, order, 1)
    assert np.array_equal(r.topk_idx.cpu().numpy(), np.where(np.isnan(picked), 0x7fffffff, order))
    plain = np.isfinite(picked).all(1)
    with np.errstate(over="ignore"):
        p = np.exp((picked[plain] - picked[plain, :1]).astype(np.float64))
    # exp and the quotient in fp32: a few units in the last place
    assert np.allclose(r.topk_w.cpu().numpy()[plain], p / p.sum(1, keepdims=True), rtol=2e-6, atol=1e-7)


# Where the top-k is a launch of its own and where it is not: tokens of one chunk (a wave each, little work,
# more work), fewer than 128, 256 and 512 chunks with little and with more work a chunk
@pytest.mark.parametrize("kw", [
    dict(T=16, E=1024, k=8), dict(T=17, E=300, k=8, e_start=3, e_count=290), dict(T=32, E=50, k=8), dict(T=32, E=51, k=8),
    dict(T=256, E=50, k=1), dict(T=256, E=51, k=1, e_start=50, e_count=1), dict(T=257, E=4, k=1),
    dict(T=33, E=256, k=16), dict(T=33, E=257, k=16), dict(T=127 * 256, E=8, k=1), dict(T=127 * 256 + 1, E=8, k=1),
    dict(T=127 * 256 + 1, E=16, k=1), dict(T=255 * 256 + 1, E=63, k=1), dict(T=255 * 256 + 1, E=64, k=1, e_start=60, e_count=4),
    dict(T=511 * 32 + 1, E=512, k=8), dict(T=510 * 32 + 1, E=512, k=8),
])
def test_route_with_the_topk_apart(kw):
    cfg = moe_synth.small_config(d=64, I=64, **kw)
    rng = np.random.default_rng(kw["T"] + kw["k"])
    check(cfg, rng.integers(-40, 41, (cfg.T, cfg.E)).astype(np.float32) * np.float32(0.25), "top-k apart or not")


def test_route_of_few_slots_is_spread_over_the_chip():
    """One slot a token reads the same logits as eight with an eighth of the rounds: it takes no longer."""
    import paper_2604_19241_amd as moe
    T, E = 8192, 1024
    logits = torch.randn((T, E), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    us = {}
    for k in (1, 8):
        shape = moe.make_shape(T=T, d=64, E=E, k=k, I=64, e_start=0, e_count=E)
        routing = moe.alloc_routing(shape, "cuda")
        start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        times = []
        for _ in range(8):
            start.record()
            for _ in range(20):
                moe.moe_route_static(shape, logits, routing)
            stop.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(stop) * 50.0)
        us[k] = min(times)
    say(f"[route] 8192 tokens of 1024 experts: {us}")
    assert us[1] <= 1.3 * us[8], us


def test_route_backward_of_few_slots_takes_less_than_of_eight():
    """One slot a token writes the same array as eight with an eighth of the comparisons."""
    import paper_2604_19241_amd as moe
    T, E = 32768, 1024
    out = torch.empty((T, E), device="cuda")
    us = {}
    for k in (1, 8):
        shape = moe.make_shape(T=T, d=64, E=E, k=k, I=64, e_start=0, e_count=E)
        routing = moe.moe_route(shape, torch.randn((T, E), generator=torch.Generator(device="cuda").manual_seed(k), device="cuda"))
        g = torch.ones((T, k), device="cuda")
        start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        times = []
        for _ in range(8):
            start.record()
            for _ in range(20):
                moe.moe_route_backward(shape, routing, g, out=out)
            stop.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(stop) * 50.0)
        us[k] = min(times)
    say(f"[route-bwd] 32768 tokens of 1024 experts: {us}")
    assert us[1] <= 0.92 * us[8], us


# One chunk of up to 1024 slots, with up to 320 and more, and the first batch of several; the top-k in its workgroup (64 tokens and 8192 logits)
# and apart, with 16 lanes a token and with 64.
@pytest.mark.parametrize("kw", [
    dict(T=40, E=40, k=8), dict(T=41, E=40, k=8), dict(T=128, E=40, k=8), dict(T=129, E=40, k=8), dict(T=1024, E=7, k=1), dict(T=1025, E=7, k=1),
    dict(T=64, E=128, k=8, e_start=9, e_count=100), dict(T=65, E=128, k=8), dict(T=64, E=129, k=8), dict(T=32, E=256, k=8), dict(T=33, E=256, k=8),
    dict(T=64, E=200, k=16), dict(T=64, E=1024, k=16, e_start=1, e_count=1023), dict(T=102, E=512, k=10), dict(T=103, E=512, k=10),
    dict(T=127 * 128, E=64, k=2), dict(T=127 * 128 + 1, E=64, k=2), dict(T=255 * 128, E=65, k=2), dict(T=255 * 128 + 1, E=65, k=2),
])
def test_route_of_one_chunk(kw):
    cfg = moe_synth.small_config(d=64, I=64, **kw)
    rng = np.random.default_rng(kw["T"] * kw["k"])
    check(cfg, rng.integers(-40, 41, (cfg.T, cfg.E)).astype(np.float32) * np.float32(0.25), "one chunk or several")


# Of 129 to 256 experts a token has 16 lanes or, in batches bound by latency with few selected, a wave: on both sides of the line, by the kernels that are launched.
@pytest.mark.parametrize("T,E,k,select", [
    (1, 256, 1, "Wave"), (8191, 129, 2, "Wave"), (8192, 129, 2, "Row"), (5, 200, 3, "Wave"), (6, 200, 3, "Row"), (2, 256, 4, "Wave"), (3, 256, 4, "Row"),
    (1, 129, 7, "Wave"), (2, 129, 7, "Row"), (1, 256, 8, "Row"), (1, 256, 9, "Wave"), (64, 129, 1, "Wave"), (100, 129, 1, "Wave"), (256, 129, 5, "Row"),
    (4993, 144, 5, "Row"), (4992, 144, 5, "Row"), (1, 128, 1, "Row"), (1, 257, 1, "Wave"), (320, 257, 1, "Wave"), (321, 257, 1, "Wave"), (321, 129, 1, "Wave"), (21, 129, 16, "Wave"), (64, 1024, 16, "Wave"),
])
def test_route_by_lanes_of_a_token(T, E, k, select):
    import paper_2604_19241_amd as moe
    from test_gpu_launches import launches
    shape, p = moe.make_shape(T=T, d=64, E=E, k=k, I=64), ctypes.c_void_p(4096)
    r = moe.binding.MoERoutingC(*[4096] * 6)
    got = launches(lambda st: moe.load_library().moe_route(ctypes.byref(shape), p, ctypes.byref(r), p,
                                                           ctypes.c_size_t(moe.moe_workspace_bytes(shape)["route"]), st))
    assert [n for n in ("Row", "Wave") if any(n + "Select" in name for name, _, _ in got)] == [select], got
    cfg = moe_synth.small_config(T=T, d=64, E=E, k=k, I=64)
    rng = np.random.default_rng(T + E)
    check(cfg, rng.integers(-40, 41, (T, E)).astype(np.float32) * np.float32(0.25), f"{select}Select")


def routing_us(T, E, k):
    import paper_2604_19241_amd as moe
    shape = moe.make_shape(T=T, d=64, E=E, k=k, I=64)
    logits = torch.randn((T, E), generator=torch.Generator(device="cuda").manual_seed(T), device="cuda")
    routing = moe.moe_route(shape, logits)
    ws = torch.empty(moe.moe_workspace_bytes(shape)["route"], dtype=torch.uint8, device="cuda")
    args = [ctypes.byref(shape), logits.data_ptr(), ctypes.byref(routing.c_struct()), ws.data_ptr(), ws.numel(),
            torch.cuda.current_stream().cuda_stream]
    start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    times = []
    for _ in range(8):
        start.record()
        for _ in range(20):
            assert moe.load_library().moe_route(*args) == 0
        stop.record()
        torch.cuda.synchronize()
        times.append(start.elapsed_time(stop) * 50.0)
    say(f"[route] {T} tokens, {E} experts, {k} selected: {min(times):.1f} us")
    return min(times)


def test_route_of_many_experts_fills_a_cu():
    """A ninth row of 64 experts is more work (measured 1.45 times the time), but not one workgroup a CU instead of two (1.83)."""
    assert routing_us(28800, 513, 8) <= 1.65 * routing_us(28800, 512, 8)


# 1100 chunks of 256 slots, 7 % more than 1024: not a second round of long chunks (1.2 to 1.9 times the time)
@pytest.mark.parametrize("T,E,k", [(32768, 256, 8), (16384, 600, 16), (262144, 8, 1)])
def test_routing_just_past_a_round_of_long_chunks(T, E, k):
    assert routing_us(T * 1100 // 1024, E, k) <= 1.15 * routing_us(T, E, k)
