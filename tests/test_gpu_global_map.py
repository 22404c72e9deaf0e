"""GPU parity of moe_global_map (Algorithm 1 with W > 1 ranks, the part one GPU
runs): W ranks' token batches are routed one after the other on the one GPU,
their histograms stacked (standing in for the AllGather), and every rank's
destination arrays must equal the multi-rank oracle bit for bit."""
import numpy as np
import pytest
import torch

import moe_synth
import oracle
from oracle import global_map as gm
from helpers import say

pytestmark = pytest.mark.gpu

KEYS = ("dst_rank", "dst_expert", "dst_off", "dst_row", "send", "n_dst_ranks")


def run_case(W, E, k, toks, seed, zipf_s=0.0):
    import paper_2604_19241_amd as moe
    say(f"[global map] W={W} E={E} k={k} tokens per rank={toks} zipf={zipf_s}")
    rng = np.random.default_rng(seed)
    bias = -zipf_s * np.log(rng.permutation(E) + 1.0) if zipf_s > 0 else np.zeros(E)
    routings, sels, shapes = [], [], []
    for r in range(W):
        cfg = moe_synth.small_config(T=toks[r], d=64, E=E, k=k, I=64)
        logits = (rng.standard_normal((cfg.T, E)) + bias).astype(np.float32)
        shape = moe.make_shape(**cfg.shape_dict())
        routings.append(moe.moe_route(shape, torch.from_numpy(logits).cuda()))
        shapes.append(shape)
        sels.append(oracle.route(cfg.shape_dict(), logits)["topk_idx"])
        assert np.array_equal(routings[-1].topk_idx.cpu().numpy(), sels[-1])
    want = gm.global_map(sels, E)
    c_all = torch.stack([r.counts for r in routings]).contiguous()     # the AllGather's result
    assert np.array_equal(c_all.cpu().numpy(), want["c_all"])
    for r in range(W):
        got = moe.moe_global_map(shapes[r], W, r, routings[r], c_all)
        torch.cuda.synchronize()
        for key in KEYS:
            assert np.array_equal(getattr(got, key).cpu().numpy(), want["ranks"][r][key]), (r, key)
        assert np.array_equal(got.recv_offsets.cpu().numpy(), want["recv_offsets"][r]), r
    return want


@pytest.mark.parametrize("W,E,k,toks", [
    (8, 128, 8, [300, 512, 0, 700, 256, 1, 333, 640]),   # ragged batches, one rank without tokens
    (2, 8, 2, [1000, 37]),
    (4, 1024, 16, [130, 64, 200, 99]),                   # the shape limits
    (1, 16, 4, [500]),                                   # one rank: the local stable sort itself
    (64, 64, 6, [40] * 64),                              # one expert per rank, the rank limit
    (8, 512, 10, [257] * 8),
])
def test_global_map_matches_oracle(W, E, k, toks):
    run_case(W, E, k, toks, seed=7 * W + E)


# 4096 counts of all ranks, which every workgroup reads for itself, and more, which one does for all; tokens that fill workgroups of 1024
# slots, one more and one less, and a rank without any.
@pytest.mark.parametrize("W,E,k,toks", [(4, 1024, 4, [256, 257, 255, 0]), (8, 1024, 4, [512, 1, 0, 513, 511, 2, 3, 4]), (16, 272, 16, [64, 65, 63, 0] * 4)])
def test_global_map_with_and_without_a_launch_for_the_bases(W, E, k, toks):
    run_case(W, E, k, toks, seed=W + E)


# 512 workgroups of 1024 slots run at a time: with one token more the bases have a launch of their own, and the workgroups 256 slots.
@pytest.mark.parametrize("E,k,T,one", [(8, 8, 65536, True), (8, 8, 65537, False), (16, 10, 52224, True), (16, 10, 52225, False), (8, 2, 0, False)])
def test_global_map_of_more_workgroups_than_run_at_a_time(E, k, T, one):
    import ctypes
    import paper_2604_19241_amd as moe
    from test_gpu_launches import launches
    shape = moe.make_shape(T=T, d=64, E=E, k=k, I=64)
    routing, mapping, p = moe.binding.MoERoutingC(*[4096] * 6), moe.binding.MoEGlobalMapC(*[4096] * 7), ctypes.c_void_p(4096)
    got = launches(lambda st: moe.load_library().moe_global_map(ctypes.byref(shape), 2, 1, ctypes.byref(routing), p, ctypes.byref(mapping), p,
                                                                ctypes.c_size_t(8 * E), st))
    say(f"[global map] {T} tokens: {got}")
    assert [threads for _, _, threads in got] == ([1024] if one else [1024, 256] if T else [1024])
    if T:
        run_case(2, E, k, [300, T], seed=T)


def test_global_map_skewed_routing_and_statistics():
    """Zipf-biased routing; also the distinct-destination count of uniform top-8 over 8 ranks,
    which for distinct experts (16 per rank) averages 8 (1 - C(112,8)/C(128,8)) = 5.34."""
    run_case(8, 128, 8, [400] * 8, seed=3, zipf_s=1.2)
    want = run_case(8, 128, 8, [2000] * 8, seed=4)
    x = np.concatenate([r["n_dst_ranks"] for r in want["ranks"]])
    from math import comb
    assert abs(x.mean() - 8 * (1 - comb(112, 8) / comb(128, 8))) < 0.03


def test_global_map_is_bitwise_repeatable():
    import paper_2604_19241_amd as moe
    cfg = moe_synth.small_config(T=3000, d=64, E=128, k=8, I=64)
    rng = np.random.default_rng(11)
    logits = torch.from_numpy(rng.standard_normal((cfg.T, cfg.E)).astype(np.float32)).cuda()
    shape = moe.make_shape(**cfg.shape_dict())
    r = moe.moe_route(shape, logits)
    c_all = torch.stack([r.counts] * 8).contiguous()
    first = moe.moe_global_map(shape, 8, 5, r, c_all)
    for _ in range(5):
        again = moe.moe_global_map(shape, 8, 5, r, c_all)
        for key in KEYS + ("recv_offsets",):
            assert torch.equal(getattr(first, key), getattr(again, key)), key


@pytest.mark.parametrize("W,E,k", [(2, 16, 4), (8, 128, 8), (64, 64, 1)])
def test_global_map_of_tokens_without_enough_numbers(W, E, k):
    """A NaN is never selected: the slots that are left over go nowhere, the others where they do without them."""
    import paper_2604_19241_amd as moe
    T, rank = 300, W - 1
    rng = np.random.default_rng(E)
    logits = rng.standard_normal((T, E)).astype(np.float32)
    few = np.arange(0, T, 3)
    for t in few:
        logits[t, rng.permutation(E)[:E - t % k]] = np.nan   # t % k numbers left, none in some
    cfg = moe_synth.small_config(T=T, d=64, E=E, k=k, I=64)
    shape = moe.make_shape(**cfg.shape_dict())
    say(f"[global map] NaN logits {cfg.shape_dict()} W={W}")
    r = moe.moe_route(shape, torch.from_numpy(logits).cuda())
    c_all = torch.stack([r.counts] * W).contiguous()
    got = moe.moe_global_map(shape, W, rank, r, c_all)
    idx, n_epr, counts = r.topk_idx.cpu().numpy(), E // W, r.counts.cpu().numpy().astype(np.int64)
    there = idx < E
    assert there.sum() == counts.sum() and (~there).sum() == sum(k - t % k for t in few)
    e = np.where(there, idx, 0)
    off = r.inv_perm.cpu().numpy() - (np.cumsum(counts) - counts)[e] + rank * counts[e]
    total = (W * counts).reshape(W, n_epr)
    start = (np.cumsum(total, axis=1) - total).reshape(E)
    dst = np.where(there, e // n_epr, -1)
    first = there & ~np.array([[(dst[t, :j] == dst[t, j]).any() for j in range(k)] for t in range(T)])
    want = {"dst_rank": dst, "dst_expert": np.where(there, e % n_epr, -1), "dst_off": np.where(there, off, -1),
            "dst_row": np.where(there, start[e] + off, -1), "send": first, "n_dst_ranks": first.sum(axis=1)}
    for key in KEYS:
        assert np.array_equal(getattr(got, key).cpu().numpy(), want[key]), key
