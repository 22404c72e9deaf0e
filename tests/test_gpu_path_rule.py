"""Which experts with few rows run ahead of the work queue: the same bits either way, no launch without work where the
sizes rule it out, and no time lost where the queue has room for them."""
import numpy as np
import pytest
import torch

import paper_2604_19241_amd as moe
from helpers import say
from test_gpu_launches import first_call, forward_launches

pytestmark = pytest.mark.gpu
ROW_TILES = 1   # word of the workspace's head: row tiles of the queue


def batch(counts, d, I, seed=3, extra=0):
    """One token a row, in random order, then `extra` more of every expert: (shape, x, w, routing, own)."""
    E = len(counts)
    rng = np.random.default_rng(seed)
    own = np.concatenate([rng.permutation(np.repeat(np.arange(E), counts)), np.repeat(np.arange(E), extra)])
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(shape, std):
        return (torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16) * std).contiguous()

    w = [normal((E, d, I), 0.05), normal((E, d, I), 0.05), normal((E, I, d), 0.05)]
    x = normal((int(sum(counts)) + 33 * E, d), 1.0)[:len(own)].contiguous()
    shape = moe.make_shape(T=len(own), d=d, E=E, k=1, I=I)
    logits = torch.zeros((len(own), E), device="cuda")
    logits[torch.arange(len(own)), torch.from_numpy(own).cuda()] = 1.0
    return shape, x, w, moe.moe_route(shape, logits)


def forward(shape, x, w, routing):
    ws = torch.empty(moe.moe_workspace_bytes(shape)["fwd"], dtype=torch.uint8, device="cuda")
    saved = moe.alloc_saved(shape, "cuda")
    y = moe.moe_fused_forward(shape, x, *w, routing, saved=saved, ws=ws)
    assert moe.moe_device_status(ws) == 0
    row = routing.inv_perm.view(-1).long()
    return dict({k: v[row] for k, v in moe.saved_views(shape, saved).items()}, y=y), int(ws.view(torch.int32)[ROW_TILES])


# 128 experts of 2048 x 768, `few` with 1 to 32 rows and `many` with more: on the queue up to 8 times as many, ahead of it
# beyond; ahead of it with fewer where the many have 512 rows each; the smallest numbers at which the time spared
# exceeds the time taken; none with many rows.
@pytest.mark.parametrize("few,many,rows,ahead", [
    (0, 8, 40, False), (1, 8, 40, False), (63, 8, 40, False), (64, 8, 40, True), (120, 8, 40, True), (100, 28, 33, False),
    (79, 10, 40, False), (79, 10, 520, True), (1, 10, 520, False), (94, 1, 33, False), (95, 1, 33, True), (127, 1, 33, True),
    (128, 0, 0, True), (3, 0, 0, True),
])
def test_the_same_bits_on_both_paths(few, many, rows, ahead):
    E, d, I = 128, 2048, 768
    rng = np.random.default_rng(few)
    counts = np.zeros(E, np.int64)
    at = rng.permutation(E)
    counts[at[:few]] = rng.integers(1, 33, few)
    counts[at[:min(few, 3)]] = (32, 17, 1)[:min(few, 3)]
    counts[at[few:few + many]] = rows
    n = int(counts.sum())
    say(f"[path] few={few} many={many} rows={rows}")
    got, tiles = forward(*batch(counts, d, I))
    queued = counts[counts > (32 if ahead else 0)]
    assert tiles == int((-(-queued // 256)).sum()), tiles
    # the same tokens with 33 more of every expert: all on the queue
    want, tiles = forward(*batch(counts, d, I, extra=33))
    assert tiles == int((-(-(counts + 33) // 256)).sum())
    for name, v in got.items():
        assert torch.equal(v, want[name][:n]), name


# 256 experts of 2304 x 1024, none with more than 64 rows: all of them ahead of the queue where the estimate says that it is faster (192 with up to 32
# rows and 64 with more 645 us, on the queue 675 us), all on it where it is not (76 and 128 557 us, ahead of it 596 us), and the last and first numbers on its two sides.
@pytest.mark.parametrize("few,medium,ahead", [(192, 64, True), (120, 136, True), (119, 137, False), (76, 128, False)])
def test_up_to_64_rows_leave_the_queue_where_that_is_faster(few, medium, ahead):
    E, d, I = 256, 2304, 1024
    rng = np.random.default_rng(medium)
    counts = np.zeros(E, np.int64)
    at = rng.permutation(E)
    counts[at[:few]] = rng.integers(1, 33, few)
    counts[at[few:few + medium]] = rng.integers(33, 65, medium)
    n = int(counts.sum())
    say(f"[path] few={few} medium={medium}")
    got, tiles = forward(*batch(counts, d, I))
    assert tiles == (0 if ahead else few + medium), tiles
    want, tiles = forward(*batch(counts, d, I, extra=33))   # on the queue, by their own rows
    assert tiles == E
    for name, v in got.items():
        assert torch.equal(v, want[name][:n]), name


# 128 of 136 experts, `many` of them with so many rows and the others with 10: the rows that are here decide, not the tokens (24000
# of them, of which even routing would send 22588 here).
@pytest.mark.parametrize("many,rows,ahead", [(38, 50, False), (20, 200, False), (30, 560, True)])
def test_a_share_is_judged_by_its_rows(many, rows, ahead):
    T, E, ec, d, I = 24000, 136, 128, 2048, 768
    counts = np.full(ec, 10)
    counts[:many] = rows
    own = np.concatenate([np.repeat(np.arange(ec), counts), np.resize(np.arange(ec, E), T - counts.sum())])
    own = torch.from_numpy(np.random.default_rng(many).permutation(own)).cuda()
    shape = moe.make_shape(T=T, d=d, E=E, k=1, I=I, e_count=ec)
    logits = torch.zeros((T, E), device="cuda")
    logits[torch.arange(T), own] = 1.0
    g = torch.Generator(device="cuda").manual_seed(many)
    x, *w = [torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16) * 0.05 for s in ((T, d), (ec, d, I), (ec, d, I), (ec, I, d))]
    say(f"[path] share: {many} with {rows}")
    ws = torch.empty(moe.moe_workspace_bytes(shape)["fwd"], dtype=torch.uint8, device="cuda")
    y = moe.moe_fused_forward(shape, x, *w, moe.moe_route(shape, logits), ws=ws)
    assert moe.moe_device_status(ws) == 0
    queued = counts[counts > (32 if ahead else 0)]
    assert int(ws.view(torch.int32)[ROW_TILES]) == int((-(-queued // 256)).sum())
    # the same rows as a layer of their own
    here = own < ec
    whole = moe.make_shape(T=int(here.sum()), d=d, E=ec, k=1, I=I)
    want = moe.moe_fused_forward(whole, x[here].contiguous(), *w, moe.moe_route(whole, logits[here][:, :ec].contiguous()))
    assert torch.equal(y[here], want) and (y[~here] == 0).all()


def test_no_launch_for_few_rows_where_the_sizes_rule_it_out():
    first_call()
    # more rows than 32 for each of all experts, or than 128 where only some are here
    for shape in (moe.make_shape(T=256, d=512, E=8, k=2, I=1024), moe.make_shape(T=520, d=512, E=8, k=2, I=1024, e_start=4, e_count=4)):
        got = forward_launches(shape, moe.make_opts())
        say(f"[path] {got}")
        assert got[0][1] == 32 and len(got) == 3   # plan, queue, combine
    # up to 32 rows an expert on average, or experts elsewhere: there may be no expert with more rows
    for shape in (moe.make_shape(T=128, d=512, E=8, k=2, I=1024), moe.make_shape(T=256, d=512, E=8, k=2, I=1024, e_start=0, e_count=4)):
        got = forward_launches(shape, moe.make_opts())
        assert len(got) == 4 and got[0][1] > 32, got


def test_few_rows_beside_many_take_no_longer_than_many():
    """13 experts with 16 rows beside 3 with 300 are less work than with 48 rows."""
    us = {}
    for rows in (16, 48):
        shape, x, w, routing = batch([300, 300, 300] + [rows] * 13, 2048, 1408)
        y = torch.empty_like(x)
        ws = torch.empty(moe.moe_workspace_bytes(shape)["fwd"], dtype=torch.uint8, device="cuda")
        start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        times = []
        for _ in range(8):
            start.record()
            for _ in range(20):
                moe.moe_fused_forward(shape, x, *w, routing, y=y, ws=ws)
            stop.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(stop) * 50.0)
        us[rows] = min(times)
    say(f"[path] {us}")
    assert us[16] <= 1.1 * us[48], us


def test_a_captured_call_follows_the_counts_of_each_replay():
    """The choice is the device's: one graph, replayed on batches that take either path and a mix of both."""
    T, d, I, E = 3000, 1024, 1024, 128
    shape = moe.make_shape(T=T, d=d, E=E, k=1, I=I)
    g = torch.Generator(device="cuda").manual_seed(4)
    x = torch.randn((T, d), generator=g, device="cuda", dtype=torch.bfloat16)
    w = [torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16) * 0.05 for s in ((E, d, I), (E, d, I), (E, I, d))]
    token = torch.arange(T, device="cuda")
    batches = {"few": token % 128, "many": token % 60, "some": torch.where(token < 1000, token % 120, 120 + token % 8)}
    logits, y = torch.zeros((T, E), device="cuda"), torch.empty_like(x)
    routing = moe.alloc_routing(shape, "cuda")
    ws = torch.empty(moe.moe_workspace_bytes(shape)["fwd"], dtype=torch.uint8, device="cuda")

    def step():
        moe.moe_route_static(shape, logits, routing)
        moe.moe_fused_forward(shape, x, *w, routing, y=y, ws=ws)

    def load(name):
        logits.zero_()
        logits[token, batches[name]] = 1.0

    want, tiles = {}, {}
    for name in batches:
        load(name)
        step()
        want[name], tiles[name] = y.clone(), int(ws.view(torch.int32)[ROW_TILES])
    assert tiles == {"few": 0, "many": 60, "some": 8}, tiles
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for name in ("many", "few", "some", "few", "many", "some"):
        load(name)
        y.fill_(7.0)
        graph.replay()
        torch.cuda.synchronize()
        say(f"[path] replay {name}")
        assert int(ws.view(torch.int32)[ROW_TILES]) == tiles[name]
        assert torch.equal(y, want[name]), name
