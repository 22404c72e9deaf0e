"""Forward of experts with few rows (their own kernels, or the work queue beside experts with more), at the
row counts where fragments and paths change, against the oracle."""
import re
from pathlib import Path

import numpy as np
import pytest
import torch

import moe_synth
import oracle
from helpers import bits, check_elementwise, rel_l2, say, scaled_inputs, to_f64
from test_gpu_forward import REL_L2, gpu_forward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [
    [1], [16, 0, 16], [17, 15], [31, 1], [32],                       # no expert can have more than 32: no queue
    [33], [0, 1, 15, 16, 17, 31, 32, 33, 0, 48, 2], [63, 64, 65, 66], [300, 3, 129, 20, 1, 64, 7, 1, 2],
])
@pytest.mark.parametrize("d,I", [(64, 64), (320, 192), (192, 448)])
def test_forward_at_row_counts(rows, d, I):
    T, E = sum(rows), len(rows)
    cfg = moe_synth.small_config(T=T, d=d, E=E, k=1, I=I)
    inp = scaled_inputs(cfg, 5, 4.0)
    own = np.random.default_rng(T).permutation(np.repeat(np.arange(E), rows))
    inp["logits"] = torch.from_numpy(np.eye(E, dtype=np.float32)[own])
    b = bits(inp, ("x", "w_gate", "w_up", "w_down"))
    r = oracle.route(cfg.shape_dict(), inp["logits"].numpy())
    assert r["counts"].tolist() == rows
    want = oracle.forward(cfg.shape_dict(), b["x"], b["w_gate"], b["w_up"], b["w_down"], r, round_bf16=True, stages=True)
    for schedule in (0, 1, 2):
        say(f"[few rows] {rows} d={d} I={I} schedule={schedule}")
        y, _, views = gpu_forward(cfg, inp, schedule, 0)
        gu = to_f64(views["gu"])
        for name, got in (("y", to_f64(y)), ("G", gu[:, :I]), ("U", gu[:, I:]), ("h", to_f64(views["h"])), ("o", to_f64(views["o"]))):
            assert rel_l2(got, want[name]) <= REL_L2, name
            check_elementwise(name, got, want[name])


# k axes of 9, 16, 17, 33 and 129 stages of 64, and widths at which the combine's last round of columns is a
# full one, 64 columns or none
@pytest.mark.parametrize("rows", [[1], [17, 15]])
@pytest.mark.parametrize("d,I", [(576, 1088), (1024, 64), (1088, 576), (2112, 128), (192, 8256)])
def test_forward_of_a_small_batch(rows, d, I):
    test_forward_at_row_counts(rows, d, I)


# A generation step: no stash (h and o in the workspace, no G|U), several slots a token, an expert window; up to
# 32 tokens without a queue, 33 with one.  The stash changes where the stages are kept and nothing else.
@pytest.mark.parametrize("T", [1, 20, 32, 33])
@pytest.mark.parametrize("kw", [dict(E=16, k=8, e_start=5, e_count=9), dict(E=16, k=12), dict(E=4, k=4)])
def test_generation_step_without_a_stash(T, kw):
    cfg = moe_synth.small_config(T=T, d=320, I=192, **kw)
    inp = scaled_inputs(cfg, 9, 4.0)
    b = bits(inp, ("x", "w_gate", "w_up", "w_down"))
    r = oracle.route(cfg.shape_dict(), inp["logits"].numpy())
    want = oracle.forward(cfg.shape_dict(), b["x"], b["w_gate"], b["w_up"], b["w_down"], r)["y"]
    for schedule in (0, 1, 2):
        say(f"[no stash] {cfg.shape_dict()} schedule={schedule}")
        y, _, _ = gpu_forward(cfg, inp, schedule, 0, with_saved=False)
        assert rel_l2(to_f64(y), want) <= REL_L2
        check_elementwise("y", to_f64(y), want)
        assert torch.equal(y, gpu_forward(cfg, inp, schedule, 0)[0])


def widths(rows, d, I):
    """Weight columns of a task of GEMM1 and GEMM2 on 256 CUs, by the weights that the source gives the rounds."""
    text = (Path(__file__).resolve().parents[1] / "paper_2604_19241_amd" / "csrc" / "thin.hpp").read_text()
    cost = {int(c): int(w) for c, w in re.findall(r"= cost\((\d+), (\d+)\)", text)}
    assert sorted(cost) == [64, 128, 256]
    n = sum(1 for r in rows if r)
    return tuple(min((-(-n * -(-columns // c) // 256) * cost[c], -c) for c in cost)[1] * -1 for columns in (2 * I, d))


# More tasks than the 512 workgroups: a workgroup's images are used for one task after the other
@pytest.mark.parametrize("rows,I", [([2] * 16, 8256), ([1, 0, 3] * 5, 8256)])
def test_workgroups_with_several_tasks(rows, I):
    assert sum(1 for r in rows if r) * -(-2 * I // widths(rows, 64, I)[0]) > 600
    test_forward_at_row_counts(rows, 64, I)


# Tasks of 256, 128 and 64 weight columns (as many experts as make each the choice on 256 CUs), the last one of an expert cut off
# and not, in both GEMMs; k axes shorter than the stages on their way
@pytest.mark.parametrize("E,d,I,of", [(128, 448, 256, (256, 256)), (85, 512, 320, (256, 128)), (86, 64, 384, (256, 64)), (200, 576, 320, (128, 128)),
                                      (230, 128, 64, (128, 128)), (20, 320, 192, (64, 64)), (23, 128, 448, (64, 64))])
def test_widths_of_a_task(E, d, I, of):
    rows = np.random.default_rng(E).integers(0, 4, E)
    rows[:4] = (32, 31, 17, 0)
    assert widths(rows, d, I) == of
    test_forward_at_row_counts(rows.tolist(), d, I)


# Up to 64 rows, where no expert has more and 129 have some: tasks of two blocks of rows beside tasks of one, their last columns cut off
# and not, with few and with many of either, more of them than workgroups.  Against the same tokens beside an expert of 65 rows, with which
# the experts of 33 to 64 are on the work queue: the same bits.
@pytest.mark.parametrize("rows,d,I", [([33] + [1] * 128, 64, 64), ([64, 32, 1, 63] + [2] * 130, 320, 192), ([40] * 7 + [9] * 122, 1088, 576),
                                      ([33, 0, 47] + [3] * 200, 576, 320), ([1] * 140 + [50, 64], 64, 384), ([60] * 130, 192, 1088),
                                      ([33, 64] * 150 + [1, 32] * 100, 128, 448)])
def test_two_blocks_of_rows(rows, d, I):
    import paper_2604_19241_amd as moe
    E, T = len(rows) + 1, sum(rows) + 65
    cfg = moe_synth.small_config(T=T, d=d, E=E, k=1, I=I)
    dev = {key: v.cuda() for key, v in scaled_inputs(cfg, 17, 4.0).items()}
    own = torch.from_numpy(np.random.default_rng(T).permutation(np.repeat(np.arange(E - 1), rows))).cuda()
    got = {}
    for more in (0, 1):
        t, e = sum(rows) + 65 * more, E - 1 + more
        say(f"[two blocks] {rows[:8]}.. d={d} I={I} queue={more}")
        shape = moe.make_shape(T=t, d=d, E=e, k=1, I=I)
        to = torch.cat([own, torch.full((t - len(own),), E - 1, device="cuda")])
        routing = moe.moe_route(shape, torch.nn.functional.one_hot(to, e).float())
        assert routing.counts.tolist() == rows + [65] * more
        saved = moe.alloc_saved(shape, "cuda")
        ws = torch.empty(moe.moe_workspace_bytes(shape)["fwd"], dtype=torch.uint8, device="cuda")
        y = moe.moe_fused_forward(shape, dev["x"][:t], dev["w_gate"][:e], dev["w_up"][:e], dev["w_down"][:e], routing, saved=saved, ws=ws)
        assert moe.moe_device_status(ws) == 0
        assert (int(ws.view(torch.int32)[1]) > 0) == (more > 0)   # row tiles of the queue
        got[more] = dict(moe.saved_views(shape, saved), y=y)
    for name, v in got[0].items():
        assert torch.equal(v, got[1][name][:len(v)]), name
    # and a plain product in fp32: h and o within the roundings to bf16 of x W and of h
    x, r = dev["x"][:len(own)].float(), torch.argsort(own, stable=True)
    for e in sorted(set(own.tolist())):
        at = own[r] == e
        xe = x[r][at]
        g, u = xe @ dev["w_gate"][e].float(), xe @ dev["w_up"][e].float()
        h = torch.nn.functional.silu(g) * u
        assert rel_l2(to_f64(got[0]["h"][:len(own)][at]), h.double().cpu().numpy()) <= REL_L2
        o = got[0]["h"][:len(own)][at].float() @ dev["w_down"][e].float()
        assert rel_l2(to_f64(got[0]["o"][:len(own)][at]), o.double().cpu().numpy()) <= REL_L2


# The same for some of the experts, several of them a token and no stash: 150 of 200 are here, from the 18th on.
def test_two_blocks_of_rows_in_a_share():
    import paper_2604_19241_amd as moe
    T, d, I, E, k, e_start, ec = 2667, 192, 128, 200, 3, 17, 150
    dev = {key: v.cuda() for key, v in scaled_inputs(moe_synth.small_config(T=T + 70, d=d, E=E, k=k, I=I, e_start=e_start, e_count=ec), 23, 4.0).items()}
    logits = torch.rand((T + 70, E), generator=torch.Generator().manual_seed(1)).cuda()
    logits[T:, e_start + 5] = 2.0   # 70 more tokens for one expert: past 64 rows, with which all are on the work queue
    got = {}
    for n in (T, T + 70):
        shape = moe.make_shape(T=n, d=d, E=E, k=k, I=I, e_start=e_start, e_count=ec)
        routing = moe.moe_route(shape, logits[:n])
        most, medium = int(routing.counts.max()), int((routing.counts > 32).sum())
        say(f"[two blocks] share, {n} tokens, up to {most} rows, {medium} experts with more than 32")
        assert (most <= 64) == (n == T) and medium > 100
        saved = moe.alloc_saved(shape, "cuda")
        for stash in (None, saved):
            ws = torch.empty(moe.moe_workspace_bytes(shape)["fwd"], dtype=torch.uint8, device="cuda")
            y = moe.moe_fused_forward(shape, dev["x"][:n], dev["w_gate"], dev["w_up"], dev["w_down"], routing, saved=stash, ws=ws)
            assert moe.moe_device_status(ws) == 0
            assert (int(ws.view(torch.int32)[1]) > 0) == (n > T)   # row tiles of the queue
            got[n, stash is None] = y
    assert torch.equal(got[T, True], got[T, False])
    assert torch.equal(got[T, False], got[T + 70, False][:T]) and torch.equal(got[T + 70, True], got[T + 70, False])


def us_of_one_row_each(experts, d, I, E=16):
    """The layer for one token on each of so many experts, other ones from call to call."""
    import paper_2604_19241_amd as moe
    g = torch.Generator(device="cuda").manual_seed(1)
    w = [torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16) for s in ((E, d, I), (E, d, I), (E, I, d))]
    shape = moe.make_shape(T=experts, d=d, E=E, k=1, I=I)
    x = torch.randn((experts, d), generator=g, device="cuda", dtype=torch.bfloat16)
    y, ws = torch.empty_like(x), torch.empty(moe.moe_workspace_bytes(shape)["fwd"], dtype=torch.uint8, device="cuda")
    routings = []
    for first in range(E):
        logits = torch.zeros((experts, E), device="cuda")
        logits[torch.arange(experts), (first + torch.arange(experts)) % E] = 1.0
        routings.append(moe.moe_route(shape, logits))
    start, stop = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    times = []
    for _ in range(8):
        start.record()
        for r in routings:
            moe.moe_fused_forward(shape, x, *w, r, y=y, ws=ws)
        stop.record()
        torch.cuda.synchronize()
        times.append(start.elapsed_time(stop) * 1e3 / E)
    return min(times)


def test_fewer_experts_take_no_longer():
    """4 experts have tasks of 64 gate and up columns, 5 of 128: halves of a memory line are not fetched twice for that."""
    us = {n: us_of_one_row_each(n, 7168, 2048) for n in (4, 5)}
    say(f"[few rows] {us}")
    assert us[4] <= us[5], us


# A caller may bring a routing in which a token's slots share an expert: more than 32 rows of an expert in a batch
# of up to 32 tokens are run in blocks of 32.  Against the same slots as tokens of their own, whose experts are on
# the work queue: the rows have the same bits.
@pytest.mark.parametrize("T,k", [(32, 2), (20, 5), (11, 3)])
def test_slots_of_a_token_on_one_expert(T, k):
    import paper_2604_19241_amd as moe
    d, I, E = 320, 192, 6
    F = T * k
    rng = np.random.default_rng(F)
    own = np.where(rng.random(F) < (0.9 if F > 40 else 1.0), 4, rng.integers(0, E, F)).astype(np.int32)   # slot f -> expert
    perm = np.argsort(own, kind="stable").astype(np.int32)
    inv = np.empty(F, np.int32)
    inv[perm] = np.arange(F, dtype=np.int32)
    counts = np.bincount(own, minlength=E).astype(np.int32)
    assert counts.max() > 32
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    cfg = moe_synth.small_config(T=T, d=d, E=E, k=k, I=I)
    dev = {key: v.cuda() for key, v in scaled_inputs(cfg, 13, 4.0).items()}
    got = {}
    for tokens, slots in ((T, k), (F, 1)):
        say(f"[one expert] {tokens} tokens, {slots} slots, rows {counts.tolist()}")
        shape = moe.make_shape(T=tokens, d=d, E=E, k=slots, I=I)
        routing = moe.alloc_routing(shape, "cuda")
        for name, v in (("topk_idx", own), ("counts", counts), ("offsets", offsets), ("perm", perm), ("inv_perm", inv)):
            dst = getattr(routing, name)
            dst.copy_(torch.from_numpy(v).view(dst.shape))
        routing.topk_w.fill_(1.0)
        x = dev["x"] if slots == k else dev["x"].repeat_interleave(k, dim=0)
        saved = moe.alloc_saved(shape, "cuda")
        y = moe.moe_fused_forward(shape, x, dev["w_gate"], dev["w_up"], dev["w_down"], routing, saved=saved)
        got[slots] = dict(moe.saved_views(shape, saved), y=y)
    for name in ("gu", "h", "o"):
        assert torch.equal(got[k][name], got[1][name]), name
    # gates of one: y is the sum of the token's rows in slot order, in fp32
    o = got[k]["o"][torch.from_numpy(inv).cuda().long()].float().view(T, k, d)
    want = torch.zeros((T, d), device="cuda")
    for j in range(k):
        want += o[:, j]
    assert torch.equal(got[k]["y"], want.bfloat16())
