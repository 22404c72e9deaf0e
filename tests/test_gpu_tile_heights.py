"""Row tiles of 257 to 288 rows (up to three of an expert's tiles take 32 rows each of a short last one), at the row counts
where an expert gains or loses a tile: as many tasks as the rule gives, every output against the oracle element by element, and
bit for bit what tiles of 128 rows give."""
import numpy as np
import pytest
import torch

import moe_synth
import oracle
import paper_2604_19241_amd as moe
from helpers import bits, check_elementwise, queue_length, say, scaled_inputs, tiles, to_f64

pytestmark = pytest.mark.gpu


def run(cfg, inp, tile_rows):
    shape = moe.make_shape(**cfg.shape_dict())
    dev = {key: v.cuda() for key, v in inp.items()}
    routing, saved = moe.moe_route(shape, dev["logits"]), moe.alloc_saved(shape, "cuda")
    size = moe.moe_workspace_bytes(shape)
    ws = {key: torch.empty(size[key], dtype=torch.uint8, device="cuda") for key in ("fwd", "bwd")}
    opts = moe.make_opts(tile_rows=tile_rows, workers=2, spin_limit_ms=500)   # (few workers: enough tasks for each)
    w = [dev[key] for key in ("w_gate", "w_up", "w_down")]
    out = {"y": moe.moe_fused_forward(shape, dev["x"], *w, routing, saved=saved, ws=ws["fwd"], opts=opts)}
    out.update(moe.moe_fused_backward(shape, dev["dy"], dev["x"], *w, routing, saved, ws=ws["bwd"], opts=opts))
    out.update({key: v[:cfg.T] for key, v in moe.saved_views(shape, saved).items()})
    assert moe.moe_device_status(ws["fwd"]) == 0 and moe.moe_device_status(ws["bwd"]) == 0
    return out, [queue_length(ws[key]) for key in ("fwd", "bwd")]


# one fragment more and one row past it, one tile and several; two and three fragments more; the most tiles that take rows;
# columns that are cut off and k axes of one, two, three and more stages
@pytest.mark.parametrize("counts", [[257, 288, 289, 256], [512, 513, 544, 545], [576, 577, 609, 800, 864, 865], [4064, 4097]])
@pytest.mark.parametrize("d,I", [(64, 64), (128, 192), (320, 448)])
def test_higher_tiles(counts, d, I):
    E, T = len(counts), sum(counts)
    cfg = moe_synth.small_config(T=T, d=d, E=E, k=1, I=I)
    inp = scaled_inputs(cfg, 9, 4.0)
    own = np.random.default_rng(T).permutation(np.repeat(np.arange(E), counts))
    inp["logits"] = torch.from_numpy(np.eye(E, dtype=np.float32)[own])
    say(f"[heights] rows {counts} d={d} I={I}")
    got, tasks = run(cfg, inp, 256)
    n, of = sum(tiles(c) for c in counts), lambda v, size: -(-v // size)
    wgrad = E * (of(I, 256) * of(d, 256) + of(d, 256) * of(I, 128))
    assert tasks == [n * (of(I, 128) + of(d, 256)), n * (of(I, 256) + of(d, 256)) + wgrad]
    want, _ = run(cfg, inp, 128)
    for key, v in got.items():
        assert torch.equal(v, want[key]), key
    b = bits(inp, ("x", "dy", "w_gate", "w_up", "w_down"))
    r = oracle.route(cfg.shape_dict(), inp["logits"].numpy())
    ref = oracle.backward(cfg.shape_dict(), b["x"], b["dy"], b["w_gate"], b["w_up"], b["w_down"], r, round_bf16=True, acc="f32")
    ref["y"] = oracle.forward(cfg.shape_dict(), b["x"], b["w_gate"], b["w_up"], b["w_down"], r)["y"]
    for key in ("y", "dx", "dw_gate", "dw_up", "dw_down"):
        check_elementwise(key, to_f64(got[key]), ref[key])
    check_elementwise("dtopk_w", to_f64(got["dtopk_w"]), ref["dtopk_w"], whole_array_rms=True)


# Tiles of 128 rows by the sizes: below two tasks a worker forward and one and a half backward, none where the GEMMs have
# a few stages; two flags a scoreboard slot, at row counts around a slot's edges
@pytest.mark.parametrize("d,I,workers,low", [(320, 448, 0, (True, True)), (320, 448, 30, (False, False)), (320, 448, 40, (False, True)),
                                             (64, 64, 0, (False, False))])
def test_low_tiles_by_the_sizes(d, I, workers, low):
    counts = [127, 128, 129, 255, 256, 257, 384, 385, 512, 513, 1, 0, 700]
    E, T = len(counts), sum(counts)
    cfg = moe_synth.small_config(T=T, d=d, E=E, k=1, I=I)
    inp = scaled_inputs(cfg, 3, 4.0)
    own = np.random.default_rng(T).permutation(np.repeat(np.arange(E), counts))
    inp["logits"] = torch.from_numpy(np.eye(E, dtype=np.float32)[own])
    say(f"[heights] d={d} I={I} workers={workers}")
    shape = moe.make_shape(**cfg.shape_dict())
    dev = {key: v.cuda() for key, v in inp.items()}
    routing = moe.moe_route(shape, dev["logits"])
    size = moe.moe_workspace_bytes(shape)
    w = [dev[key] for key in ("w_gate", "w_up", "w_down")]
    of = lambda v, size: -(-v // size)
    wgrad = E * (of(I, 256) * of(d, 256) + of(d, 256) * of(I, 128))
    got = {}
    for tile_rows in (0, 256, 128):
        saved = moe.alloc_saved(shape, "cuda")
        ws = {key: torch.empty(size[key], dtype=torch.uint8, device="cuda") for key in ("fwd", "bwd")}
        opts = moe.make_opts(tile_rows=tile_rows, workers=workers, spin_limit_ms=500)
        got[tile_rows] = {"y": moe.moe_fused_forward(shape, dev["x"], *w, routing, saved=saved, ws=ws["fwd"], opts=opts)}
        got[tile_rows].update(moe.moe_fused_backward(shape, dev["dy"], dev["x"], *w, routing, saved, ws=ws["bwd"], opts=opts))
        assert moe.moe_device_status(ws["fwd"]) == 0 and moe.moe_device_status(ws["bwd"]) == 0
        if tile_rows == 0:
            tasks = [queue_length(ws[key]) for key in ("fwd", "bwd")]
    n = [sum(of(c, 128) if l else of(c, 256) for c in counts) for l in low]
    few = sum(1 for c in counts if 0 < c <= 32)   # ahead of the queue or on it: as the plan's own rule says
    assert tasks[0] in (n[0] * (of(I, 128) + of(d, 256)), (n[0] - few) * (of(I, 128) + of(d, 256)))
    assert tasks[1] == n[1] * (of(I, 256) + of(d, 256)) + wgrad
    for tile_rows in (256, 128):
        for key, v in got[tile_rows].items():
            assert torch.equal(v, got[0][key]), (tile_rows, key)


# A share of the experts: the rows that it has choose the tiles, not those that even routing would give it.  Even routing of 4000
# tokens over 64 experts would make low tiles right for 4 of them, of 20000 over 8 tall ones.
@pytest.mark.parametrize("T,E,rows,workers,height", [(4000, 64, 900, 16, 256), (20000, 8, 150, 64, 128)])
def test_tiles_follow_the_rows_of_a_share(T, E, rows, workers, height):
    n, d, I = 4, 320, 448
    cfg = moe_synth.small_config(T=T, d=d, E=E, k=1, I=I, e_start=2, e_count=n)
    inp = scaled_inputs(cfg, 5, 4.0)
    there = [e for e in range(E) if not 2 <= e < 2 + n]
    own = np.concatenate([np.repeat(np.arange(2, 2 + n), rows), np.resize(there, T - n * rows)])
    inp["logits"] = torch.from_numpy(np.eye(E, dtype=np.float32)[np.random.default_rng(T).permutation(own)])
    say(f"[heights] share of {n} of {E}, {rows} rows each, {T} tokens")
    shape = moe.make_shape(**cfg.shape_dict())
    dev = {key: v.cuda() for key, v in inp.items()}
    routing = moe.moe_route(shape, dev["logits"])
    assert routing.counts.tolist() == [rows] * n
    size = moe.moe_workspace_bytes(shape)
    w = [dev[key] for key in ("w_gate", "w_up", "w_down")]
    of = lambda v, size: -(-v // size)
    wgrad = n * (of(I, 256) * of(d, 256) + of(d, 256) * of(I, 128))
    got = {}
    for tile_rows in (0, 384 - height):
        saved = moe.alloc_saved(shape, "cuda")
        ws = {key: torch.empty(size[key], dtype=torch.uint8, device="cuda") for key in ("fwd", "bwd")}
        opts = moe.make_opts(tile_rows=tile_rows, workers=workers, spin_limit_ms=500)
        got[tile_rows] = {"y": moe.moe_fused_forward(shape, dev["x"], *w, routing, saved=saved, ws=ws["fwd"], opts=opts)}
        got[tile_rows].update(moe.moe_fused_backward(shape, dev["dy"], dev["x"], *w, routing, saved, ws=ws["bwd"], opts=opts))
        assert moe.moe_device_status(ws["fwd"]) == 0 and moe.moe_device_status(ws["bwd"]) == 0
        tasks = [queue_length(ws[key]) for key in ("fwd", "bwd")]
        tiles_of = n * of(rows, tile_rows or height)
        assert tasks == [tiles_of * (of(I, 128) + of(d, 256)), tiles_of * (of(I, 256) + of(d, 256)) + wgrad], tile_rows
    for key, v in got[0].items():
        assert torch.equal(v, got[384 - height][key]), key
