"""Row tiles of 257 to 288 rows (up to three of an expert's tiles take 32 rows each of a short last one), at the row counts
where an expert gains or loses a tile: as many tasks as the rule gives, every output against the oracle element by element, and
bit for bit what tiles of 128 rows give."""
import numpy as np
import pytest
import torch

import moe_synth
import oracle
import paper_2604_19241_amd as moe
from helpers import bits, check_elementwise, say, scaled_inputs, to_f64

pytestmark = pytest.mark.gpu
LENGTHS = 8   # word of the workspace's head that the eight list lengths start at


def tiles(rows):
    n = -(-rows // 256)
    short = -(-(rows - 256 * (n - 1)) // 32)
    return n - 1 if n <= 16 and short <= min(3, n - 1) else n


def run(cfg, inp, tile_rows):
    shape = moe.make_shape(**cfg.shape_dict())
    dev = {key: v.cuda() for key, v in inp.items()}
    routing, saved = moe.moe_route(shape, dev["logits"]), moe.alloc_saved(shape, "cuda")
    size = moe.moe_workspace_bytes(shape)
    ws = {key: torch.empty(size[key], dtype=torch.uint8, device="cuda") for key in ("fwd", "bwd")}
    opts = moe.make_opts(tile_rows=tile_rows, spin_limit_ms=500)
    w = [dev[key] for key in ("w_gate", "w_up", "w_down")]
    out = {"y": moe.moe_fused_forward(shape, dev["x"], *w, routing, saved=saved, ws=ws["fwd"], opts=opts)}
    out.update(moe.moe_fused_backward(shape, dev["dy"], dev["x"], *w, routing, saved, ws=ws["bwd"], opts=opts))
    out.update({key: v[:cfg.T] for key, v in moe.saved_views(shape, saved).items()})
    assert moe.moe_device_status(ws["fwd"]) == 0 and moe.moe_device_status(ws["bwd"]) == 0
    return out, [int(ws[key].view(torch.int32)[LENGTHS:LENGTHS + 8].sum()) for key in ("fwd", "bwd")]


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
    got, tasks = run(cfg, inp, 0)
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
