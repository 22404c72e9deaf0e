"""The work queue's plan: the lists that the experts are dealt to carry equal work."""
import numpy as np
import pytest
import torch

import moe_synth
import paper_2604_19241_amd as moe
from helpers import say

pytestmark = pytest.mark.gpu
LISTS = 8
LENGTHS = 8   # word of the workspace's head that the eight list lengths start at


# One expert of 256 with most of the rows, 31 or 32 with `rows` each, the others with none.  The experts with rows are
# two of every 16 ids: dealt by id among those without, boustrophedon, they would all come to one list.
@pytest.mark.parametrize("rows", [33, 48, 200])
@pytest.mark.parametrize("pair", [(0, 15), (3, 12), (7, 8)])
@pytest.mark.parametrize("most", [40, 8192, 20000])
def test_lists_have_equal_length(rows, pair, most):
    E, d, I = 256, 64, 64
    counts = np.zeros(E, np.int64)
    few = np.isin(np.arange(E) % 16, pair)
    few[0] = False
    counts[few] = rows
    counts[0] = most
    own = np.repeat(np.arange(E), counts)
    cfg = moe_synth.small_config(T=len(own), d=d, E=E, k=1, I=I)
    shape = moe.make_shape(**cfg.shape_dict())
    logits = torch.zeros((cfg.T, E), device="cuda")
    logits[torch.arange(cfg.T), torch.from_numpy(own).cuda()] = 1.0
    x = torch.randn((cfg.T, d), device="cuda").bfloat16()
    w = [torch.zeros(s, dtype=torch.bfloat16, device="cuda") for s in ((E, d, I), (E, d, I), (E, I, d))]
    routing, saved = moe.moe_route(shape, logits), moe.alloc_saved(shape, "cuda")
    size = moe.moe_workspace_bytes(shape)
    ws = {key: torch.empty(size[key], dtype=torch.uint8, device="cuda") for key in ("fwd", "bwd")}
    moe.moe_fused_forward(shape, x, *w, routing, saved=saved, ws=ws["fwd"])
    moe.moe_fused_backward(shape, x, x, *w, routing, saved, ws=ws["bwd"])
    tiles = lambda n: -(-n // 256)
    # tasks of an expert with rows: a tile of each GEMM; the weight gradients of every expert have two more
    for key, small, large, extra in (("fwd", 2 * tiles(rows), 2 * tiles(most), 0), ("bwd", 2 * tiles(rows), 2 * tiles(most), 2)):
        got = sorted(ws[key].view(torch.int32)[LENGTHS:LENGTHS + LISTS].tolist())
        say(f"[plan] {key} rows={rows} most={most} ids={pair}: {got}")
        assert sum(got) == few.sum() * small + large + E * extra
        # one list has the large expert beside its share; the others differ by no more than an expert or two
        others = got[:-1] if large > 2 * small else got
        assert others[-1] - others[0] <= 2 * small + extra, (key, got)
