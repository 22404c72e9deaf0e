"""A token's outputs do not depend, bit for bit, on what else is in the batch: experts with few rows run on
kernels of their own, which add every product in the order of the work queue's tiles."""
import numpy as np
import pytest
import torch

import moe_synth
from helpers import say, scaled_inputs
from test_gpu_forward import gpu_forward

pytestmark = pytest.mark.gpu


def run(cfg, inp, n, own, schedule=0):
    """The first n tokens, token t on expert own[t] alone: their G|U, h and o in token order, and y."""
    cfg = moe_synth.small_config(T=n, d=cfg.d, E=cfg.E, k=1, I=cfg.I)
    part = dict(inp, x=inp["x"][:n], logits=torch.from_numpy(np.eye(cfg.E, dtype=np.float32)[own[:n]]))
    y, routing, views = gpu_forward(cfg, part, schedule, 0)
    row = routing.inv_perm.view(-1).long()
    return {"gu": views["gu"][row], "h": views["h"][row], "o": views["o"][row], "y": y}


# few rows (one fragment is 32 rows) against more than 32 of every expert; k axes of one stage and of more
# and fewer than the loads in flight, odd and even; column tiles that are cut off
@pytest.mark.parametrize("rows", [[1], [3, 16, 0, 17], [31, 1], [32, 2, 15, 32, 9]])
@pytest.mark.parametrize("d,I", [(64, 64), (128, 192), (192, 320), (320, 448), (576, 1088), (2048, 768), (2112, 128)])
def test_forward_does_not_depend_on_the_batch(rows, d, I):
    E, n = len(rows), sum(rows)
    rng = np.random.default_rng(n + d)
    own = np.concatenate([rng.permutation(np.repeat(np.arange(E), rows)), np.repeat(np.arange(E), 48)])
    cfg = moe_synth.small_config(T=len(own), d=d, E=E, k=1, I=I)
    inp = scaled_inputs(cfg, 7, 4.0)
    say(f"[batch] rows {rows} d={d} I={I}")
    few, many = run(cfg, inp, n, own), run(cfg, inp, len(own), own)
    for name, got in few.items():
        assert torch.equal(got, many[name][:n]), name
