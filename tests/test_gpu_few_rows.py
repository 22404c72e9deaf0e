"""Forward of experts with few rows (their own kernels) beside experts on the work queue, at the
row counts where fragments and paths change, against the oracle."""
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


# k axes of 18, 34 and 66 steps, dealt unevenly to the four waves of a task, more tasks than CUs, and
# widths at which the combine's last round of columns is a full one, 64 columns or none
@pytest.mark.parametrize("rows", [[1], [17, 15]])
@pytest.mark.parametrize("d,I", [(576, 1088), (1024, 64), (1088, 576), (2112, 128), (192, 8256)])
def test_forward_of_a_small_batch(rows, d, I):
    test_forward_at_row_counts(rows, d, I)
