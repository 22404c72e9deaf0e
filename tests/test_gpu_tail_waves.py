"""The tail kernel of the backward pass, whose waves are (token, round of 1024 columns) or (token, gate
gradients), at widths where the last round is full, 64 columns or the only one, with and without gates."""
import pytest
import torch

import moe_synth
from helpers import scaled_inputs
from test_gpu_backward import KEYS, check_backward, gpu_fwd_bwd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,k", [(1, 1024, 1), (3, 1088, 2), (5, 2112, 9), (37, 64, 8)])
def test_tail_waves(T, d, k):
    cfg = moe_synth.small_config(T=T, d=d, E=16, k=k, I=128)
    inp = scaled_inputs(cfg, 3, 4.0)
    check_backward(cfg, seed=3, schedule=0, tile_rows=0, wscale=4.0)
    inside, _ = gpu_fwd_bwd(cfg, inp, 1, 0)      # the tail as tasks of the persistent kernel: a wave a token
    with_gates, _ = gpu_fwd_bwd(cfg, inp, 0, 0)
    without, _ = gpu_fwd_bwd(cfg, inp, 0, 0, want_dtopk_w=False)
    for key in ("dx", "dtopk_w"):
        assert torch.equal(with_gates[key], inside[key]), key
    assert without["dtopk_w"] is None
    for key in KEYS:
        if key != "dtopk_w":
            assert torch.equal(with_gates[key], without[key]), key
