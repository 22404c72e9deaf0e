"""Every entry point works on the stream that is current when it is called, behind what that stream has to do first."""
import pytest
import torch

import paper_2604_19241_amd as moe
from helpers import say

pytestmark = pytest.mark.gpu


def test_calls_follow_the_current_stream():
    T, d, E, k, I = 700, 128, 16, 4, 192
    g = torch.Generator(device="cuda").manual_seed(2)

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)

    inputs = {"logits": torch.randn((T, E), generator=g, device="cuda"), "x": normal(T, d), "dy": normal(T, d)}
    w = [normal(E, d, I) * 0.05, normal(E, d, I) * 0.05, normal(E, I, d) * 0.05]
    shape = moe.make_shape(T=T, d=d, E=E, k=k, I=I)
    buf = {name: torch.zeros_like(v) for name, v in inputs.items()}
    dst, src = torch.zeros(4096, dtype=torch.uint8, device="cuda"), torch.zeros(4096, dtype=torch.uint8, device="cuda")

    def run():
        for name, v in inputs.items():
            buf[name].copy_(v)
        src.fill_(3)
        static = moe.moe_route_static(shape, buf["logits"], moe.alloc_routing(shape, "cuda"))
        routing = moe.moe_route(shape, buf["logits"])
        saved = moe.alloc_saved(shape, "cuda")
        ws = torch.empty(moe.moe_workspace_bytes(shape)["fwd"], dtype=torch.uint8, device="cuda")
        y = moe.moe_fused_forward(shape, buf["x"], *w, routing, saved=saved, ws=ws)
        grads = moe.moe_fused_backward(shape, buf["dy"], buf["x"], *w, routing, saved)
        dlogits = moe.moe_route_backward(shape, routing, grads["dtopk_w"])
        send = moe.moe_global_map(shape, 2, 1, routing, torch.stack([routing.counts] * 2))
        moe.moe_calibration_copy(dst, src)
        assert moe.moe_device_status(ws) == 0
        return [static.perm, static.topk_w, routing.perm, y, *grads.values(), dlogits, send.dst_row, send.recv_offsets, dst]

    want = [v.clone() for v in run()]
    torch.cuda.synchronize()
    for v in (*buf.values(), src, dst):
        v.zero_()
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    say("[streams] behind a delay on a stream of its own")
    with torch.cuda.stream(stream):
        torch.cuda._sleep(40_000_000)   # the inputs are not there before that is over
        got = run()
    stream.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(got, want))
