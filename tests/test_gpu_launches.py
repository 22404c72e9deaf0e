"""What the entry points launch, read from a captured (and never executed) graph: the grids of every kernel."""
import ctypes

import pytest
import torch

import paper_2604_19241_amd as moe
from helpers import say

pytestmark = pytest.mark.gpu


class Dim3(ctypes.Structure):
    _fields_ = [(n, ctypes.c_uint32) for n in "xyz"]


class KernelNodeParams(ctypes.Structure):
    _fields_ = [("block", Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", Dim3),
                ("params", ctypes.c_void_p), ("shared", ctypes.c_uint32)]


def hip():
    with open("/proc/self/maps") as f:
        lib = ctypes.CDLL(next(line.split()[-1] for line in f if "libamdhip64" in line))
    lib.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    lib.hipKernelNameRefByPtr.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
    return lib


def launches(call):
    """[(kernel name, workgroups, threads a workgroup)] of call(stream), in order."""
    lib = hip()
    stream = torch.cuda.Stream()
    st, graph = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p()
    torch.cuda.synchronize()
    assert lib.hipStreamBeginCapture(st, 2) == 0   # relaxed
    rc = call(st)
    ended = lib.hipStreamEndCapture(st, ctypes.byref(graph))
    assert rc == moe.binding.MOE_OK, rc
    assert ended == 0
    n = ctypes.c_size_t()
    assert lib.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert lib.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
    out = []
    for node in nodes:
        p = KernelNodeParams()
        assert lib.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
        name = (lib.hipKernelNameRefByPtr(p.func, st) or b"?").decode()
        out.append((name, p.grid.x * p.grid.y * p.grid.z, p.block.x * p.block.y * p.block.z))
    assert lib.hipGraphDestroy(graph) == 0
    return out


# Any aligned address will do for a call whose kernels never run.
def forward_launches(shape, opts):
    p, lib = ctypes.c_void_p(4096), moe.load_library()
    r = moe.binding.MoERoutingC(*([4096] * 6))
    return launches(lambda st: lib.moe_fused_forward(
        ctypes.byref(shape), p, p, p, p, ctypes.byref(r), p, None, p, ctypes.c_size_t(moe.moe_workspace_bytes(shape)["fwd"]),
        ctypes.byref(opts), st))


def first_call():
    """What the library looks up once per device cannot be looked up during a capture."""
    shape = moe.make_shape(T=40, d=64, E=2, k=1, I=64)
    dev = {"device": "cuda"}
    x, w = torch.zeros((40, 64), dtype=torch.bfloat16, **dev), torch.zeros((2, 64, 64), dtype=torch.bfloat16, **dev)
    r = moe.moe_route(shape, torch.zeros((40, 2), **dev))
    saved = moe.alloc_saved(shape, "cuda")
    moe.moe_fused_forward(shape, x, w, w, w, r, saved=saved)
    moe.moe_fused_backward(shape, x, x, w, w, w, r, saved)
    torch.cuda.synchronize()


@pytest.mark.parametrize("T", [20, 600])
@pytest.mark.parametrize("workers", [1, 5, 0])
def test_workers_bounds_every_launch_of_the_forward_gemms(T, workers):
    first_call()
    shape = moe.make_shape(T=T, d=1024, E=128, k=8, I=768)
    got = forward_launches(shape, moe.make_opts(workers=workers))
    say(f"[launches] T={T} workers={workers}: {got}")
    gemms = [(name, groups) for name, groups, threads in got if "tail" not in name]
    plan = 32 if T > 32 else 0   # workgroups of the first launch that write the queue
    groups = [n - (plan if i == 0 else 0) for i, (_, n) in enumerate(gemms)]
    assert len(groups) == (3 if plan else 2)
    if workers:
        assert max(groups) <= workers, gemms
    else:
        assert min(groups) >= 128, gemms


# Experts of 33 to 64 rows leave the queue in layers of more than 128 experts alone: elsewhere the launches have no code for them.
@pytest.mark.parametrize("experts,two", [(128, False), (129, True)])
def test_launches_for_few_rows_have_no_more_code_than_they_may_run(experts, two):
    first_call()
    got = forward_launches(moe.make_shape(T=300, d=256, E=160, k=4, I=128, e_count=experts), moe.make_opts())
    say(f"[launches] {experts} experts: {got}")
    names = [name for name, _, _ in got if "first" in name or "second" in name]
    assert len(names) == 2 and all(("ILb1E" in name or "<true>" in name) == two for name in names), names


def every_launch_fits(got):
    say(f"[launches] {got}")
    assert all(0 < groups and groups * threads < 2 ** 32 for _, groups, threads in got), got


# 2^32 work-items a launch are too many: one wave for each of these tokens and rounds of columns would be
@pytest.mark.parametrize("T,d", [(2 ** 25, 1088), (2 ** 26, 64), (2 ** 27 - 16, 64)])
def test_long_batches_of_narrow_tokens_can_be_launched(T, d):
    first_call()
    shape = moe.make_shape(T=T, d=d, E=2, k=1, I=64)
    every_launch_fits(forward_launches(shape, moe.make_opts()))
    p, lib = ctypes.c_void_p(4096), moe.load_library()
    r = moe.binding.MoERoutingC(*([4096] * 6))
    for gates in (p, None):
        every_launch_fits(launches(lambda st: lib.moe_fused_backward(
            ctypes.byref(shape), p, p, p, p, p, ctypes.byref(r), p, p, p, p, p, gates, p,
            ctypes.c_size_t(moe.moe_workspace_bytes(shape)["bwd"]), None, st)))


# more than the 2^24 waves of one launch: two for dX with the gates and one combine, three and two
@pytest.mark.parametrize("T,d", [(2 ** 23 + 5, 64), (2 ** 24 + 37, 64)])
def test_tail_kernels_of_several_launches(T, d):
    g = torch.Generator(device="cuda").manual_seed(d)
    I, E = 64, 2
    x, dy = (torch.randn((T, d), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    w = [torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16) * 0.05 for s in ((E, d, I), (E, d, I), (E, I, d))]
    logits = torch.randn((T, E), generator=g, device="cuda")

    def both(sel):
        n = len(x[sel])
        shape = moe.make_shape(T=n, d=d, E=E, k=1, I=I)
        r, saved = moe.moe_route(shape, logits[sel]), moe.alloc_saved(shape, "cuda")
        y = moe.moe_fused_forward(shape, x[sel], *w, r, saved=saved)
        out = moe.moe_fused_backward(shape, dy[sel], x[sel], *w, r, saved)
        return {"y": y, "dx": out["dx"], "dtopk_w": out["dtopk_w"]}

    say(f"[tail] T={T} d={d}")
    whole = both(slice(0, T))
    # a token's rows do not depend on the batch: the same tokens in pieces that one round of waves covers
    step = 2 ** 22
    for t in list(range(0, T, step)):
        sel = slice(t, min(T, t + step))
        for name, want in both(sel).items():
            assert torch.equal(whole[name][sel], want), (name, t)
