"""The workloads that the speed of the fused MoE layer is followed on.

A case is one pass through the public entry points as a user's program makes it, with the
buffers such a program keeps (workspaces, stash, output and routing arrays):

  decode   moe_route_static into routing arrays kept from step to step, then moe_fused_forward
           without a stash: one layer of a generation step over `T` running sequences;
  prefill  moe_route, then moe_fused_forward without a stash: one layer over the tokens of a prompt;
  train    moe_route, moe_fused_forward with its stash, moe_fused_backward (gradients of x, of the
           three weights and of the gates), moe_route_backward: one layer of a training step, the
           weight gradients in bf16 or, with `accumulate`, added to fp32 gradient buffers;
  map      moe_route over all experts, then moe_global_map for rank 3 of `W`: the index stage in
           front of an expert-parallel token exchange, where the expert work is elsewhere.

T tokens of width d, E experts of inner width I of which [0, E_loc) are local, k experts a token.
Layer shapes are those of the paper's model table and of the benchmark workloads (moe_synth.py).
"""
import math

import torch

import paper_2604_19241_amd as moe

# (d, I, E, k) of the layers: the benchmark's workloads and the paper's model table
TINY = (512, 1024, 8, 2)
MIXTRAL = (4096, 14336, 8, 2)
DEEPSEEK_MOE_16B = (2048, 1408, 64, 6)
DEEPSEEK_OCR_2 = (1280, 896, 64, 6)
DEEPSEEK_V2 = (5120, 1536, 160, 6)
DEEPSEEK_R1 = (7168, 2048, 256, 8)
QWEN3_30B = (2048, 768, 128, 8)
QWEN3_235B = (4096, 1536, 128, 8)
QWEN3_NEXT = (2048, 512, 512, 10)
QWEN3_OMNI = (1024, 384, 128, 6)
KIMI_LINEAR = (2304, 1024, 256, 8)


def _case(kind, layer, T, E_loc=None, zipf=0.0, accumulate=False, W=0):
    d, I, E, k = layer
    return {"kind": kind, "T": T, "d": d, "I": I, "E": E, "E_loc": E if E_loc is None else E_loc, "k": k,
            "zipf": zipf, "accumulate": accumulate, "W": W}


def listed():
    cases = {
        # one sequence generating: the smallest call there is, all latency and launches
        "decode-1": _case("decode", QWEN3_30B, 1),
        # a small batch of sequences: 2 rows an expert on average, every expert's weights streamed
        "decode-32": _case("decode", QWEN3_30B, 32),
        # a large batch at one rank of eight: the tokens of all ranks, an eighth of the experts, 8 rows each
        "decode-share-256": _case("decode", DEEPSEEK_R1, 256, E_loc=32),
        # a short prompt of odd length on many small experts (20 rows each)
        "prefill-1021": _case("prefill", QWEN3_NEXT, 1021),
        # an ordinary prompt of odd length (384 rows an expert, inner width no multiple of 256)
        "prefill-4099": _case("prefill", DEEPSEEK_MOE_16B, 4099),
        # few large experts: 1024 rows each, the longest inner width
        "prefill-large-experts": _case("prefill", MIXTRAL, 4096),
        # a very small training step: launches and latency in both directions
        "train-tiny": _case("train", TINY, 256),
        # the benchmark's training step
        "train": _case("train", QWEN3_30B, 8192),
        # the same under skewed routing, odd length: one expert has an eighth of the rows, some have none
        "train-skewed": _case("train", QWEN3_30B, 8001, zipf=1.2),
        # one rank's share of a wide layer: 256 rows for each of 32 local experts
        "train-share": _case("train", DEEPSEEK_R1, 8192, E_loc=32),
        # one rank of eight with the tokens of all ranks, 1875 rows for each of 32 local experts,
        # weight gradients accumulated over micro-batches in fp32
        "train-accumulate": _case("train", KIMI_LINEAR, 60001, E_loc=32, accumulate=True),
        # the index stage of expert parallelism alone
        "map": _case("map", DEEPSEEK_R1, 32768, W=8),
    }
    return [dict(c, name=n) for n, c in cases.items()]


def _experts_hit(c):
    """Local experts that at least one token selects, on average."""
    if c["zipf"] > 0:
        z = [r ** -c["zipf"] for r in range(1, c["E"] + 1)]
        p = [min(1.0, c["k"] * v / sum(z)) for v in z]
    else:
        p = [c["k"] / c["E"]] * c["E"]
    return c["E_loc"] / c["E"] * sum(1.0 - (1.0 - v) ** c["T"] for v in p)


def _rows(c):
    return c["T"] * c["k"] * c["E_loc"] / c["E"]


def work(case):
    c = case
    T, d, I, E, k = c["T"], c["d"], c["I"], c["E"], c["k"]
    rows, tables = _rows(c), 4.0 * (4 * T * k + 2 * c["E_loc"])
    route = 4.0 * T * E + tables
    if c["kind"] == "map":
        return {"bytes": route + 4.0 * (2 * T * k + 5 * T * k + T + 2 * c["W"] * E), "flops": 0.0}
    weights = 6.0 * _experts_hit(c) * d * I
    tokens = 2.0 * T * d
    forward = tokens + weights + tokens
    if c["kind"] != "train":
        return {"bytes": route + forward, "flops": 6.0 * rows * d * I}
    stash = 2.0 * rows * 3 * I
    # every local expert's gradient is written; added to, it is read as well
    grads = 6.0 * c["E_loc"] * d * I * (4 if c["accumulate"] else 1)
    backward = 2 * tokens + weights + stash + tokens + grads + 4.0 * T * k
    return {"bytes": route + forward + stash + backward + 4.0 * (3 * T * k + T * E), "flops": 18.0 * rows * d * I}


def draw(rng):
    """One more case: a kind, a layer, a share of its experts, a length, all at random."""
    most = max(work(c)["bytes"] for c in listed()), max(work(c)["flops"] for c in listed())
    while True:
        kind = rng.choice(["decode", "decode", "prefill", "prefill", "train", "train", "train", "map"])
        layer = rng.choice([TINY, MIXTRAL, DEEPSEEK_MOE_16B, DEEPSEEK_OCR_2, DEEPSEEK_V2, DEEPSEEK_R1, QWEN3_30B,
                            QWEN3_235B, QWEN3_NEXT, QWEN3_OMNI, KIMI_LINEAR])
        low, high = {"decode": (1, 512), "prefill": (200, 16384), "train": (200, 65536), "map": (1000, 65536)}[kind]
        T = round(math.exp(rng.uniform(math.log(low), math.log(high))))
        E = layer[2]
        ranks = rng.choice([1, 1, 2, 4, 8])
        if kind == "map":
            c = _case(kind, layer, T, W=rng.choice([2, 4, 8]))
        else:
            c = _case(kind, layer, T, E_loc=max(2, E // ranks), zipf=rng.choice([0.0, 0.0, 0.0, 0.6, 1.2]),
                      accumulate=kind == "train" and rng.random() < 0.3)
        w = work(c)
        # a small share of a long batch has buffers for rows that it never gets: bounded as well
        held = 2.0 * T * c["k"] * (3 * c["d"] + 10 * c["I"]) if kind != "map" else 0.0
        if w["bytes"] <= 0.7 * most[0] and w["flops"] <= 0.7 * most[1] and held <= 3e10:
            return c


def _normal(shape, std, g):
    out = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    step = max(1, (1 << 27) // max(1, out.numel() // shape[0]))
    for i in range(0, shape[0], step):
        n = min(step, shape[0] - i)
        out[i:i + n] = torch.randn((n,) + tuple(shape[1:]), generator=g, device="cuda") * std
    return out


def prepare(case, seed):
    c = case
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    T, d, I, E, k, n = c["T"], c["d"], c["I"], c["E"], c["k"], c["E_loc"]
    shape = moe.make_shape(T=T, d=d, E=E, k=k, I=I, e_start=0, e_count=n)
    size = moe.moe_workspace_bytes(shape)

    def buffer(nbytes):
        return torch.empty(max(nbytes, 256), dtype=torch.uint8, device="cuda")

    s = {"kind": c["kind"], "W": c["W"], "shape": shape, "opts": None}
    x = _normal((T, d), 1.0, g)
    logits = x.float() @ _normal((d, E), 0.02, g).float()
    if c["zipf"] > 0:
        rank = torch.randperm(E, generator=g, device="cuda") + 1
        logits -= c["zipf"] * torch.log(rank.float())
    s["logits"] = logits.contiguous()
    s["ws_route"] = buffer(size["route"])
    if c["kind"] == "map":
        # the other ranks' histograms: counts of the same size, as an all-gather hands them over
        mean = T * k / E
        s["c_all"] = (mean * (0.8 + 0.4 * torch.rand((c["W"], E), generator=g, device="cuda"))).to(torch.int32)
        s["ws_map"] = buffer(8 * E)
        return s
    s["x"] = x
    s["w"] = [_normal((n, d, I), 0.02, g), _normal((n, d, I), 0.02, g), _normal((n, I, d), 0.02, g)]
    s["y"] = torch.empty((T, d), dtype=torch.bfloat16, device="cuda")
    s["ws_fwd"] = buffer(size["fwd"])
    if c["kind"] == "decode":
        s["routing"] = moe.alloc_routing(shape, "cuda")
    if c["kind"] == "train":
        s["dy"] = _normal((T, d), 1.0, g)
        s["saved"] = moe.alloc_saved(shape, "cuda")
        s["opts"] = moe.make_opts(dw_accumulate=1) if c["accumulate"] else None
        s["ws_bwd"] = buffer(moe.moe_backward_workspace_bytes(shape, s["opts"]))
        kind = torch.float32 if c["accumulate"] else torch.bfloat16
        s["grads"] = {"dx": torch.empty_like(x), "dtopk_w": torch.empty((T, k), dtype=torch.float32, device="cuda")}
        for name, w in zip(("dw_gate", "dw_up", "dw_down"), s["w"]):
            s["grads"][name] = torch.zeros(w.shape, dtype=kind, device="cuda")
        s["dlogits"] = torch.empty((T, E), dtype=torch.float32, device="cuda")
    return s


def _tables(r):
    return {name: getattr(r, name) for name in ("topk_idx", "topk_w", "counts", "offsets", "perm", "inv_perm")}


def run(state):
    s, shape = state, state["shape"]
    if s["kind"] == "decode":
        r = moe.moe_route_static(shape, s["logits"], s["routing"])
    else:
        r = moe.moe_route(shape, s["logits"], ws=s["ws_route"])
    if s["kind"] == "map":
        return {"routing": _tables(r), "map": vars(moe.moe_global_map(shape, s["W"], min(3, s["W"] - 1), r, s["c_all"], ws=s["ws_map"]))}
    w_gate, w_up, w_down = s["w"]
    if s["kind"] != "train":
        y = moe.moe_fused_forward(shape, s["x"], w_gate, w_up, w_down, r, y=s["y"], ws=s["ws_fwd"])
        return {"routing": _tables(r), "y": y}
    y = moe.moe_fused_forward(shape, s["x"], w_gate, w_up, w_down, r, y=s["y"], saved=s["saved"], ws=s["ws_fwd"])
    grads = moe.moe_fused_backward(shape, s["dy"], s["x"], w_gate, w_up, w_down, r, s["saved"], ws=s["ws_bwd"],
                                   opts=s["opts"], out=s["grads"])
    dlogits = moe.moe_route_backward(shape, r, grads["dtopk_w"], out=s["dlogits"])
    return {"routing": _tables(r), "y": y, "grads": grads, "dlogits": dlogits}


def tolerance(case):
    # Measured once on every listed case against the layer in fp32 without the roundings to bf16
    # between its stages: y 2.9e-3 (largest element 0.037), gradients up to 3.5e-3, the gate and
    # logit gradients 1.7e-3 (largest element 0.13, where the terms of a logit's gradient cancel).
    # About three to four times that; the index arrays have to be the same.
    if case["kind"] == "map":
        return {"rel": 1e-6}   # gates only
    return {"rel": 1e-2, "max": 0.15 if case["kind"] != "train" else 0.4}


def _gates(s, c):
    """Selected experts (ties to the lower id) and their gates in 64 bits."""
    v, idx = torch.sort(s["logits"].double(), dim=1, descending=True, stable=True)
    return idx[:, :c["k"]], torch.softmax(v[:, :c["k"]], dim=1)


def exact(case, seed):
    """What run returns for these inputs as plain torch computes it in 64 bits, without any rounding
    between the stages.  None for the index arrays, which are whole numbers."""
    c = case
    s = prepare(case, seed)
    idx, gate = _gates(s, c)
    tables = dict.fromkeys(("topk_idx", "topk_w", "counts", "offsets", "perm", "inv_perm"))
    tables["topk_w"] = gate
    if c["kind"] == "map":
        names = ("dst_rank", "dst_expert", "dst_off", "dst_row", "send", "n_dst_ranks", "recv_offsets")
        return {"routing": tables, "map": dict.fromkeys(names)}
    train = c["kind"] == "train"
    y = torch.zeros((c["T"], c["d"]), dtype=torch.float64, device="cuda")
    if train:
        dx, dgate = torch.zeros_like(y), torch.zeros_like(gate)
        dw = [torch.zeros(w.shape, dtype=torch.float64, device="cuda") for w in s["w"]]
    for e in range(c["E_loc"]):
        tok, slot = torch.nonzero(idx == e, as_tuple=True)
        if tok.numel() == 0:
            continue
        wg, wu, wd = (w[e].double() for w in s["w"])
        x, p = s["x"][tok].double(), gate[tok, slot][:, None]
        g, u = x @ wg, x @ wu
        sig = torch.sigmoid(g)
        h = g * sig * u
        y.index_add_(0, tok, p * (h @ wd))
        if train:
            dy = s["dy"][tok].double()
            raw = dy @ wd.T
            dgate[tok, slot] = (raw * h).sum(1)
            dh = p * raw
            dg, du = dh * u * sig * (1.0 + g * (1.0 - sig)), dh * g * sig
            dw[0][e], dw[1][e], dw[2][e] = x.T @ dg, x.T @ du, h.T @ (p * dy)
            dx.index_add_(0, tok, dg @ wg.T + du @ wu.T)
    if not train:
        return {"routing": tables, "y": y}
    dlogits = torch.zeros((c["T"], c["E"]), dtype=torch.float64, device="cuda")
    dlogits.scatter_(1, idx, gate * (dgate - (gate * dgate).sum(1, keepdim=True)))
    grads = {"dx": dx, "dtopk_w": dgate, "dw_gate": dw[0], "dw_up": dw[1], "dw_down": dw[2]}
    return {"routing": tables, "y": y, "grads": grads, "dlogits": dlogits}
