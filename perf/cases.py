"""The work that users have this library do, as cases that can be timed and compared: whole layers through
XMoELayer / XMoE2Layer (training steps and forward passes), and the dispatch metadata of the redundancy-bypassing
exchange through the function-level API.

Shapes are those of xmoe_inputs.CONFIGS (and of the paper's model table behind them) or generic ones in between.
A case is a dict of plain values:
  what     "train" (forward + backward, all gradients), "forward" (the layer's output), "rbd" (dispatch metadata)
  expert   "swiglu" | "mlp2";  act: activation of the two-matrix expert
  dtype    "bf16" | "f32"
  T, d, E, k, f, E_s   tokens, model width, experts, experts per token, expert width, shared experts
  skew     steepness of the load profile (0: near-uniform), capacity: rows an expert keeps at most (0: dropless)
  epn      experts per destination node ("rbd")
"""
import math

import torch

import paper_2508_13337_amd as xm

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(name, what="train", expert="swiglu", act="", dtype="bf16", T=8192, d=2048, E=64, k=6, f=1408, E_s=0, skew=0.0,
          capacity=0, epn=0):
    c = dict(what=what, expert=expert, act=act, dtype=dtype, T=T, d=d, E=E, k=k, f=f, E_s=E_s, skew=skew,
             capacity=capacity, epn=epn)
    return dict(c, name=name) if name else c


def listed():
    return [
        # a toy float32 layer (unit tests, debugging, notebooks): launches and host calls are all there is to it
        _case("tiny_f32", dtype="f32", T=256, d=128, E=8, k=2, f=64),
        # full-precision training of a small model: float32 arithmetic at ordinary sizes
        _case("f32", dtype="f32", T=2048, d=1024, E=16, k=4, f=704, E_s=1),
        # bf16 training at widths that are no multiple of any tile
        _case("odd_bf16", T=3001, d=1000, E=24, k=3, f=712, E_s=1),
        # one decoding step of a small batch: every active expert's weights are read for a handful of rows
        _case("decode", what="forward", T=8, E_s=2),
        # prompt processing of one request: a few dozen rows per expert
        _case("prefill", what="forward", T=509, E_s=2),
        # a small micro-batch (gradient accumulation, pipeline stages): about a hundred rows per expert
        _case("microbatch", T=1021, E_s=2),
        # the DeepSeek-MoE-16B-shaped training step, near-uniform load
        _case("dsmoe16b", E_s=2),
        # the same with a Zipf-skewed load and token dropping at 1.25 times the mean load
        _case("skew_capped", E_s=2, skew=1.25, capacity=960),
        # the paper's own two-matrix expert at its Small shapes
        _case("small_mlp2", expert="mlp2", act="gelu"),
        # long-sequence training: 65536 tokens of one sequence
        _case("longseq", T=65536),
        # the large fine-grained layer: 256 experts, 23 GB of weights and as much of gradients
        _case("large", T=4096, d=7168, E=256, k=8, f=2048, E_s=1),
        # routing, ERI-arrays and stage 0 of the redundancy-bypassing dispatch with its token buffers
        _case("rbd", what="rbd", epn=8),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: every family of listed() over its range, none dearer than the largest listed one."""
    most_flops, most_bytes, most_f32 = 1.1e13, 9e10, 2e11
    while True:
        kind = rng.choice(["train", "train", "mlp2", "micro", "forward", "forward", "odd", "f32", "f32", "rbd"])
        E = rng.choice([4, 8, 16, 24, 32, 64, 96, 128, 256])
        k = rng.randint(1, min(8, E))
        skew = rng.choice([0.0, 0.0, 0.0, 0.6, 1.25])
        if kind in ("train", "mlp2", "micro", "forward"):
            d, f = 64 * _log(rng, 8, 112), 64 * _log(rng, 4, 40)
            T = {"forward": lambda: _log(rng, 1, 4096), "micro": lambda: _log(rng, 64, 2048)}.get(
                kind, lambda: _log(rng, 2048, 65536))()
            E_s = rng.choice([0, 0, 1, 2])
            expert = "mlp2" if kind == "mlp2" or (kind != "train" and rng.random() < 0.25) else "swiglu"
            act = rng.choice(["gelu", "gelu", "silu", "identity"]) if expert == "mlp2" else ""
            capacity = 0
            if expert == "swiglu" and kind == "train" and rng.random() < 0.25:
                capacity = max(1, int(rng.uniform(0.8, 1.5) * T * k / E))
            c = _case("", what="forward" if kind == "forward" else "train", expert=expert, act=act, T=T, d=d, E=E, k=k,
                      f=f, E_s=0 if expert == "mlp2" else E_s, skew=skew, capacity=capacity)
        elif kind == "odd":
            step = rng.choice([8, 8, 8, 2, 1])
            c = _case("", T=_log(rng, 128, 8192), d=step * (_log(rng, 64, 2048) // step), E=E, k=k,
                      f=step * (_log(rng, 64, 1500) // step), E_s=rng.choice([0, 1]), skew=skew)
        elif kind == "f32":
            c = _case("", dtype="f32", T=_log(rng, 64, 4096), d=_log(rng, 64, 1536), E=E, k=k, f=_log(rng, 48, 1024),
                      E_s=rng.choice([0, 1]), skew=skew)
        else:
            epn = rng.choice([e for e in (1, 2, 4, 8, 16) if E % e == 0])
            c = _case("", what="rbd", T=_log(rng, 256, 16384), d=64 * _log(rng, 8, 64), E=E, k=k, epn=epn)
        w = work(c)
        slow = c["dtype"] == "f32" or c["d"] % 64 or c["f"] % 64
        if w["flops"] <= (most_f32 if slow else most_flops) and w["bytes"] <= most_bytes:
            return c


def prepare(case, seed):
    """The layer object, weights, gradient buffers and one batch, all on the GPU."""
    c = case
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    dt = DTYPES[c["dtype"]]
    T, d, E, k, f, E_s = (c[n] for n in ("T", "d", "E", "k", "f", "E_s"))

    def normal(shape, std):
        return torch.empty(shape, dtype=dt, device="cuda").normal_(0.0, std, generator=g)

    s = {"case": c, "x": normal((T, d), 1.0), "w": {"w_router": normal((d, E), d ** -0.5), "bias": None}}
    if c["skew"]:      # bias[e] = -skew * 1.2 * ln(rank of e), ranks in random order
        rank = torch.randperm(E, generator=g, device="cuda") + 1
        s["w"]["bias"] = -c["skew"] * 1.2 * torch.log(rank.float())
    if c["what"] == "rbd":
        i32 = dict(dtype=torch.int32, device="cuda")
        B = T * k
        s["rand_key"] = torch.randint(-2 ** 31, 2 ** 31 - 1, (B,), generator=g, **i32)
        s["logits"] = torch.empty((T, E), dtype=torch.float32, device="cuda")
        s["topk_idx"], s["topk_w"] = torch.empty((T, k), **i32), torch.empty((T, k), dtype=torch.float32, device="cuda")
        s["eri"] = {"tokens_per_expert": torch.empty(E, **i32), "expert_offsets": torch.empty(E + 1, **i32),
                    "token_ids": torch.empty(B, **i32), "expert_ids": torch.empty(B, **i32),
                    "combine_weights": torch.empty(B, dtype=torch.float32, device="cuda"),
                    "row_of_slot": torch.empty(B, **i32)}
        s["meta"] = {n: torch.empty(B, **i32) for n in (
            "pilot_token_ids", "pilot_expert_ids", "replica_token_ids", "replica_expert_ids", "s1_mapping_indices",
            "s1_mapping_experts", "merge_src")}
        s["meta"].update({n: torch.empty(E, **i32) for n in ("pilot_tokens_per_expert", "replica_tokens_per_expert")})
        s["meta"].update({n: torch.empty(E + 1, **i32) for n in ("pilot_offsets", "replica_offsets")})
        s["absolute"] = torch.empty(B, **i32)
        s["pilots"], s["replicas"] = (torch.zeros((B, d), dtype=dt, device="cuda") for _ in range(2))
        s["ws"] = xm.alloc_workspace(max(xm.xmoe_workspace_bytes(xm.WS_BUILD_ERI, T, d, E, k, 0, xm.XMOE_BF16),
                                         xm.xmoe_workspace_bytes(xm.WS_RBD_STAGE0, T, d, E, k, 0, xm.XMOE_BF16)))
        return s
    names = ("w1", "w2") if c["expert"] == "mlp2" else ("wg", "wu", "wd")
    for n in names:
        s["w"][n] = normal((E + E_s,) + ((f, d) if n in ("w2", "wd") else (d, f)), 0.02)
    if c["expert"] == "mlp2":
        s["layer"] = xm.XMoE2Layer(T, d, E, k, f, dt, act=c["act"])
    else:
        s["layer"] = xm.XMoELayer(T, d, E, k, f, dt, E_s=E_s, max_token_count=c["capacity"] or None)
    if c["what"] == "train":
        s["dout"] = normal((T, d), 1.0)
        s["grads"] = {"d" + n: torch.empty_like(s["w"][n]) for n in ("w_router",) + names}
    return s


def run(state):
    s, c = state, state["case"]
    if c["what"] == "rbd":
        e, m = s["eri"], s["meta"]
        xm.xmoe_gate_logits(s["x"], s["w"]["w_router"], s["w"]["bias"], s["logits"])
        xm.xmoe_route(s["logits"], c["k"], s["topk_idx"], s["topk_w"])
        xm.xmoe_build_eri(s["topk_idx"], s["topk_w"], c["E"], e["tokens_per_expert"], e["expert_offsets"],
                          e["token_ids"], e["expert_ids"], e["combine_weights"], e["row_of_slot"], s["ws"])
        xm.xmoe_rbd_stage0(s["topk_idx"], s["rand_key"], e["token_ids"], e["expert_ids"], e["expert_offsets"],
                           e["row_of_slot"], c["epn"], m, s["ws"])
        xm.xmoe_dispatch(s["x"], m["pilot_token_ids"], s["pilots"])
        xm.xmoe_rbd_absolute_index(m["s1_mapping_indices"], m["s1_mapping_experts"], m["pilot_offsets"], s["absolute"])
        xm.xmoe_dispatch(s["pilots"], s["absolute"], s["replicas"])
        return [e, m, s["absolute"], s["pilots"], s["replicas"]]
    layer = s["layer"]
    out = layer.forward(s["x"], s["w"])
    if c["what"] == "forward":
        return [out, layer.topk_idx, layer.topk_w]
    dx = layer.backward(s["x"], s["w"], s["dout"], s["grads"])
    return [out, dx, s["grads"], layer.topk_idx, layer.topk_w]


def _rows(c):
    """Expected rows of every routed expert: shares follow rank^(-1.2 skew), no expert gets a token twice."""
    share = [float(e + 1) ** (-1.2 * c["skew"]) for e in range(c["E"])]
    T, B = c["T"], c["T"] * c["k"]
    lo, hi = 0.0, B / min(share)
    for _ in range(60):
        mid = (lo + hi) / 2
        lo, hi = (mid, hi) if sum(min(T, mid * p) for p in share) < B else (lo, mid)
    rows = [min(T, hi * p) for p in share]
    return [min(r, c["capacity"]) for r in rows] if c["capacity"] else rows


def work(case):
    c = case
    T, d, E, k, f, E_s = (c[n] for n in ("T", "d", "E", "k", "f", "E_s"))
    size = 4 if c["dtype"] == "f32" else 2
    token = T * d * size
    gate = 2 * T * d * E
    if c["what"] == "rbd":
        # tokens in; the token rows of pilots and replicas out; 15 integers for each of the T*k entries
        return {"bytes": token + d * E * size + T * k * (d * size + 15 * 4), "flops": gate}
    matrices = 2 if c["expert"] == "mlp2" else 3
    rows = _rows(c)
    flops = 2 * matrices * d * f * (sum(rows) + E_s * T) + gate
    read = (sum(-math.expm1(-r) for r in rows) + E_s) * matrices * d * f * size + d * E * size    # experts with rows
    if c["what"] == "forward":
        return {"bytes": 2 * token + read + 8 * T * k, "flops": flops}
    written = (E + E_s) * matrices * d * f * size + d * E * size
    return {"bytes": 4 * token + read + written + 8 * T * k, "flops": 3 * flops}


def tolerance(case):
    # four times what the path shows against itself in float64 (same routing), over the listed and some drawn cases:
    # bf16 3.5e-3 in every gradient (stored intermediates are rounded to bf16), float32 1.2e-6 (weight gradients of
    # long segments); the integer outputs and the row copies of "rbd" are the same bits, its float32 softmax is not
    # pinned beyond its rounding
    if case["what"] == "rbd":
        return {"rel": 1e-6, "max": 4e-6}
    return {"rel": 5e-6, "max": 2e-4} if case["dtype"] == "f32" else {"rel": 1.4e-2, "max": 0.3}


def _act64(name, h):
    """act(h) and its derivative."""
    if name == "identity":
        return h, torch.ones_like(h)
    if name == "gelu":
        phi = torch.exp(-0.5 * h * h) / math.sqrt(2.0 * math.pi)
        cdf = 0.5 * torch.erfc(-h / math.sqrt(2.0))
        return h * cdf, cdf + h * phi
    sig = torch.sigmoid(h)
    return h * sig, sig * (1.0 + h * (1.0 - sig))


def exact(case, seed):
    """What run() returns for these inputs, in float64 throughout (routing included: where two logits are closer than
    float32 can tell, a token may go elsewhere than run() sends it).  Whole-number outputs are left out."""
    s, c = prepare(case, seed), case
    T, d, E, k = (c[n] for n in ("T", "d", "E", "k"))
    keep = torch.float64 if c["dtype"] == "f32" else torch.float32      # bf16 results need no more
    w, x = s["w"], s["x"].double()
    logits = x @ w["w_router"].double()
    if w["bias"] is not None:
        logits += w["bias"].double()
    p = torch.softmax(logits, dim=1)
    idx = torch.sort(logits, dim=1, descending=True, stable=True).indices[:, :k]
    topk_w = p.gather(1, idx)
    flat_e, flat_w = idx.reshape(-1), topk_w.reshape(-1)
    order = torch.sort(flat_e, stable=True).indices                     # rows: flat entries by expert, stable
    if c["what"] == "rbd":
        return [{"combine_weights": flat_w[order]}, None, None, None, None]
    ends = torch.cumsum(torch.bincount(flat_e, minlength=E), 0).tolist()
    train = c["what"] == "train"
    out, dx, dw = torch.zeros_like(x), torch.zeros_like(x), torch.zeros_like(flat_w)
    dout = s["dout"].double() if train else None
    names = ("w1", "w2") if c["expert"] == "mlp2" else ("wg", "wu", "wd")
    grads = {"d" + n: torch.zeros(w[n].shape, dtype=keep, device="cuda") for n in names} if train else {}
    for e in range(E + (c["E_s"] if c["expert"] != "mlp2" else 0)):
        if e < E:
            slot = order[(ends[e - 1] if e else 0):ends[e]]
            if c["capacity"] and len(slot) > c["capacity"]:              # the heaviest ones stay, ties: lower slot
                slot = slot[torch.sort(flat_w[slot], descending=True, stable=True).indices[:c["capacity"]]]
            tok, scale = slot // k, flat_w[slot][:, None]
        else:
            tok, scale = torch.arange(T, device="cuda"), torch.ones((T, 1), dtype=torch.float64, device="cuda")
        if len(tok) == 0:
            continue
        X = x[tok]
        m = [w[n][e].double() for n in names]
        first = [X @ a for a in m[:-1]]
        if c["expert"] == "mlp2":
            A, slope = _act64(c["act"], first[0])
        else:
            silu, slope = _act64("silu", first[0])
            A = silu * first[1]
        Y = A @ m[-1]
        out.index_add_(0, tok, scale * Y)
        if not train:
            continue
        if e < E:
            dw[slot] = (dout[tok] * Y).sum(1)
        dY = scale * dout[tok]
        dA = dY @ m[-1].t()
        back = [dA * slope] if c["expert"] == "mlp2" else [dA * first[1] * slope, dA * silu]
        grads["d" + names[-1]][e] = A.t() @ dY
        for n, a, b in zip(names, m, back):
            grads["d" + n][e] = X.t() @ b
            dx.index_add_(0, tok, b @ a.t())
    if not train:
        return [out.to(keep), None, topk_w]
    inner = torch.zeros_like(p).scatter_(1, idx, dw.reshape(T, k))
    dlogits = p * (inner - (p * inner).sum(1, keepdim=True))
    grads["dw_router"] = (x.t() @ dlogits).to(keep)
    dx += dlogits @ w["w_router"].double().t()
    return [out.to(keep), dx.to(keep), grads, None, topk_w]
