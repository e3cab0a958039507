"""Timing cases: what a program that serves Mixture-of-Experts layers with this library asks it for.

A decode case is one or more decode steps through a stack of `layers` MoE layers, called as a serving loop calls
them: begin_token, then layer_step for every layer with that layer's residual r_l.  The residuals are given (a
first-order autoregressive stream, correlation 0.9 from layer to layer) and do not depend on the outputs, so that a
rounding difference in one layer cannot move the next one to other experts.  A prefill case is a prompt through
prefill_layer_step.  The layers of a stack read the expert blocks of one host pool layer; each layer has its own
router, gain, default vectors and device slots, so bytes moved and kernels run are those of distinct layers.

`slots` against the experts that the steps of a pass use decides what a case spends its time on: with enough slots
the working set stays on the device after the first pass (a warm cache: the kernels and the host path count), with
few of them every step waits for transfers over the host link.
"""
import math

import numpy as np
import torch

from paper_2603_19289_amd import moe_spec as M
from paper_2603_19289_amd.engine import Engine

W_STD, D_STD, RHO, EPS = 0.02, 0.05, 0.9, 1e-6
MODES = {"on_demand": M.MODE_ON_DEMAND, "speculative": M.MODE_SPECULATIVE, "prefetch_hint": M.MODE_PREFETCH_HINT}
COPIES = {"kernel": M.COPY_KERNEL, "dma2": M.COPY_DMA2}


def _case(name, kind, hidden, experts, top_k, inter, *, layers, batch, slots, dtype="bf16", mode="speculative",
          tokens=1, copy="kernel", clusters=0, estimator=False):
    """batch: tokens per decode step, or tokens of the prompt."""
    c = dict(kind=kind, hidden=hidden, experts=experts, top_k=top_k, inter=inter, layers=layers, batch=batch,
             slots=slots, dtype=dtype, mode=mode, tokens=tokens, copy=copy, clusters=clusters, estimator=estimator)
    return dict(name=name, **c) if name else c


def listed():
    tiny, qwen, oss, mix = (256, 8, 2, 512), (2048, 128, 8, 768), (2880, 32, 4, 2880), (4096, 8, 2, 14336)
    return [
        # the smallest stack, float32, half of its experts on the device: launches, hand-overs and small copies
        _case("tiny_f32_b1", "decode", *tiny, layers=4, batch=1, slots=4, dtype="f32", tokens=4),
        # one user, 128 small experts, working set cached: the method's ordinary decode step without transfers
        _case("qwen_b1_warm", "decode", *qwen, layers=12, batch=1, slots=32, tokens=2),
        # the same layers without speculation: the true experts, found in the cache
        _case("qwen_b1_on_demand_warm", "decode", *qwen, layers=12, batch=1, slots=32, tokens=2, mode="on_demand"),
        # one user, layer sizes that are no multiple of 128 (2880)
        _case("oss_b1_warm", "decode", *oss, layers=8, batch=1, slots=12, tokens=2),
        # one user, few large experts
        _case("mixtral_b1_warm", "decode", *mix, layers=4, batch=1, slots=4),
        # a small batch of unrelated sequences, every expert cached
        _case("oss_b8_warm", "decode", *oss, layers=6, batch=8, slots=32),
        # a larger batch of sequences in four groups of like ones
        _case("qwen_b32_warm", "decode", *qwen, layers=6, batch=32, slots=128, clusters=4),
        # the learned estimator instead of the next layer's router, on every layer
        _case("qwen_b4_estimator_warm", "decode", *qwen, layers=8, batch=4, slots=96, estimator=True),
        # the headline workload: 16 slots, most predicted experts travel over the link while layers compute
        _case("qwen_b1_offload", "decode", *qwen, layers=8, batch=1, slots=16, tokens=4, copy="dma2"),
        # loading on demand with more routed experts than slots: several cache waves per layer
        _case("oss_b8_on_demand_offload", "decode", *oss, layers=2, batch=8, slots=8, mode="on_demand"),
        # an ordinary prompt: every expert of a layer is streamed
        _case("qwen_prefill_512", "prefill", *qwen, layers=2, batch=512, slots=16, copy="dma2"),
        # the longest prompt the library takes
        _case("mixtral_prefill_32k", "prefill", *mix, layers=1, batch=32768, slots=3, copy="dma2"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["tiny", "warm", "warm", "warm", "batch", "batch", "batch", "offload", "prefill", "prefill"])
    if kind == "tiny":
        experts, top_k = rng.randint(4, 16), rng.randint(1, 4)
        return _case(None, "decode", 8 * rng.randint(16, 64), experts, top_k, 8 * rng.randint(16, 128),
                     layers=rng.randint(2, 5), batch=_log(rng, 1, 8), slots=rng.randint(top_k, experts), dtype="f32",
                     mode=rng.choice(sorted(MODES)), tokens=rng.randint(1, 4))
    # expert shapes between the listed models', with at most 2 GB of blocks per layer
    hidden, experts = 8 * rng.randint(128, 512), _log(rng, 8, 128)
    top_k = rng.randint(2, max(2, min(8, experts // 4)))
    inter = 8 * (_log(rng, 512, max(520, min(14336, 2 * 10 ** 9 // (6 * hidden * experts)))) // 8)
    sizes = (hidden, experts, top_k, inter)
    if kind == "prefill":
        # the tokens of the longest listed prompt, or fewer: at most as many products as there
        most = min(32768, int(32768 * 2 * 4096 * 14336 / (top_k * hidden * inter)))
        return _case(None, "prefill", *sizes, layers=1, batch=_log(rng, 100, max(101, most)),
                     slots=rng.randint(max(2, top_k), max(2, top_k, experts // 4)), copy="dma2")
    mode = rng.choice(["speculative", "speculative", "on_demand", "prefetch_hint"])
    if kind == "warm":
        return _case(None, "decode", *sizes, layers=rng.randint(3, 8), batch=1, slots=rng.randint(min(experts, 2 * top_k), experts),
                     mode=mode, estimator=mode != "on_demand" and rng.random() < 0.15)
    if kind == "batch":
        return _case(None, "decode", *sizes, layers=rng.randint(2, 5), batch=_log(rng, 2, 64), slots=experts, mode=mode,
                     clusters=rng.choice([0, 0, 4]), estimator=mode != "on_demand" and rng.random() < 0.15)
    return _case(None, "decode", *sizes, layers=2, batch=_log(rng, 1, 8), slots=rng.randint(top_k, max(top_k, experts // 4)),
                 mode=mode, copy=rng.choice(["kernel", "dma2"]))


# ---- inputs


def _normal(g, shape, std, dtype):
    return torch.empty(shape, dtype=torch.float32, device="cuda").normal_(0.0, std, generator=g).to(dtype)


def _inputs(case, seed):
    """Everything random of a case, on the GPU, from the seed alone."""
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 1000003 + 17)
    L, H, E, I, B, T = (case[k] for k in ("layers", "hidden", "experts", "inter", "batch", "tokens"))
    wt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    x = {"router_w": _normal(g, (L, E, H), W_STD, wt), "dvecs": _normal(g, (L, E, H), D_STD, wt),
         "rms_gain": 1.0 + _normal(g, (L, H), 0.1, torch.float32)}
    x["experts"] = torch.empty((E, 3 * H * I), dtype=wt, device="cuda")     # W_gate [I,H] | W_up [I,H] | W_down [H,I]
    for e in range(E):
        x["experts"][e] = _normal(g, (3 * H * I,), W_STD, wt)
    if case["estimator"]:
        dm = H // 32 * 8                                                    # latent size, about a quarter of hidden
        F = 2 * dm
        x["estimator"] = {
            "proj": _normal(g, (dm, H), H ** -0.5, wt), "layer_emb": _normal(g, (L, dm), 0.5, wt),
            "ffn_in": _normal(g, (F, dm), dm ** -0.5, wt), "ffn_out": _normal(g, (dm, F), F ** -0.5, wt),
            "ln_gain": 1.0 + _normal(g, (dm,), 0.1, torch.float32), "ln_bias": _normal(g, (dm,), 0.1, torch.float32),
            "head": _normal(g, (E, dm), dm ** -0.5, wt)}
    r = torch.empty((T, L, B, H), dtype=torch.float32, device="cuda")

    def rows():                                                             # clusters: like sequences share most of it
        own = torch.empty((T, B, H), dtype=torch.float32, device="cuda").normal_(generator=g)
        if not case["clusters"]:
            return own
        shared = torch.empty((T, case["clusters"], H), dtype=torch.float32, device="cuda").normal_(generator=g)
        return math.sqrt(0.99) * shared[:, torch.arange(B, device="cuda") % case["clusters"]] + 0.1 * own

    v = rows()
    for l in range(L):
        r[:, l] = v
        v = RHO * v + math.sqrt(1 - RHO * RHO) * rows()
    x["r"] = r
    return x


def _host(t):
    t = t.cpu().contiguous()
    return t.view(torch.int16).numpy().view(np.uint16) if t.dtype == torch.bfloat16 else t.numpy()


def prepare(case, seed):
    """The engine with its tables, the pinned pool and the residuals; a warm cache is warmed by one pass."""
    x = _inputs(case, seed)
    pool = torch.empty(x["experts"].shape, dtype=x["experts"].dtype, pin_memory=True)
    pool.copy_(x.pop("experts"))
    prefill = case["kind"] == "prefill"
    L, B, T = case["layers"], case["batch"], case["tokens"]
    eng = Engine(n_layers=L, hidden=case["hidden"], n_experts=case["experts"], top_k=case["top_k"], inter=case["inter"],
                 dtype=case["dtype"], max_batch=64 if prefill else B, slots=case["slots"], mode=MODES[case["mode"]],
                 resident={k: _host(x[k]) for k in ("router_w", "rms_gain", "dvecs")}, experts=[pool] * L, rms_eps=EPS,
                 predict_in_on_demand=0, copy_engine=COPIES[case["copy"]], max_prefill_tokens=B if prefill else 0,
                 estimator={k: _host(v) for k, v in x["estimator"].items()} if case["estimator"] else None)
    r, out = x["r"], torch.zeros_like(x["r"])
    state = {"engine": eng, "prefill": prefill, "r": [list(t) for t in r], "rows": [list(t) for t in out], "out": out}
    if prefill:
        state["ids"] = torch.zeros((L, B, case["top_k"]), dtype=torch.int32, device="cuda")
        state["gates"] = torch.zeros((L, B, case["top_k"]), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    if not prefill and case["slots"] >= min(case["experts"], T * B * case["top_k"]):
        run(state)
        torch.cuda.synchronize()
    return state


def run(state):
    eng, out = state["engine"], state["out"]
    with torch.cuda.stream(eng.compute):
        if state["prefill"]:
            for l, (r, o) in enumerate(zip(state["r"][0], state["rows"][0])):
                M.moe_spec_prefill_layer_step(eng.ctx, l, r.data_ptr(), r.shape[0], o.data_ptr(),
                                              state["ids"][l].data_ptr(), state["gates"][l].data_ptr())
            return {"out": out, "ids": state["ids"], "gates": state["gates"]}
        for rs, outs in zip(state["r"], state["rows"]):
            eng.begin_token()
            for l, (r, o) in enumerate(zip(rs, outs)):
                eng.layer_step(l, r, o, sync_input=False)
    return {"out": out}


def work(case):
    H, E, k, I, L, B, T = (case[n] for n in ("hidden", "experts", "top_k", "inter", "layers", "batch", "tokens"))
    w = 4 if case["dtype"] == "f32" else 2
    prefill, predicts = case["kind"] == "prefill", case["kind"] == "decode" and case["mode"] != "on_demand"
    rows = min(B, 2 * case["clusters"]) if case["clusters"] else B         # like sequences pick like experts
    used = E if prefill else E * (1.0 - (1.0 - k / E) ** rows)             # distinct experts of a step
    step = used * 3 * H * I * w + E * H * w + 2 * B * H * 4
    flops = 6.0 * B * k * H * I + 2.0 * B * E * H
    per_token = T * L * step
    all_flops = T * L * flops
    if predicts:
        dm = H // 32 * 8
        next_w = dm * H + 4 * dm * dm + E * dm if case["estimator"] else E * H
        per_token += T * (L - 1) * (next_w * w + used * H * w)
        all_flops += T * (L - 1) * 2.0 * B * (next_w + k * H)
    return {"bytes": per_token, "flops": all_flops}


def tolerance(case):
    """About four times the distance from the 64-bit result (float32 weights 1.5e-7; bf16 weights 2e-6 to 6e-5).
    float32 weights: sums of up to a few thousand products in another order.  bf16 weights: a SwiGLU value whose float32
    pre-image lies beside a rounding boundary moves to the neighbouring bf16 value when its sum is taken in another
    order; one such value moves an output element by a few thousandths of the row's root mean square."""
    return {"rel": 2e-6, "max": 4e-5} if case["dtype"] == "f32" else {"rel": 3e-4, "max": 1.2e-2}


# ---- the same outputs in 64 bits


def _round_bf16(x):
    """float64 -> nearest bfloat16, ties to even, as float64."""
    u = x.contiguous().view(torch.int64)
    u = (u + 0x00000FFFFFFFFFFF + ((u >> 45) & 1)) & ~0x00001FFFFFFFFFFF
    return u.view(torch.float64)


def exact(case, seed):
    x = _inputs(case, seed)
    L, H, E, k, I, B, T = (case[n] for n in ("layers", "hidden", "experts", "top_k", "inter", "batch", "tokens"))
    bf16 = case["dtype"] == "bf16"
    rnd = _round_bf16 if bf16 else (lambda v: v)
    router, dvecs, gain = x["router_w"].double(), x["dvecs"].double(), x["rms_gain"].double()
    prefill = case["kind"] == "prefill"

    def norm(v, l):
        return rnd(v * gain[l] / torch.sqrt(v.square().mean(-1, keepdim=True) + float(np.float32(EPS))))

    def select(z):
        top, ids = torch.topk(z, k, dim=-1)
        return ids, torch.softmax(top, dim=-1)

    def estimate(q, l):
        w = {n: v.double() for n, v in x["estimator"].items()}
        u = q @ w["proj"].T + w["layer_emb"][l]
        u = u + torch.nn.functional.silu(u @ w["ffn_in"].T) @ w["ffn_out"].T
        d = u - u.mean(-1, keepdim=True)
        u = d / torch.sqrt(d.square().mean(-1, keepdim=True) + float(np.float32(1e-5))) * w["ln_gain"] + w["ln_bias"]
        return u @ w["head"].T

    def experts(s, ids, gates):
        o = torch.zeros((s.shape[0], H), dtype=torch.float64, device="cuda")
        for e in torch.unique(ids).tolist():
            b, j = torch.nonzero(ids == e, as_tuple=True)
            block = x["experts"][e]
            gate, up = block[:H * I].view(I, H).double(), block[H * I:2 * H * I].view(I, H).double()
            down = block[2 * H * I:].view(H, I).double()
            for c in range(0, b.numel(), 4096):                             # in parts: the prompt may be long
                bb, jj = b[c:c + 4096], j[c:c + 4096]
                v = s[bb]
                h = rnd(torch.nn.functional.silu(v @ gate.T) * (v @ up.T))
                o[bb] += gates[bb, jj, None] * (h @ down.T)
        return o

    out = torch.zeros((T, L, B, H), dtype=torch.float64, device="cuda")
    all_gates = torch.zeros((L, B, k), dtype=torch.float64, device="cuda")
    for t in range(T):
        pending = None
        for l in range(L):
            r = x["r"][t, l].double()
            s = norm(r, l)
            true_ids, true_gates = select(s @ router[l].T)
            all_gates[l] = true_gates
            ids, gates = (true_ids, true_gates) if pending is None or case["mode"] != "speculative" else pending
            out[t, l] = experts(s, ids, gates)
            if not prefill and case["mode"] == "speculative" and l + 1 < L:
                q = norm(r + (true_gates[..., None] * dvecs[l][true_ids]).sum(-2), l + 1)
                pending = select(estimate(q, l) if case["estimator"] else q @ router[l + 1].T)
    return {"out": out, "ids": None, "gates": all_gates} if prefill else {"out": out}
