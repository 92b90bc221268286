"""The calls that a serving program makes of the MoE layer, over their real range of sizes.

A pass is one call of a public entry point (for the re-layout, the short sequence of calls that a
scale-up consists of) on tensors that are already on the GPU.  The layer object, its weight pools and
its placement are made beforehand: a program keeps them for as long as it serves.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2510_02613_amd.layer import MoELayer

# Layer shapes of the repository's workloads.  n_local: logical experts [0, n_local) live on this rank;
# shared_div: the rank's own share of the batch (data parallel) is 1/shared_div of the tokens, and the
# shared experts serve that share.  max_tokens: what the serving program sizes its workspace for.
QWEN3 = dict(hidden=2048, inter=768, n_experts=128, top_k=8, n_local=128, spare=0, act="bf16", router="f32",
             gate="softmax", n_group=1, topk_group=1, renormalize=True, scale=1.0, n_shared=0, shared_div=1,
             zipf=0.0, max_tokens=8192)
DSV3 = dict(hidden=7168, inter=2048, n_experts=256, top_k=8, n_local=32, spare=0, act="bf16", router="bf16",
            gate="sigmoid_group", n_group=8, topk_group=4, renormalize=True, scale=2.5, n_shared=1, shared_div=8,
            zipf=0.0, max_tokens=8192)
DSV2 = dict(hidden=2048, inter=1408, n_experts=64, top_k=6, n_local=64, spare=0, act="bf16", router="f32",
            gate="softmax", n_group=1, topk_group=1, renormalize=False, scale=1.0, n_shared=2, shared_div=1,
            zipf=0.0, max_tokens=4096)
TINY = dict(hidden=128, inter=64, n_experts=8, top_k=2, n_local=8, spare=0, act="f32", router="f32",
            gate="softmax", n_group=1, topk_group=1, renormalize=True, scale=1.0, n_shared=0, shared_div=1,
            zipf=0.0, max_tokens=2600)


def listed():
    return [
        # the fp32 layer at its smallest: the parity configuration, all launch latency
        dict(TINY, name="f32_tiny", entry="forward", tokens=64),
        # the fp32 layer at the upper end of the tested sizes, none of them a multiple of a tile
        dict(TINY, name="f32_ragged", entry="forward", tokens=1500, hidden=264, inter=264, n_experts=40, top_k=4,
             n_local=30, spare=3, n_shared=1, shared_div=2),
        # one user decodes: one token through all experts of a Qwen3-30B-A3B-shaped layer
        dict(QWEN3, name="qwen3_token", entry="forward", tokens=1),
        # an ordinary decode batch of the same layer
        dict(QWEN3, name="qwen3_decode", entry="forward", tokens=48),
        # a decode batch with a short prompt chunk mixed in, odd size
        dict(QWEN3, name="qwen3_chunk", entry="forward", tokens=333),
        # prefill
        dict(QWEN3, name="qwen3_prefill", entry="forward", tokens=4096),
        # a DeepSeek-V3-shaped rank of EP=8, few tokens, through the entry that needs no workspace
        dict(DSV3, name="dsv3_static", entry="static", tokens=8),
        # the same rank at the benchmark's decode size
        dict(DSV3, name="dsv3_decode", entry="forward", tokens=64),
        # the same rank when many data-parallel replicas decode together
        dict(DSV3, name="dsv3_wide_decode", entry="forward", tokens=512),
        # and at prefill size: the benchmark's headline
        dict(DSV3, name="dsv3_prefill", entry="forward", tokens=8192),
        # scale-up of a Qwen3-shaped rank under Zipf-skewed load: the second half of the experts is copied into
        # free slots while a batch is served on the first half, then the placement is switched and the next batch runs
        dict(QWEN3, name="qwen3_relayout", entry="relayout", tokens=4096, n_local=64, zipf=1.2),
        # tokens that arrive routed (after the dispatch exchange), DeepSeek-V2-Lite-shaped, odd batch
        dict(DSV2, name="dsv2_routed", entry="routed", tokens=1777),
    ]


def _log_int(rng, lo, hi):
    """A whole number spread evenly over the logarithm of [lo, hi], often an odd one."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """Another case: any of the layer shapes, expert-parallel degree, load skew and batch size that the listed ones stand for."""
    kind = rng.choice(("qwen3", "qwen3", "qwen3", "dsv3", "dsv3", "dsv3", "dsv2", "relayout", "small"))
    if kind == "qwen3":
        c = dict(QWEN3, tokens=_log_int(rng, 1, 6000), n_local=rng.choice((32, 64, 128)), zipf=rng.choice((0.0, 0.0, 1.2)))
    elif kind == "dsv3":
        c = dict(DSV3, tokens=_log_int(rng, 1, 8000), n_local=rng.choice((16, 32)))
    elif kind == "dsv2":
        c = dict(DSV2, tokens=_log_int(rng, 1, 4000), n_local=rng.choice((16, 32, 64)))
    elif kind == "relayout":
        return dict(QWEN3, entry="relayout", tokens=_log_int(rng, 16, 4000), n_local=rng.choice((32, 64)), zipf=rng.choice((0.0, 1.2)))
    else:
        group = rng.choice((True, False))
        act = rng.choice(("f32", "bf16"))
        n_experts = rng.choice((16, 32, 64)) if group else rng.choice((8, 24, 40, 96))
        c = dict(TINY, act=act, router="f32" if act == "f32" else rng.choice(("f32", "bf16")), tokens=_log_int(rng, 1, 2500),
                 hidden=8 * rng.randint(8, 64), inter=8 * rng.randint(1, 33), n_experts=n_experts, top_k=rng.randint(1, 4),
                 n_local=rng.randint(n_experts // 2, n_experts), spare=rng.choice((0, 3)), n_shared=rng.choice((0, 1, 2)),
                 shared_div=rng.choice((1, 2, 8)), renormalize=rng.choice((True, False)), scale=rng.choice((1.0, 2.5)))
        if group:
            c.update(gate="sigmoid_group", n_group=4, topk_group=rng.choice((2, 3)))
    c["entry"] = rng.choice(("forward", "forward", "forward", "routed"))
    if c["entry"] == "forward" and c["tokens"] <= 64:
        c["entry"] = rng.choice(("forward", "forward", "static"))
    return c


# A token whose k-th and next expert (or last kept and next group) score this close is not drawn: which of the
# two is taken is up to the rounding of a 32-bit sum.
_CLEAR = 2e-5


def _clear_tokens(case, x, router, bias):
    """Truth value per token: its selection does not hang on rounding."""
    k, E = case["top_k"], case["n_experts"]
    out = []
    rt = router.double().t().contiguous()
    for x0 in x.split(2048):
        s = x0.double() @ rt
        if bias is not None:
            s += bias.double()
        ok = torch.ones(s.shape[0], dtype=torch.bool, device=s.device)
        if case["gate"] == "sigmoid_group":
            s = torch.sigmoid(s)
            per = E // case["n_group"]
            g = s.view(-1, case["n_group"], per).topk(min(2, per), dim=2).values.sum(2)
            best = g.sort(dim=1, descending=True)
            kept = case["topk_group"]
            if kept < case["n_group"]:
                ok &= best.values[:, kept - 1] - best.values[:, kept] > _CLEAR
                drop = torch.zeros_like(g, dtype=torch.bool).scatter_(1, best.indices[:, kept:], True)
                s = s.masked_fill(drop.repeat_interleave(per, dim=1), -1.0)
        if k < E:
            top = s.topk(k + 1, dim=1).values
            ok &= top[:, k - 1] - top[:, k] > _CLEAR
        out.append(ok)
    return torch.cat(out)


def _slots(case):
    return case["n_local"] + case["spare"] + case["n_shared"]


def _shared_tokens(case):
    return case["tokens"] // case["shared_div"] if case["n_shared"] else 0


def prepare(case, seed):
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev).manual_seed(seed)
    host = np.random.default_rng(seed)
    H, I, E, k, T = case["hidden"], case["inter"], case["n_experts"], case["top_k"], case["tokens"]
    dt = {"bf16": torch.bfloat16, "f32": torch.float32}
    act, S = dt[case["act"]], _slots(case)
    elt = torch.int16 if case["act"] == "bf16" else torch.float32   # how the layer carries its activations

    router = (torch.randn(E, H, generator=gen, device=dev) * 0.02).to(dt[case["router"]])
    bias = None
    if case["zipf"]:
        bias = (-case["zipf"] * np.log(host.permutation(E) + 1.0)).astype(np.float32)
    x = torch.randn(T + T // 8 + 32, H, generator=gen, device=dev).to(act)
    x = x[_clear_tokens(case, x, router, None if bias is None else torch.from_numpy(bias).to(dev))][:T].contiguous()
    assert x.shape[0] == T

    raw = router.view(torch.int16).cpu().numpy().view(np.uint16) if case["router"] == "bf16" else router.cpu().numpy()
    layer = MoELayer(hidden=H, inter=I, n_experts=E, top_k=k, n_slots=S, max_tokens=max(T, case["max_tokens"]),
                     act_dtype=case["act"], router_dtype=case["router"], gate=case["gate"], n_group=case["n_group"],
                     topk_group=case["topk_group"], renormalize=case["renormalize"], routed_scale=case["scale"],
                     n_shared=case["n_shared"], router_w=raw, logit_bias=bias, device=dev)
    layer.w13.view(act).normal_(0.0, 0.02, generator=gen)
    layer.w2.view(act).normal_(0.0, 0.02, generator=gen)

    # the local experts sit in slots in any order: placement is data; the shared experts take the last slots
    slots = host.permutation(case["n_local"] + case["spare"])[:case["n_local"]]
    full = np.full(E, -1, np.int64)
    full[:case["n_local"]] = slots
    shared = list(range(S - case["n_shared"], S)) or None
    state = dict(entry=case["entry"], act=act, layer=layer, x=x.view(elt), out=torch.empty_like(x).view(elt),
                 shared=(0, _shared_tokens(case)), full=full.tolist())
    if case["entry"] == "relayout":
        half = case["n_local"] // 2
        first = full.copy()
        first[half:] = -1
        state.update(first=first.tolist(), fill=slots[half:].tolist(), out2=torch.empty_like(state["out"]),
                     side=torch.cuda.Stream(dev),
                     new13=torch.empty((half, 2 * I, H), dtype=act, device=dev).normal_(0.0, 0.02, generator=gen).view(elt),
                     new2=torch.empty((half, H, I), dtype=act, device=dev).normal_(0.0, 0.02, generator=gen).view(elt))
    else:
        layer.set_expert_map(state["full"], shared)
    if case["entry"] == "routed":
        # what the other ranks' gates sent here: k distinct experts per token, weights that add up to the gate's scale
        score = torch.rand(T, E, generator=gen, device=dev)
        w = torch.softmax(torch.randn(T, k, generator=gen, device=dev), dim=1) * case["scale"]
        state.update(ids=score.topk(k, dim=1).indices.to(torch.int32).contiguous(), w=w.contiguous())
    return state


def run(state):
    layer, x, out, act = state["layer"], state["x"], state["out"], state["act"]
    if state["entry"] == "forward":
        layer.forward(x, out=out, shared_range=state["shared"])
    elif state["entry"] == "routed":
        layer.forward_routed(x, state["ids"], state["w"], out=out, shared_range=state["shared"])
    elif state["entry"] == "static":
        layer.forward_static(x, out=out, shared_range=state["shared"])
    else:
        layer.set_expert_map(state["first"])
        for i, slot in enumerate(state["fill"]):
            layer.load_expert_async(slot, state["new13"][i], state["new2"][i], state["side"])
        layer.forward(x, out=out)
        layer.set_expert_map(state["full"])
        layer.forward(x, out=state["out2"])
        return out.view(act), state["out2"].view(act)
    return out.view(act)


def _batch_work(case, n_local):
    """Bytes and flops of one batch over the first n_local experts: every active expert's weights once, the
    tokens in and out, the router; three products per (token, local expert)."""
    H, I, E, k, T = case["hidden"], case["inter"], case["n_experts"], case["top_k"], case["tokens"]
    es, rs = (2 if case["act"] == "bf16" else 4), (2 if case["router"] == "bf16" else 4)
    # chance that a token takes an expert: k/E, or falling off with the expert's rank
    p = np.arange(1, E + 1, dtype=np.float64) ** -case["zipf"]
    took = 1.0 - (1.0 - p / p.sum()) ** k if case["zipf"] else np.full(E, k / E)
    active = n_local * float(np.mean(1.0 - (1.0 - took) ** T))
    shared_rows = _shared_tokens(case) * case["n_shared"]
    if shared_rows:
        active += case["n_shared"]
    gated = case["entry"] != "routed"
    rows = T * k * n_local / E + shared_rows
    return (active * 3 * H * I * es + 2 * T * H * es + (E * H * rs if gated else 8 * T * k),
            rows * 6 * H * I + (2 * T * H * E if gated else 0))


def work(case):
    b, f = _batch_work(case, case["n_local"])
    if case["entry"] == "relayout":
        half = case["n_local"] // 2
        b1, f1 = _batch_work(case, half)
        b, f = b + b1 + 2 * half * 3 * case["hidden"] * case["inter"] * 2, f + f1   # every filled slot is read and written once
    return {"bytes": b, "flops": f}


def tolerance(case):
    # bf16: the two intermediates and the result are rounded to 8 bits of mantissa; fp32: sums of some hundred terms
    return {"rel": 5e-3, "max": 5e-2} if case["act"] == "bf16" else {"rel": 1e-5, "max": 1e-4}
