"""The calls whose speed this repository is measured by, through the public entry points of paper_2605_03884_amd.

A case is a dict of plain values: `op` names the path, the rest is its shape and options.

  handoff      sender and receiver: (scores -> widths ->) card -> dense fp16 cache
  handoff_kc   the same for a uniform card whose keys are grouped per channel
  inject       receiver: a card into per-layer caches behind a prefix, in one call or layer by layer, keys realigned or not
  requantize   forwarding agent: new widths for the tokens, card to card
  attend       one decode step of attention directly over a card
  attend_kc    the same over a card with per-channel key groups
  widths       the controller's scores and the objective-following widths

Inputs are made on the GPU from the seed alone: K ~ N(0, 1) with 2 % of the channels of every (layer, head) scaled by
10 .. 50, V ~ N(0, 1) times a per-token scale in [0.5, 4], scores ~ U(0, 1).
"""
import math

import torch

import paper_2605_03884_amd as qkv

WIDTHS = (2, 4, 8, 16)
PREFIX = 64                       # tokens a receiver's own cache holds in front of the injected ones


def _case(op, layers, kv_heads, tokens, head_dim=128, group_size=32, budget=3.0, width=0, rep=0, rope=0, layerwise=False,
          old_budget=0.0, name=None):
    c = dict(op=op, layers=layers, kv_heads=kv_heads, tokens=tokens, head_dim=head_dim, group_size=group_size, budget=budget,
             width=width, rep=rep, rope=rope, layerwise=layerwise, old_budget=old_budget)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest handoff: one layer, two heads, 256 tokens; launches and host work only
        _case("handoff", 1, 2, 256, budget=5.0, name="handoff_tiny"),
        # a short shared context of a Llama-3.1-8B shaped cache at the paper's 30/40/25/5 % mix
        _case("handoff", 32, 8, 1024, budget=5.0, name="handoff_1k_b5"),
        # the headline handoff: 8K tokens at an average of 3 bits
        _case("handoff", 32, 8, 8192, budget=3.0, name="handoff_8k_b3"),
        # one rank of eight in tensor-parallel serving, a full 128K-token context: long token tables, few planes
        _case("handoff", 32, 1, 131072, budget=4.0, name="handoff_128k_shard_b4"),
        # uniform 4-bit card with the keys grouped per channel (per-channel key / per-token value scheme)
        _case("handoff_kc", 32, 8, 8192, width=4, name="handoff_kc_8k_u4"),
        # a receiver that fills its caches layer by layer behind a prefix, keys realigned; 3877 tokens is the paper's nominal 8K
        _case("inject", 32, 8, 3877, budget=4.0, rope=64, layerwise=True, name="inject_layers_3877_rope"),
        # an agent that forwards an 8K card at a lower budget
        _case("requantize", 32, 8, 8192, old_budget=3.0, budget=2.5, name="requantize_8k_b3_b2.5"),
        # the first hop of the 32K multi-hop chain taken card to card
        _case("requantize", 32, 8, 32768, old_budget=6.0, budget=4.0, name="requantize_32k_b6_b4"),
        # one decode step over a short card
        _case("attend", 32, 8, 1024, budget=5.0, rep=4, name="attend_1k_b5"),
        # one decode step over the headline card: 32 query heads on 8 KV heads
        _case("attend", 32, 8, 8192, budget=3.0, rep=4, name="attend_8k_b3"),
        # more query heads per KV head, the smaller head dimension, a ragged length
        _case("attend", 32, 4, 3877, head_dim=64, group_size=64, budget=4.0, rep=8, name="attend_3877_d64_r8"),
        # the controller over 8K tokens: features -> scores -> widths that follow the budgeted objective
        _case("widths", 0, 0, 8192, head_dim=0, group_size=0, budget=4.0, name="widths_8k"),
    ]


def draw(rng):
    def tokens(lo, hi, step=1):
        t = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        return max(step, t // step * step)

    op = rng.choice(["handoff", "handoff", "handoff", "handoff_kc", "inject", "inject", "requantize", "requantize", "attend", "attend",
                     "attend", "attend_kc", "widths"])
    if op == "widths":
        return _case(op, 0, 0, tokens(100, 131072), head_dim=0, group_size=0, budget=round(rng.uniform(2.2, 12.0), 2))
    kc = op.endswith("_kc")
    d = rng.choice([64, 128, 128, 128] if kc else [64, 128, 128, 128, 256])
    g = 32 if kc else rng.choice([x for x in (32, 32, 64, 128) if x <= d])
    heads = rng.choice([1, 2, 4, 8, 8])
    t = tokens(200, 131072 if op == "handoff" else 32768, 64 if kc else 1)
    room = 12 << 20 if op == "requantize" else 6 << 20           # rows of 128 values, keys and values together
    layers = min(rng.choice([1, 8, 16, 24, 32, 32, 48, 64]), max(1, room * 128 // (2 * heads * t * d)))
    uniform = kc or rng.random() < 0.25
    c = _case(op, layers, heads, t, d, g, budget=round(rng.uniform(2.2, 8.0), 2),
              width=rng.choice([2, 4, 4, 8]) if uniform and op != "requantize" else 0)
    if op == "inject":
        c["rope"] = rng.choice([0, 64, -1000, 4096])
        c["layerwise"] = rng.random() < 0.5
    if op == "requantize":
        c["old_budget"] = round(rng.uniform(c["budget"], 8.0), 2)
    if op.startswith("attend"):
        c["rep"] = rng.choice([1, 2, 4, 4, 5, 8, 16])
    return c


# ---- inputs -------------------------------------------------------------------------------------------------------


def _generator(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 1000003 + stream) & ((1 << 62) - 1))
    return g


def _kv(case, seed):
    L, H, T, D = (case[x] for x in ("layers", "kv_heads", "tokens", "head_dim"))
    g = _generator(seed, 1)
    k = torch.randn((L, H, T, D), dtype=torch.float16, device="cuda", generator=g)
    v = torch.randn((L, H, T, D), dtype=torch.float16, device="cuda", generator=g)
    n_out = max(1, math.ceil(0.02 * D))
    ch = torch.rand((L, H, D), device="cuda", generator=g).topk(n_out, dim=-1).indices
    f = 10.0 + 40.0 * torch.rand((L, H, n_out), device="cuda", generator=g)
    factor = torch.ones((L, H, D), device="cuda").scatter_(2, ch, f)
    k.mul_(factor.half().view(L, H, 1, D))
    v.mul_((0.5 * 8.0 ** torch.rand((T,), device="cuda", generator=g)).half().view(1, 1, T, 1))
    return k, v


def _scores(case, seed, stream=2):
    return torch.rand((case["tokens"],), device="cuda", generator=_generator(seed, stream))


def _bits(case, scores, budget):
    """The widths a caller has in hand: uniform, or by rank of the score with the class counts of the budget."""
    T = case["tokens"]
    if case["width"]:
        return torch.full((T,), case["width"], dtype=torch.uint8, device="cuda"), [T * (w == case["width"]) for w in WIDTHS]
    counts = qkv.budget_counts(T, budget)
    by_rank = torch.repeat_interleave(torch.tensor([16, 8, 4, 2], dtype=torch.uint8, device="cuda"),
                                      torch.tensor(counts[::-1], device="cuda"))
    bits = torch.empty((T,), dtype=torch.uint8, device="cuda")
    bits[torch.sort(scores, descending=True, stable=True).indices] = by_rank
    return bits, counts


def _desc(case):
    return qkv.Desc.make(case["layers"], case["kv_heads"], case["tokens"], case["head_dim"], case["group_size"], model_id=1, sender_id=2)


def _card(case, seed, budget):
    k, v = _kv(case, seed)
    bits, counts = _bits(case, _scores(case, seed), budget)
    desc = _desc(case)
    card = torch.empty(qkv.card_bytes(desc, counts), dtype=torch.uint8, device="cuda")
    (qkv.quantize_pack_kc if case["op"].endswith("_kc") else qkv.quantize_pack)(desc, k, v, bits, counts, card)
    return desc, card


def _features(case, seed):
    T, g = case["tokens"], _generator(seed, 3)
    f = torch.rand((T, 6), device="cuda", generator=g)
    seg = torch.randint(0, 3, ((T + 63) // 64,), device="cuda", generator=g).repeat_interleave(64)[:T].float() * 0.5
    f[:, 4] += 0.5 * (seg > 0).float()
    f[:, 5] = seg
    w1 = (torch.randn((64, 6), device="cuda", generator=g) / math.sqrt(6.0)).cpu()
    b1 = (torch.randn((64,), device="cuda", generator=g) * 0.1).cpu()
    w2 = (torch.randn((64,), device="cuda", generator=g) * 0.125).abs().cpu()
    return f, w1, b1, w2


def prepare(case, seed):
    op = case["op"]
    s = {"case": case, "status": torch.zeros(1, dtype=torch.int32, device="cuda")}
    if op == "widths":
        f, w1, b1, w2 = _features(case, seed)
        s.update(features=f, params=qkv.Controller.make(w1, b1, w2), scores=torch.empty(case["tokens"], device="cuda"),
                 bits=torch.empty(case["tokens"], dtype=torch.uint8, device="cuda"),
                 counts=torch.empty(4, dtype=torch.int64, device="cuda"))
        return s
    L, H, T, D = (case[x] for x in ("layers", "kv_heads", "tokens", "head_dim"))
    if op in ("handoff", "handoff_kc"):
        s["desc"] = _desc(case)
        s["k"], s["v"] = _kv(case, seed)
        if case["width"]:
            s["bits"], s["counts"] = _bits(case, None, 0.0)
        else:
            s["scores"] = _scores(case, seed)
            s["bits"] = torch.empty(T, dtype=torch.uint8, device="cuda")
            s["counts"] = qkv.budget_counts(T, case["budget"])
        s["card"] = torch.empty(qkv.card_bytes(s["desc"], s["counts"]), dtype=torch.uint8, device="cuda")
        s["k_out"], s["v_out"] = torch.empty_like(s["k"]), torch.empty_like(s["v"])
        return s
    if op == "requantize":
        s["desc"], s["card"] = _card(case, seed, case["old_budget"])
        s["scores"] = _scores(case, seed, 4)
        s["bits"] = torch.empty(T, dtype=torch.uint8, device="cuda")
        s["card_out"] = torch.empty(qkv.card_bytes(s["desc"], qkv.budget_counts(T, case["budget"])), dtype=torch.uint8, device="cuda")
        return s
    s["desc"], s["card"] = _card(case, seed, case["budget"])
    g = _generator(seed, 5)
    if op == "inject":
        s["k_cache"] = torch.zeros((L, H, PREFIX + T, D), dtype=torch.float16, device="cuda")
        s["v_cache"] = torch.zeros_like(s["k_cache"])
        for x in (s["k_cache"], s["v_cache"]):
            x[:, :, :PREFIX] = torch.randn((L, H, PREFIX, D), device="cuda", generator=g).half()
        s["k_layers"] = [s["k_cache"][l, :, PREFIX:] for l in range(L)]
        s["v_layers"] = [s["v_cache"][l, :, PREFIX:] for l in range(L)]
        return s
    hq = H * case["rep"]
    s["q"] = torch.randn((L, hq, D), device="cuda", generator=g).half()
    s["out"] = torch.empty((L, hq, D), device="cuda")
    s["lse"] = torch.empty((L, hq), device="cuda")
    s["workspace"] = torch.empty(qkv.card_attend_workspace(s["desc"], hq), dtype=torch.uint8, device="cuda")
    return s


# ---- one pass -------------------------------------------------------------------------------------------------------


def run(s):
    case, op = s["case"], s["case"]["op"]
    if op == "widths":
        qkv.controller_scores(s["features"], s["params"], scores=s["scores"])
        qkv.assign_bits_greedy(s["scores"], case["budget"], bits=s["bits"], counts=s["counts"])
        return s["scores"], s["bits"], s["counts"]
    desc, card, status = s["desc"], s["card"], s["status"]
    if op == "handoff":
        if case["width"]:
            qkv.quantize_pack(desc, s["k"], s["v"], s["bits"], s["counts"], card)
        else:
            qkv.assign_quantize_pack(desc, s["k"], s["v"], s["scores"], case["budget"], card, bits=s["bits"])
        qkv.unpack_dequant(card, desc, s["k_out"], s["v_out"], status=status)
        return s["k_out"], s["v_out"], card, s["bits"], status
    if op == "handoff_kc":
        qkv.quantize_pack_kc(desc, s["k"], s["v"], s["bits"], s["counts"], card)
        qkv.unpack_dequant_kc(card, desc, s["k_out"], s["v_out"], status=status)
        return s["k_out"], s["v_out"], card, status
    if op == "inject":
        base = 500000.0 if case["rope"] else 0.0
        if case["layerwise"]:
            for l in range(case["layers"]):
                qkv.inject_layers(card, desc, s["k_layers"][l:l + 1], s["v_layers"][l:l + 1], l, rope_base=base, rope_delta=case["rope"],
                                  status=status if l == 0 else None)
        else:
            qkv.inject_layers(card, desc, s["k_layers"], s["v_layers"], 0, rope_base=base, rope_delta=case["rope"], status=status)
        return s["k_cache"], s["v_cache"], status
    if op == "requantize":
        _, counts = qkv.assign_bits(s["scores"], case["budget"], bits=s["bits"])
        qkv.requantize(card, desc, s["bits"], counts, s["card_out"], status=status)
        return s["card_out"], s["bits"], status
    attend = qkv.card_attend if op == "attend" else qkv.card_attend_kc
    attend(card, desc, s["q"], case["head_dim"] ** -0.5, s["out"], lse=s["lse"], workspace=s["workspace"], status=status)
    return s["out"], s["lse"], status


# ---- what a pass cannot do without ----------------------------------------------------------------------------------


def _card_size(case, budget):
    T, P, D = case["tokens"], 2 * case["layers"] * case["kv_heads"], case["head_dim"]
    counts = [T * (w == case["width"]) for w in WIDTHS] if case["width"] else qkv.budget_counts(T, budget)
    rows = sum(n * (D * w // 8 + (0 if w == 16 else 4 * (D // case["group_size"]))) for n, w in zip(counts, WIDTHS))
    return P * rows + 9 * T


def work(case):
    op, T = case["op"], case["tokens"]
    if op == "widths":
        return {"bytes": T * (24 + 4 + 1), "flops": T * 2 * (6 * 64 + 64)}
    values = 2 * case["layers"] * case["kv_heads"] * T * case["head_dim"]
    if op == "requantize":                              # old card in, new card out; decode and quantize every value
        return {"bytes": _card_size(case, case["old_budget"]) + _card_size(case, case["budget"]) + 5 * T, "flops": 7 * values}
    card = _card_size(case, case["budget"])
    if op in ("handoff", "handoff_kc"):                 # cache in, card out, card in, cache out
        return {"bytes": 4 * values + 2 * card + 5 * T, "flops": 7 * values}
    if op == "inject":
        return {"bytes": 2 * values + card, "flops": 2 * values + (1.5 * values if case["rope"] else 0)}
    hq = case["layers"] * case["kv_heads"] * case["rep"]
    return {"bytes": card - 8 * T + hq * (case["head_dim"] * 6 + 4), "flops": 4 * hq * T * case["head_dim"]}


def tolerance(case):
    # Cards, widths and rebuilt caches are defined to the bit (roundings and their order are part of the format), so are the
    # controller's scores (the order of its sums is part of the definition).
    if not case["op"].startswith("attend"):
        return "exact"
    # fp32 sums of exact fp16 products, hardware 2^x: 5e-7 .. 9e-7 from 64 bits over the ranges, about five times that
    return {"rel": 5e-6, "max": 5e-5}


# ---- the same in 64 bits --------------------------------------------------------------------------------------------


def _dequantized(x, bits, group, per_channel=False):
    """What a card's reader gets for x [heads, tokens, head_dim] at the tokens' widths, before its last rounding (float64)."""
    H, T, D = x.shape
    out = x.double()
    for w in (2, 4, 8):
        at = (bits == w).nonzero().flatten()
        if not len(at):
            continue
        rows = x[:, at]
        if per_channel:                                 # 32 tokens of one channel form a group; the card is uniform
            rows = rows.view(H, T // 32, 32, D).transpose(2, 3).contiguous()
        grouped = rows.reshape(-1, group).float()
        mn, mx = grouped.amin(1, keepdim=True), grouped.amax(1, keepdim=True)
        scale = ((mx - mn) / torch.full_like(mx, 2 ** w - 1)).half().float()      # a tensor: dividing by a number multiplies by its inverse
        inv = torch.where(scale > 0, 1.0 / scale, torch.zeros_like(scale))
        code = torch.round((grouped - mn).double() * inv.double()).clamp(max=2 ** w - 1)
        value = code * scale.double() + mn.double()
        if per_channel:
            value = value.view(H, T // 32, D, 32).transpose(2, 3).reshape(H, T, D)
        out[:, at] = value.reshape(H, len(at), D)
    return out


def exact(case, seed):
    op, T, D = case["op"], case["tokens"], case["head_dim"]
    if op == "requantize":
        return None                                     # bytes only
    if op == "widths":
        f, w1, b1, w2 = _features(case, seed)
        hidden = torch.relu(f.double() @ w1.double().cuda().t().contiguous() + b1.double().cuda())
        return hidden @ w2.double().cuda(), None, None
    k, v = _kv(case, seed)
    bits, _ = _bits(case, _scores(case, seed), case["budget"])
    L, H, G, kc = case["layers"], case["kv_heads"], case["group_size"], op.endswith("_kc")
    if op.startswith("attend"):
        rep, scale = case["rep"], D ** -0.5
        q = torch.randn((L, H * rep, D), device="cuda", generator=_generator(seed, 5)).half().double().view(L, H, rep, D)
        outs, lses = [], []
        for l in range(L):
            kd = _dequantized(k[l], bits, G, kc).float().half().double()
            vd = _dequantized(v[l], bits, G).float().half().double()
            sc = torch.matmul(kd, q[l].transpose(1, 2).contiguous()) * scale            # [H, T, rep]
            lses.append(torch.logsumexp(sc, dim=1))
            p = torch.softmax(sc, dim=1).transpose(1, 2).contiguous()
            outs.append(torch.matmul(p, vd))
        return torch.stack(outs).view(L, H * rep, D), torch.stack(lses).view(L, H * rep), None
    k_out = torch.stack([_dequantized(k[l], bits, G, kc) for l in range(L)])
    v_out = torch.stack([_dequantized(v[l], bits, G) for l in range(L)])
    if op != "inject":
        return (k_out, v_out, None, None, None) if op == "handoff" else (k_out, v_out, None, None)
    if case["rope"]:
        half = D // 2
        angle = case["rope"] * 500000.0 ** (-2.0 * torch.arange(half, dtype=torch.float64, device="cuda") / D)
        a, b = k_out[..., :half], k_out[..., half:]
        k_out = torch.cat([a * angle.cos() - b * angle.sin(), b * angle.cos() + a * angle.sin()], dim=-1)
    g = _generator(seed, 5)
    prefix = [torch.randn((L, H, PREFIX, D), device="cuda", generator=g).half().double() for _ in range(2)]
    return torch.cat([prefix[0], k_out], dim=2), torch.cat([prefix[1], v_out], dim=2), None
