"""The workloads this framework's speed is judged on: decode steps of a block-diffusion language model and the
vocabulary projection that ends them, through the public calls of paper_2601_17917_amd.

Two kinds of case:
  step     per layer: (rotary embedding of the query and key rows,) pruned-suffix attention; then the unmask over stored
           logits; (then the append of the block's K/V to every layer's cache).
  project  the unmask fed by the vocabulary projection (sdllm_lm_head_unmask), the logits never stored.
"calls" says how the program makes its calls: "bound" marshals them once and repeats them, as a serving loop over fixed
buffers does; "plain" uses the one-shot functions.  Sizes follow the repository's own workloads (workloads.py) unless
a comment says otherwise; weights and activations are seeded normal draws of the shapes and scales used there.
"""
import math

import torch

import paper_2601_17917_amd as sd

TAU0 = 0.9
THETA = 500000.0
EOS = 2


def _step(name, dtype, B, Hq, Hkv, D, P, K, S, n_keep, V, **more):
    case = {"name": name, "kind": "step", "dtype": dtype, "B": B, "Hq": Hq, "Hkv": Hkv, "D": D, "P": P, "K": K, "S": S,
            "n_keep": n_keep, "keep": "window", "V": V, "layers": 1, "masked_lo": 1.0, "masked_hi": 1.0,
            "boost": False, "alpha": 0.3, "qkv_std": 1.0, "logit_std": 4.0, "rope": False, "interleaved": False,
            "append": False, "calls": "bound"}
    case.update(more)
    return case


def _project(name, B, K, V, Hd, packed, **more):
    case = {"name": name, "kind": "project", "dtype": "bf16", "B": B, "K": K, "V": V, "Hd": Hd, "packed": packed,
            "masked_lo": 1.0, "masked_hi": 1.0, "boost": False, "alpha": 0.3, "logit_std": 4.0, "calls": "bound"}
    case.update(more)
    return case


def listed():
    return [
        # the smallest call: one tiny fp32 layer, as a script that checks its numerics in fp32 makes it
        _step("fp32_small_step", "fp32", 1, 4, 4, 64, 64, 32, 224, 16, 2048, masked_lo=0.5, masked_hi=0.5, alpha=0.0,
              logit_std=3.0, append=True, calls="plain"),
        # the same check on a full-size layer: grouped-query heads, fp32 logits over a generic 32000-entry vocabulary
        _step("fp32_layer_step", "fp32", 2, 32, 8, 128, 608, 32, 128, 32, 32000, boost=True, masked_lo=0.5,
              masked_hi=0.5),
        # interactive use: one sequence, one layer of a 7-8B model with its rotary embedding, half of the block decided
        _step("layer_step_b1", "bf16", 1, 32, 32, 128, 608, 32, 128, 32, 126464, boost=True, masked_lo=0.5,
              masked_hi=0.5, qkv_std=1.0 / math.sqrt(128.0), rope=True),
        # a small batch with the pruned suffix, at the start of a generation (nothing decided, no block finished)
        _step("pruned_step_b8", "bf16", 8, 32, 32, 128, 1024, 32, 992, 32, 126464, alpha=0.0),
        # the same with the whole suffix kept: full-context attention, bound by the matrix cores
        _step("full_suffix_b8", "bf16", 8, 32, 32, 128, 1024, 32, 992, 992, 126464, alpha=0.0),
        # grouped-query heads 7:1, a larger batch whose sequences are at different points of their blocks
        _step("gqa_step_b16", "bf16", 16, 28, 4, 128, 512, 32, 224, 32, 152064, masked_lo=0.1, masked_hi=1.0, rope=True),
        # long context: all 32 layers, then the unmask and the append of the finished block into all 32 caches
        _step("long_context_stack", "bf16", 4, 32, 32, 128, 5120, 64, 960, 64, 126464, layers=32, append=True,
              calls="plain"),
        # block-causal topology (no suffix), grouped-query heads 4:1, a block that finishes and is appended
        _step("block_causal_b8", "bf16", 8, 32, 8, 128, 1248, 32, 0, 0, 152064, boost=True, masked_lo=0.5, masked_hi=0.5,
              append=True),
        # 64-wide heads and sizes that are a multiple of nothing: ragged key tiles, a ragged vocabulary, kept rows
        # scattered over the suffix, two layers
        _step("head64_ragged_b3", "bf16", 3, 16, 4, 64, 1213, 27, 203, 37, 50257, keep="scattered", layers=2, rope=True,
              interleaved=True, masked_lo=0.3, masked_hi=0.9),
        # the projection for one sequence half-way through its block (a read of the weight), packed weight
        _project("projection_b1", 1, 32, 126464, 4096, True, boost=True, masked_lo=0.5, masked_hi=0.5),
        # the projection at the start of a batch of blocks, weight as the checkpoint holds it
        _project("projection_b8", 8, 32, 126464, 4096, False, alpha=0.0),
        # the projection of the larger batch, sequences at different points of their blocks, packed weight
        _project("projection_b16", 16, 32, 152064, 3584, True, masked_lo=0.1, masked_hi=1.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_step(rng):
    fp32 = rng.random() < 0.2
    D = rng.choice([32, 64, 80, 128]) if fp32 else rng.choice([64, 128, 128])
    Hkv = rng.choice([1, 2, 4, 8, 16, 32])
    Hq = Hkv * rng.choice([g for g in (1, 2, 4, 7, 8) if Hkv * g <= 64])
    K = rng.choice([8, 16, 32, 32, 64, 128, rng.randint(5, 100)])
    S = 0 if rng.random() < 0.15 else _log_int(rng, 8, 2048)
    n_keep = rng.choice([S, min(S, K), min(S, _log_int(rng, 8, 1024))])
    case = _step("", "fp32" if fp32 else "bf16", _log_int(rng, 1, 16), Hq, Hkv, D, _log_int(rng, 16, 8192), K, S, n_keep,
                 _log_int(rng, 2000, 152064), keep=rng.choice(["window", "window", "scattered"]),
                 layers=rng.choice([1, 1, 2, 4, 8]), masked_lo=rng.choice([0.1, 0.5, 1.0]), masked_hi=1.0,
                 boost=rng.random() < 0.5, alpha=rng.choice([0.0, 0.3, 0.6]), rope=rng.random() < 0.5,
                 interleaved=rng.random() < 0.3, append=rng.random() < 0.5, calls=rng.choice(["bound", "plain"]))
    del case["name"]
    return case


def _draw_project(rng):
    case = _project("", _log_int(rng, 1, 16), rng.choice([16, 32, 32, 64, rng.randint(5, 60)]),
                    rng.choice([32000, 126464, 152064, _log_int(rng, 8000, 152064)]), 32 * _log_int(rng, 24, 160),
                    rng.random() < 0.5, masked_lo=rng.choice([0.1, 0.5, 1.0]), masked_hi=1.0, boost=rng.random() < 0.5,
                    alpha=rng.choice([0.0, 0.3, 0.6]), calls=rng.choice(["bound", "plain"]))
    del case["name"]
    return case


def draw(rng):
    """One more case of the same ranges: heads 1..64 of width 64 / 128 (fp32: 32..128), batches 1..16, prefixes 16..8192,
    suffixes 0..2048 kept in part or whole, vocabularies 2000..152064, model widths 768..5120."""
    while True:
        case = _draw_step(rng) if rng.random() < 0.7 else _draw_project(rng)
        w = work(case)
        limit = 2e11 if case["dtype"] == "fp32" else 4e11
        if w["bytes"] <= 3e9 and w["flops"] <= limit:
            return case


# ---------------------------------------------------------------------------------------------
def _gen(seed, what):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + what) & 0x7FFFFFFFFFFFFFFF)
    return g


def _normal(seed, what, shape, std, dtype):
    x = torch.randn(shape, generator=_gen(seed, what), device="cuda", dtype=dtype)
    return x.mul_(std) if std != 1.0 else x


def _block_state(case, seed, state):
    """tokens / masked / eos_seen as views of one buffer, and the values a step starts from."""
    B, K, V = case["B"], case["K"], case["V"]
    g = _gen(seed, 1)
    frac = case["masked_lo"] + (case["masked_hi"] - case["masked_lo"]) * torch.rand((B, 1), generator=g, device="cuda")
    count = (frac * K).floor().clamp(1, K)
    order = torch.rand((B, K), generator=g, device="cuda").argsort(1).argsort(1)
    masked = (order < count).to(torch.uint8)
    tokens = torch.randint(0, V, (B, K), generator=g, device="cuda", dtype=torch.int32)
    tokens[masked != 0] = -1
    n = B * K
    fresh = torch.cat([tokens.view(-1).view(torch.uint8), masked.view(-1),
                       torch.zeros((B,), dtype=torch.uint8, device="cuda")])
    live = fresh.clone()
    state["fresh"], state["live"] = fresh, live
    state["tokens"] = live[:4 * n].view(torch.int32).view(B, K)
    state["masked"] = live[4 * n:5 * n].view(B, K)
    state["eos"] = live[5 * n:]
    state["confidence"] = torch.zeros((B, K), dtype=torch.float32, device="cuda")


def _keep_idx(case, seed):
    S, n = case["S"], case["n_keep"]
    if n == 0:
        return None
    if n == S:
        idx = torch.arange(S, device="cuda")
    elif case["keep"] == "window":      # the nearest positions and the trailing one
        idx = torch.arange(n, device="cuda")
        idx[n - 1] = S - 1
    else:
        idx = torch.rand((S,), generator=_gen(seed, 2), device="cuda").argsort()[:n].sort().values
    return idx.to(torch.int32)


def _prepare_step(case, seed):
    dt = torch.float32 if case["dtype"] == "fp32" else torch.bfloat16
    B, Hq, Hkv, D, K, S, L = (case[k] for k in ("B", "Hq", "Hkv", "D", "K", "S", "layers"))
    P, std, cap = case["P"], case["qkv_std"], case["P"] + case["K"] + case["S"]
    s = {"case": case, "keep": _keep_idx(case, seed)}
    some = S > 0 and case["n_keep"] > 0
    s["q_block"] = _normal(seed, 10, (L, B, Hq, K, D), std, dt)
    s["q_suffix"] = _normal(seed, 11, (L, B, Hq, S, D), std, dt) if some else [None] * L
    s["k_caches"] = _normal(seed, 12, (L, B, Hkv, cap, D), std, dt)
    s["v_caches"] = _normal(seed, 13, (L, B, Hkv, cap, D), std, dt)
    s["k_blocks"] = _normal(seed, 14, (L, B, Hkv, K, D), std, dt)
    s["v_blocks"] = _normal(seed, 15, (L, B, Hkv, K, D), std, dt)
    s["k_suffix"] = _normal(seed, 16, (L, B, Hkv, S, D), std, dt) if some else [None] * L
    s["v_suffix"] = _normal(seed, 17, (L, B, Hkv, S, D), std, dt) if some else [None] * L
    for x in ("q", "k"):                # rotated rows go to tensors of their own, so that a pass can be repeated
        heads = "%s_block" % x if x == "q" else "k_blocks"
        s[x + "_rot"] = torch.zeros_like(s[heads]) if case["rope"] else s[heads]
        s[x + "_rot_suffix"] = torch.zeros_like(s[x + "_suffix"]) if case["rope"] and some else s[x + "_suffix"]
    V = case["V"]
    ld = (V + 7) // 8 * 8               # rows of the logits are 16-byte aligned
    s["logits"] = _normal(seed, 18, (B, K, ld), case["logit_std"], dt)
    if case["boost"]:
        g = _gen(seed, 3)
        top = torch.randint(0, V, (B, K, 1), generator=g, device="cuda")
        s["logits"].scatter_(2, top, (18 + 8 * torch.rand((B, K, 1), generator=g, device="cuda")).to(dt))
    _block_state(case, seed, s)
    if case["calls"] == "bound":
        s["bound"] = _step_calls(s, sd.bind_rope_gathered, sd.bind_block_attention, sd.bind_confidence_unmask,
                                 sd.bind_kv_append, P)
    return s


def _step_calls(s, rope, attention, unmask, append, P):
    """The step's calls in order.  With the bind_* functions this marshals them, with the others it makes them."""
    case, keep = s["case"], s["keep"]
    made = {"rope": [], "attention": []}
    for i in range(case["layers"]):
        if case["rope"]:
            for x, src in (("q", "q_block"), ("k", "k_blocks")):
                made["rope"].append(rope(s[src][i], s[x + "_suffix"][i], keep, P, THETA, case["interleaved"],
                                         s[x + "_rot"][i], s[x + "_rot_suffix"][i]))
        made["attention"].append(attention(s["q_rot"][i], s["q_rot_suffix"][i], s["k_caches"][i], s["v_caches"][i],
                                           s["k_rot"][i], s["v_blocks"][i], s["k_rot_suffix"][i], s["v_suffix"][i], keep,
                                           P))
    made["unmask"] = unmask(s["logits"], s["tokens"], s["masked"], TAU0, case["alpha"], V=case["V"],
                            confidence=s["confidence"], eos_seen=s["eos"], eos_id=EOS)
    made["append"] = append(s["k_caches"], s["v_caches"], s["k_rot"], s["v_blocks"], P) if case["append"] else None
    return made


def _run_step(s):
    case = s["case"]
    s["live"].copy_(s["fresh"])
    if case["calls"] == "bound":
        b = s["bound"]
        outs = []
        for i, call in enumerate(b["attention"]):
            for r in b["rope"][2 * i:2 * i + 2]:
                r()
            outs.append(call())
        flags = b["unmask"]()
        if b["append"] is not None:
            b["append"]()
    else:
        made = _step_calls(s, sd.rope_gathered, sd.block_attention, sd.confidence_unmask, sd.kv_append, case["P"])
        outs, flags = made["attention"], made["unmask"]
    out = {"attention": outs, "tokens": s["tokens"], "masked": s["masked"], "eos": s["eos"], "n_committed": flags[0],
           "block_done": flags[1], "confidence": s["confidence"]}
    if case["rope"]:
        out["q_rot"], out["k_rot"] = s["q_rot"], s["k_rot"]
        if s["keep"] is not None:
            out["q_rot_suffix"], out["k_rot_suffix"] = s["q_rot_suffix"], s["k_rot_suffix"]
    if case["append"]:
        out["k_caches"], out["v_caches"] = s["k_caches"], s["v_caches"]
    return out


def _prepare_project(case, seed):
    B, K, V, Hd = case["B"], case["K"], case["V"], case["Hd"]
    s = {"case": case}
    h = _normal(seed, 20, (B, K, Hd), 1.0, torch.bfloat16)
    w = _normal(seed, 21, (V, Hd), case["logit_std"] / math.sqrt(Hd), torch.bfloat16)
    if case["boost"]:                   # one token per position whose logit is U(18, 26)
        g = _gen(seed, 3)
        top = torch.randint(0, V, (B * K,), generator=g, device="cuda")
        hf = h.view(B * K, Hd).float()
        val = 18 + 8 * torch.rand((B * K, 1), generator=g, device="cuda")
        # two positions may draw one token: the sum of both rows is the same in every run
        w[top] = 0
        w.index_put_((top,), (val * hf / (hf * hf).sum(-1, keepdim=True)).to(torch.bfloat16), accumulate=True)
    s["hidden"] = h
    s["weight"] = sd.lm_head_pack_weight(w) if case["packed"] else w
    _block_state(case, seed, s)
    if case["calls"] == "bound":
        s["bound"] = sd.bind_lm_head_unmask(h, s["weight"], s["tokens"], s["masked"], TAU0, case["alpha"],
                                            confidence=s["confidence"], eos_seen=s["eos"], eos_id=EOS)
    return s


def _run_project(s):
    case = s["case"]
    s["live"].copy_(s["fresh"])
    if case["calls"] == "bound":
        flags = s["bound"]()
    else:
        flags = sd.lm_head_unmask(s["hidden"], s["weight"], s["tokens"], s["masked"], TAU0, case["alpha"],
                                  confidence=s["confidence"], eos_seen=s["eos"], eos_id=EOS)
    return {"tokens": s["tokens"], "masked": s["masked"], "eos": s["eos"], "n_committed": flags[0],
            "block_done": flags[1], "confidence": s["confidence"]}


def prepare(case, seed):
    return _prepare_step(case, seed) if case["kind"] == "step" else _prepare_project(case, seed)


def run(state):
    return _run_step(state) if state["case"]["kind"] == "step" else _run_project(state)


def work(case):
    e = 4 if case["dtype"] == "fp32" else 2
    B, K, V = case["B"], case["K"], case["V"]
    rows = B * K * (case["masked_lo"] + case["masked_hi"]) / 2          # masked positions (mean of the law)
    if case["kind"] == "project":
        return {"bytes": V * case["Hd"] * e + rows * case["Hd"] * e, "flops": 2.0 * rows * V * case["Hd"]}
    L, Hq, Hkv, D = case["layers"], case["Hq"], case["Hkv"], case["D"]
    Nq = K + case["n_keep"]
    Nkv = case["P"] + Nq
    by = L * (2 * B * Hkv * Nkv * D * e + 2 * B * Hq * Nq * D * e) + rows * V * e
    if case["rope"]:
        by += L * 2 * B * (Hq + Hkv) * Nq * D * e
    if case["append"]:
        by += 4 * L * B * Hkv * K * D * e
    return {"bytes": float(by), "flops": 4.0 * L * B * Hq * Nq * Nkv * D}


def tolerance(case):
    # About four times what the calls differ by from the same operations in 64 bits (largest of the listed cases):
    # bf16 2.3e-3 (largest 1.7e-2), fp32 6.6e-7 (6e-6), projection 3.9e-6 (1.4e-5).
    # Whole numbers of a step come from stored logits and do not move.  A projection's logits are fp32 sums whose order
    # may differ: two tokens closer than that can trade places.
    if case["kind"] == "project":
        return {"rel": 2e-5, "max": 1e-4, "differ": 0.005}
    if case["dtype"] == "fp32":
        return {"rel": 3e-6, "max": 3e-5}
    return {"rel": 1e-2, "max": 0.07}
