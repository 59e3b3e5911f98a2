"""The work that a rollout-and-update loop has this library do, as cases that can be timed and compared.

One case is one call (or the few calls that belong together) of a training loop of the GRPO kind: the decode
attention of one layer for all live trajectories, the transition before it, the prompt's prefill, the statistics
of the sampled tokens, and the advantages and the policy loss.  The listed shapes are the repository's own
workloads; `draw` spreads over the ranges around them.

A decode loop keeps its buffers from step to step, so `prepare` lays out the descriptors that such a program
keeps and `run` enqueues them; the calls that come once per batch are made through the tensor functions.
Lengths are a fixed set per case (the quantiles of its distribution), dealt out anew by every seed, so that the
work of a case does not depend on the seed.
"""
from __future__ import annotations

import math
from statistics import NormalDist

import numpy as np
import torch

VOCAB = 151936                                  # the vocabulary of the benchmark's token statistics


# ---------------------------------------------------------------- the cases
def _decode(name, P, G, Hq, Hkv, d, dtype, Lp, Ls, plen="const", slen="uniform", median=0, page=0, finished=0.0,
            append=False):
    c = dict(kind="decode", P=P, G=G, Hq=Hq, Hkv=Hkv, d=d, dtype=dtype, Lp=Lp, Ls=Ls, plen=plen, slen=slen,
             median=median, page=page, finished=finished, append=append)
    return dict(name=name, **c) if name else c


def _tree(name, B, Hq, Hkv, group0, cap0, group1, cap1, Ls, median):
    c = dict(kind="tree", B=B, Hq=Hq, Hkv=Hkv, group0=group0, cap0=cap0, group1=group1, cap1=cap1, Ls=Ls, median=median)
    return dict(name=name, **c) if name else c


def _prefill(name, P, Hq, Hkv, L, plen):
    c = dict(kind="prefill", P=P, Hq=Hq, Hkv=Hkv, L=L, plen=plen)
    return dict(name=name, **c) if name else c


def _stats(name, rows, vocab, dtype, ref):
    c = dict(kind="stats", rows=rows, vocab=vocab, dtype=dtype, ref=ref)
    return dict(name=name, **c) if name else c


def _loss(name, P, G, T, agg, terms):
    c = dict(kind="loss", P=P, G=G, T=T, agg=agg, terms=terms)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # a check run on one prompt in fp32: the smallest call, one launch
        _decode("tiny_f32", 1, 4, 2, 1, 64, "f32", 64, 32),
        # a small rollout (3B-shaped policy, 8 prompts x 8): latency of two launches
        _decode("vlm3b", 8, 8, 16, 2, 128, "bf16", 452, 512),
        # the benchmark's rollout step (7B-shaped policy, 32 prompts x 8)
        _decode("vlm7b", 32, 8, 28, 4, 128, "bf16", 1280, 2048),
        # the same step on 8-bit K/V stores
        _decode("vlm7b_e4m3", 32, 8, 28, 4, 128, "e4m3", 1280, 2048),
        # many prompts, groups of 16, short answers: KV groups of 128 query rows
        _decode("highbatch", 128, 16, 16, 2, 128, "bf16", 640, 1024, slen="lognormal", median=200),
        # multi-turn prompts on a paged store, a quarter of the trajectories finished: the whole step of a layer,
        # transition (rotary embedding, K/V append) and attention
        _decode("agentic_paged_step", 16, 8, 28, 4, 128, "bf16", 1344, 4096, plen="agentic", slen="lognormal",
                median=300, page=64, finished=0.25, append=True),
        # a policy with heads of 64 columns (the other head dimension the calls take)
        _decode("heads_of_64", 32, 8, 14, 2, 64, "bf16", 452, 1024),
        # two levels of shared segments: a prompt shared by 8, a first turn shared by 2
        _tree("tree_two_levels", 128, 28, 4, 8, 1344, 2, 512, 4096, 300),
        # the prompts' own pass, once per prompt: the benchmark's 32 prompts
        _prefill("prefill_vlm7b", 32, 28, 4, 1280, "const"),
        # the same for a few ragged prompts
        _prefill("prefill_ragged", 8, 16, 2, 452, "uniform"),
        # log-probs, entropy and KL to the reference policy for one micro-batch of the update
        _stats("token_stats", 4096, VOCAB, "bf16", True),
        # advantages and the clipped loss with its gradient for one batch of answers
        _loss("advantage_and_loss", 512, 8, 4096, "token", True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode"] * 5 + ["tree", "prefill", "prefill", "stats", "loss"])
    if kind == "decode":
        dtype = rng.choice(["bf16", "bf16", "bf16", "e4m3", "f32"])
        d = 64 if dtype == "f32" else rng.choice([128, 128, 128, 64])
        while True:
            P, G = _log_int(rng, 1, 128), rng.choice([1, 4, 5, 8, 8, 16])
            Hkv, r = rng.choice([1, 2, 4, 8]), rng.choice([1, 2, 4, 5, 7, 8])
            Lp, Ls = _log_int(rng, 24, 4096), _log_int(rng, 16, 4096)
            rows = P * Lp + P * G * Ls / 2                       # keys read once
            per_head = P * G * r * (Lp + Ls / 2)                 # keys times the query heads that meet them
            stores = (P * Lp + P * G * (Ls + 64)) * Hkv * d * 4
            if dtype == "f32" and (per_head * Hkv > 2e6 or P > 8):
                continue
            if d == 64 and (per_head * Hkv > (2e6 if dtype == "e4m3" else 4e6) or Lp + Ls > 2500):
                continue
            if rows * Hkv * d * 4 <= 1.2e9 and stores <= 8e9 and G * r <= 256:
                break
        slen = rng.choice(["uniform", "lognormal"])
        page = rng.choice([0, 0, 32, 64, 128]) if dtype != "f32" else 0
        return _decode("", P, G, Hkv * r, Hkv, d, dtype, Lp, Ls, plen=rng.choice(["const", "uniform"]), slen=slen,
                       median=max(1, Ls // 5) if slen == "lognormal" else 0, page=page,
                       finished=rng.choice([0.0, 0.25, 0.5]) if page else 0.0,
                       append=bool(page) and rng.random() < 0.5)
    if kind == "tree":
        Hkv, r = rng.choice([1, 2, 4]), rng.choice([2, 4, 7, 8])
        group1, ratio = rng.choice([1, 2, 4]), rng.choice([2, 2, 4])
        group0 = min(group1 * ratio, 8)
        B = group0 * _log_int(rng, 1, 24)
        return _tree("", B, Hkv * r, Hkv, group0, _log_int(rng, 32, 2048), group1, _log_int(rng, 16, 1024),
                     _log_int(rng, 64, 4096), _log_int(rng, 16, 500))
    if kind == "prefill":
        Hkv, r = rng.choice([1, 2, 4, 8]), rng.choice([1, 2, 4, 5, 7, 8])
        while True:
            P, L = _log_int(rng, 1, 32), _log_int(rng, 48, 4096)
            if P * L * L * Hkv * r <= 32 * 1280 * 1280 * 28 and P * L * Hkv * r <= 32 * 1280 * 28:
                break
        return _prefill("", P, Hkv * r, Hkv, L, rng.choice(["const", "uniform"]))
    if kind == "stats":
        dtype = rng.choice(["bf16", "bf16", "f32"])
        vocab = rng.choice([VOCAB, VOCAB, 32000, rng.randrange(30000, 60000)])   # odd ones as views of padded rows
        return _stats("", _log_int(rng, 16, 4096 if dtype == "bf16" else 2048), vocab, dtype, rng.random() < 0.5)
    return _loss("", _log_int(rng, 2, 512), rng.choice([4, 8, 16]), _log_int(rng, 64, 4096 if rng.random() < 0.5 else 1000),
                 rng.choice(["token", "seq"]), rng.random() < 0.7)


# ---------------------------------------------------------------- lengths
def _quantiles(kind, n, cap, median=0):
    """n lengths: the quantiles of their distribution, in increasing order."""
    u = (np.arange(n) + 0.5) / max(n, 1)
    if kind == "const":
        x = np.full(n, cap)
    elif kind == "uniform":                                      # 0 .. cap
        x = np.floor(u * (cap + 1))
    elif kind == "lognormal":                                    # median * exp(z), cut at the capacity
        x = np.rint([median * math.exp(NormalDist().inv_cdf(v)) for v in u])
    elif kind == "agentic":                                      # three images and their turns: cap - 384 .. cap
        x = cap - 384 + np.rint(u * 384)
    else:
        raise ValueError(kind)
    return np.clip(x, 0, cap).astype(np.int32)


def _prompt_lens(c):
    x = _quantiles(c["plen"], c["P"], c["Lp"])
    return np.maximum(x, c["Lp"] // 2) if c["plen"] == "uniform" else x


def _dealt(lens, seed, which):
    return np.random.default_rng([seed, which]).permutation(lens).astype(np.int32)


# ---------------------------------------------------------------- inputs
def _gen(seed, which):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1009 + which)
    return g


def _normal(shape, dtype, seed, which, gain=1.0):
    out = torch.empty(shape, dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device="cuda")
    g, flat = _gen(seed, which), out.view(-1)
    for lo in range(0, flat.numel(), 1 << 26):
        x = torch.randn(min(1 << 26, flat.numel() - lo), generator=g, device="cuda")
        flat[lo:lo + x.numel()] = x * gain if gain != 1.0 else x
    return out


def _kv(shape, dtype, seed, which):
    """A K or V store; e4m3: its bytes and the factor per KV head (dimension 1 of every store)."""
    if dtype != "e4m3":
        return _normal(shape, dtype, seed, which), None
    out = torch.empty(shape, dtype=torch.uint8, device="cuda")
    # N(0, 1) by a per-head factor of about max / 448, as a serving engine's quantiser leaves it
    fac = (5.0 + torch.rand(shape[1], generator=_gen(seed, 90), device="cuda")) / 448.0
    g = _gen(seed, which)
    step = max(1, (1 << 26) // max(1, shape[1] * shape[2] * shape[3]))
    inv = (1.0 / fac).view(1, -1, 1, 1)
    for i in range(0, shape[0], step):
        x = torch.randn((min(step, shape[0] - i),) + tuple(shape[1:]), generator=g, device="cuda")
        out[i:i + x.shape[0]] = (x * inv).clamp_(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
    return out, fac


def _lens(x):
    return torch.from_numpy(x).cuda()


def _sections(d):
    return (16, 24, 24) if d == 128 else (8, 12, 12)


def prepare(case, seed):
    return {"decode": _prepare_decode, "tree": _prepare_tree, "prefill": _prepare_prefill, "stats": _prepare_stats,
            "loss": _prepare_loss}[case["kind"]](case, seed)


def _decode_inputs(c, seed):
    """Everything of a decode case that comes from the seed."""
    P, G, Hq, Hkv, d, dt = (c[k] for k in ("P", "G", "Hq", "Hkv", "d", "dtype"))
    B, qt = P * G, "f32" if dt == "f32" else "bf16"
    s = {"c": c, "plens": _lens(_dealt(_prompt_lens(c), seed, 1))}
    slens = _dealt(_quantiles(c["slen"], B, c["Ls"], c["median"]), seed, 2)
    s["slens"] = _lens(slens)
    s["q"] = _normal((B, Hq, d), qt, seed, 3, 2.0)
    s["kp"], s["kfac"] = _kv((P, Hkv, c["Lp"], d), dt, seed, 4)
    s["vp"], s["vfac"] = _kv((P, Hkv, c["Lp"], d), dt, seed, 5)
    if c["page"]:
        ps = c["page"]
        per = (slens + ps) // ps                                 # pages of each sequence, with room for the next token
        n, width = int(per.sum()), -(-(c["Ls"] + 1) // ps)
        ids = np.random.default_rng([seed, 6]).permutation(n).astype(np.int32)
        table = np.full((B, width), -1, np.int32)
        at = 0
        for b in range(B):
            table[b, :per[b]] = ids[at:at + per[b]]
            at += per[b]
        s["table"] = _lens(table)
        s["ks"], _ = _kv((n, Hkv, ps, d), dt, seed, 7)
        s["vs"], _ = _kv((n, Hkv, ps, d), dt, seed, 8)
        act = np.ones(B, np.uint8)
        act[:int(c["finished"] * B)] = 0
        s["active"] = _lens(np.random.default_rng([seed, 9]).permutation(act))
    else:
        s["ks"], _ = _kv((B, Hkv, c["Ls"], d), dt, seed, 7)
        s["vs"], _ = _kv((B, Hkv, c["Ls"], d), dt, seed, 8)
    if c["append"]:
        s["k_new"], s["v_new"] = _normal((B, Hkv, d), qt, seed, 10), _normal((B, Hkv, d), qt, seed, 11)
        pos = s["plens"].repeat_interleave(G) + s["slens"]
        s["pos"] = torch.stack([pos, pos, pos]).to(torch.int32).contiguous()
        s["inv_freq"] = (1e6 ** (-torch.arange(0, d, 2, dtype=torch.float64) / d)).float().cuda()
    return s


def _prepare_decode(c, seed):
    from paper_2512_21450_amd import binding as lib
    s = _decode_inputs(c, seed)
    B, scale = c["P"] * c["G"], 1.0 / math.sqrt(c["d"])
    s["out"] = torch.zeros((B, c["Hq"], c["d"]), dtype=torch.float32, device="cuda")
    s["lse"] = torch.zeros((B, c["Hq"]), dtype=torch.float32, device="cuda")
    q, lens = s["q"], s["slens"]
    if c["append"]:                                              # the step's own copies: rotated in place, counted up
        s["q_step"], s["lens_step"] = q.clone(), lens.clone()
        q, lens = s["q_step"], s["lens_step"]
        s["append"] = lib.kv_append_desc_from_tensors(q, s["k_new"], s["v_new"], s["pos"], s["inv_freq"],
                                                      _sections(c["d"]), s["ks"], s["vs"], lens, s["table"],
                                                      s["active"], s["kfac"], s["vfac"])
    if c["page"]:
        s["desc"] = lib.paged_desc_from_tensors(q, s["kp"], s["vp"], s["plens"], s["ks"], s["vs"], s["table"], lens,
                                                scale, c["G"], s["out"], s["lse"], s["active"], k_scale=s["kfac"],
                                                v_scale=s["vfac"])
        need = lib.rl_decode_attn_paged_workspace_bytes(s["desc"])
    else:
        s["desc"] = lib.desc_from_tensors(q, s["kp"], s["vp"], s["plens"], s["ks"], s["vs"], lens, scale, c["G"],
                                          s["out"], s["lse"], k_scale=s["kfac"], v_scale=s["vfac"])
        need = lib.rl_decode_attn_workspace_bytes(s["desc"])
    s["ws"] = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
    s["desc"].workspace, s["desc"].workspace_bytes = s["ws"].data_ptr(), s["ws"].numel()
    return s


def _tree_inputs(c, seed):
    B, Hq, Hkv, d = c["B"], c["Hq"], c["Hkv"], 128
    s = {"c": c, "q": _normal((B, Hq, d), "bf16", seed, 3, 2.0), "levels": []}
    for l in (0, 1):
        n, cap = B // c["group%d" % l], c["cap%d" % l]
        lens = _quantiles("agentic" if l == 0 and cap > 768 else "uniform", n, cap)
        s["levels"].append((_normal((n, Hkv, cap, d), "bf16", seed, 20 + l), _normal((n, Hkv, cap, d), "bf16", seed, 30 + l),
                            _lens(_dealt(lens, seed, 40 + l)), c["group%d" % l]))
    s["ks"], s["vs"] = _normal((B, Hkv, c["Ls"], d), "bf16", seed, 7), _normal((B, Hkv, c["Ls"], d), "bf16", seed, 8)
    s["slens"] = _lens(_dealt(_quantiles("lognormal", B, c["Ls"], c["median"]), seed, 2))
    return s


def _prepare_tree(c, seed):
    from paper_2512_21450_amd import binding as lib
    s = _tree_inputs(c, seed)
    s["out"] = torch.zeros((c["B"], c["Hq"], 128), dtype=torch.float32, device="cuda")
    s["lse"] = torch.zeros((c["B"], c["Hq"]), dtype=torch.float32, device="cuda")
    s["desc"] = lib.tree_desc_from_tensors(s["q"], s["levels"], s["ks"], s["vs"], s["slens"], 1.0 / math.sqrt(128),
                                           s["out"], s["lse"])
    s["ws"] = torch.empty(max(lib.rl_decode_attn_tree_workspace_bytes(s["desc"]), 256), dtype=torch.uint8, device="cuda")
    s["desc"].workspace, s["desc"].workspace_bytes = s["ws"].data_ptr(), s["ws"].numel()
    return s


def _prefill_lens(c):
    x = _quantiles(c["plen"], c["P"], c["L"])
    return np.maximum(x, c["L"] // 2) if c["plen"] == "uniform" else x


def _prepare_prefill(c, seed):
    P, Hq, Hkv, L, d = c["P"], c["Hq"], c["Hkv"], c["L"], 128
    return {"c": c, "q": _normal((P, L, Hq, d), "bf16", seed, 3), "k": _normal((P, Hkv, L, d), "bf16", seed, 4),
            "v": _normal((P, Hkv, L, d), "bf16", seed, 5), "lens": _lens(_dealt(_prefill_lens(c), seed, 1)),
            "out": torch.zeros((P, L, Hq, d), dtype=torch.float32, device="cuda"),
            "lse": torch.zeros((P, L, Hq), dtype=torch.float32, device="cuda")}


def _prepare_stats(c, seed):
    n, V = c["rows"], c["vocab"]
    wide = -(-V // 8) * 8                                        # rows start on 16 bytes
    s = {"c": c, "logits": _normal((n, wide), c["dtype"], seed, 3, 3.0)[:, :V], "ref": None}
    if c["ref"]:
        s["ref"] = _normal((n, wide), c["dtype"], seed, 4, 0.3)[:, :V]
        for lo in range(0, n, 256):
            s["ref"][lo:lo + 256] += s["logits"][lo:lo + 256]
    ids = torch.randint(0, V, (n,), generator=_gen(seed, 5), device="cuda", dtype=torch.int32)
    ids[::10] = s["logits"][::10].argmax(dim=1).to(torch.int32)
    s["ids"] = ids
    return s


def _prepare_loss(c, seed):
    P, G, T = c["P"], c["G"], c["T"]
    B = P * G
    s = {"c": c, "lens": _lens(_dealt(_quantiles("lognormal", B, T, max(1, T // 3)), seed, 2))}
    uni = lambda which, shape=(B, T): torch.rand(shape, generator=_gen(seed, which), device="cuda")
    s["logprob"] = -3.0 * uni(3).square()
    s["old"] = s["logprob"] + 0.1 * torch.randn((B, T), generator=_gen(seed, 4), device="cuda")
    s["kl"] = 0.05 * uni(5) if c["terms"] else None
    s["entropy"] = 2.0 * uni(6) if c["terms"] else None
    # a right-or-wrong reward and a format reward, as rule-based scoring gives them
    s["metrics"] = torch.stack([(uni(7, (B,)) < 0.4).float(), uni(8, (B,))]).contiguous()
    s["weights"] = torch.tensor([0.9, 0.1], device="cuda")
    return s


# ---------------------------------------------------------------- one pass
def run(s):
    from paper_2512_21450_amd import binding as lib
    c = s["c"]
    if c["kind"] == "decode":
        stream = torch.cuda.current_stream().cuda_stream
        if c["append"]:
            s["q_step"].copy_(s["q"])                            # the projection's output and the batch's lengths of this step
            s["lens_step"].copy_(s["slens"])
            _ok(lib, lib.rl_kv_append_rope_raw(s["append"], stream))
        _ok(lib, lib.rl_decode_attn_paged_raw(s["desc"], stream) if c["page"] else lib.rl_decode_attn_raw(s["desc"], stream))
        if c["append"]:
            return {"out": s["out"], "lse": s["lse"], "q": s["q_step"], "lens": s["lens_step"], "k": s["ks"], "v": s["vs"]}
        return {"out": s["out"], "lse": s["lse"]}
    if c["kind"] == "tree":
        _ok(lib, lib.rl_decode_attn_tree_raw(s["desc"], torch.cuda.current_stream().cuda_stream))
        return {"out": s["out"], "lse": s["lse"]}
    if c["kind"] == "prefill":
        out, lse = lib.rl_prefill_attn(s["q"], s["k"], s["v"], s["lens"], 1.0 / math.sqrt(128), s["out"], s["lse"])
        return {"out": out, "lse": lse}
    if c["kind"] == "stats":
        return lib.rl_token_logprob(s["logits"], s["ids"], 1.0, s["ref"])
    rewards, adv = lib.rl_group_advantage(s["metrics"], s["weights"], c["G"])
    stats, grad = lib.rl_policy_loss(s["logprob"], s["old"], adv, s["lens"], 0.2, 0.28, s["kl"], s["entropy"], 0.01, 0.001,
                                     agg=lib.RL_AGG_TOKEN_MEAN if c["agg"] == "token" else lib.RL_AGG_SEQ_MEAN)
    return {"rewards": rewards, "advantages": adv, "stats": stats, "grad": grad}


def _ok(lib, rc):
    if rc != lib.RLDA_OK:
        raise lib.RldaError(rc)


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    c = case
    if c["kind"] == "decode":
        P, G, Hq, Hkv, d = (c[k] for k in ("P", "G", "Hq", "Hkv", "d"))
        B = P * G
        e = {"f32": 4, "bf16": 2, "e4m3": 1}[c["dtype"]]
        live = B - int(c["finished"] * B)
        kp = float(_prompt_lens(c).sum())
        ks = float(_quantiles(c["slen"], B, c["Ls"], c["median"]).sum()) * live / B + (live if c["append"] else 0)
        io = B * Hq * (d * ((4 if e == 4 else 2) + 4) + 4) + 4 * (P + B)
        step = B * (Hq + 4 * Hkv) * d * 2 + live * Hkv * d * 2 if c["append"] else 0
        return {"bytes": (kp + ks) * Hkv * d * 2 * e + io + step,
                "flops": 4.0 * d * Hq * (kp * G * live / B + ks)}
    if c["kind"] == "tree":
        B, Hq, Hkv, d = c["B"], c["Hq"], c["Hkv"], 128
        n = [float(_quantiles("agentic" if l == 0 and c["cap%d" % l] > 768 else "uniform", B // c["group%d" % l], c["cap%d" % l]).sum())
             for l in (0, 1)]
        ks = float(_quantiles("lognormal", B, c["Ls"], c["median"]).sum())
        return {"bytes": (n[0] + n[1] + ks) * Hkv * d * 4 + B * Hq * (d * 6 + 4),
                "flops": 4.0 * d * Hq * (n[0] * c["group0"] + n[1] * c["group1"] + ks)}
    if c["kind"] == "prefill":
        x = _prefill_lens(c).astype(np.float64)
        rows, pairs = float(x.sum()), float((x * (x + 1) / 2).sum())
        return {"bytes": rows * 128 * (c["Hq"] * 6 + c["Hkv"] * 4) + rows * c["Hq"] * 4, "flops": 4.0 * 128 * c["Hq"] * pairs}
    if c["kind"] == "stats":
        e, m = 4 if c["dtype"] == "f32" else 2, 2 if c["ref"] else 1
        return {"bytes": float(c["rows"]) * c["vocab"] * e * m + c["rows"] * 4 * (6 if c["ref"] else 4),
                "flops": 4.0 * c["rows"] * c["vocab"] * m}
    B = c["P"] * c["G"]
    tokens = float(_quantiles("lognormal", B, c["T"], max(1, c["T"] // 3)).sum())
    return {"bytes": tokens * 4 * (4 if c["terms"] else 2) + B * c["T"] * 4.0 + B * 4 * 5, "flops": 12.0 * tokens}


# Relative errors measured against 64 bits over the listed cases and draws, about four times the largest seen.
# Decode at 128 columns and prefill hold the softmax weights in 16 bits; at 64 columns everything is 32-bit, unless
# the step also returns its rotated query (16 bits).  The KL of two close distributions cancels.
def tolerance(case):
    k = case["kind"]
    if k == "decode" and case["d"] == 64 and not case["append"]:
        return {"rel": 3e-6, "max": 1e-4}
    if k in ("decode", "tree", "prefill"):
        return {"rel": 6e-3, "max": 0.1}
    if k == "stats":
        return {"rel": 2e-4, "max": 4e-3}
    return {"rel": 1e-5, "max": 1e-3}


# ---------------------------------------------------------------- the same in 64 bits
def exact(case, seed):
    with torch.no_grad():
        return {"decode": _exact_decode, "tree": _exact_tree, "prefill": _exact_prefill, "stats": _exact_stats,
                "loss": _exact_loss}[case["kind"]](case, seed)


def _wide(t, fac=None):
    """A store's values in 64 bits; fac: the factor per KV head, dimension -3 of `t`."""
    if t.dtype == torch.uint8:
        t = t.view(torch.float8_e4m3fn).float()
    t = t.double()
    return t if fac is None else t * fac.double().view(-1, 1, 1)


def _attend(q, ks, vs, scale):
    """q [Hq, d] over the keys ks / vs (lists of [Hkv, n, d]): out [Hq, d], lse [Hq]."""
    Hq, d = q.shape
    k, v = torch.cat(ks, 1), torch.cat(vs, 1)
    if k.shape[1] == 0:
        return torch.zeros_like(q), torch.full((Hq,), -math.inf, dtype=torch.float64, device=q.device)
    qg = q.view(k.shape[0], -1, d)
    s = torch.matmul(qg, k.transpose(1, 2).contiguous()) * scale
    lse = torch.logsumexp(s, -1)
    return torch.matmul(torch.exp(s - lse[..., None]), v).reshape(Hq, d), lse.reshape(Hq)


def _rotate(x, ang):
    """The rotary embedding in the rotate-half pairing; x [B, H, d], ang [B, d / 2]."""
    h = x.shape[-1] // 2
    c, s = ang.cos()[:, None], ang.sin()[:, None]
    return torch.cat([x[..., :h] * c - x[..., h:] * s, x[..., h:] * c + x[..., :h] * s], -1)


def _exact_decode(c, seed):
    s = _decode_inputs(c, seed)
    P, G, d = c["P"], c["G"], c["d"]
    B, scale = P * G, 1.0 / math.sqrt(d)
    q, lens = s["q"].double(), s["slens"].clone()
    active = s.get("active")
    act = [True] * B if active is None else [bool(a) for a in active.tolist()]
    table = s["table"].long() if c["page"] else None
    ps = c["page"]
    more = {}
    if c["append"]:
        ang = s["pos"][0].double()[:, None] * s["inv_freq"].double()
        q = _rotate(q, ang)
        k_new, v_new = _rotate(s["k_new"].double(), ang), s["v_new"].double()
        for b, n in enumerate(lens.tolist()):
            if act[b]:
                pg = int(table[b, n // ps])
                for store, new, fac in ((s["ks"], k_new, s["kfac"]), (s["vs"], v_new, s["vfac"])):
                    row = new[b] if fac is None else new[b] / fac.double()[:, None]
                    if store.dtype == torch.uint8:               # what the store holds is rounded to its type
                        store[pg, :, n % ps] = row.float().clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
                    else:
                        store[pg, :, n % ps] = row.to(store.dtype)
                lens[b] += 1
        whole = lambda t: None if t.dtype == torch.uint8 else t.double()
        more = {"q": q, "lens": None, "k": whole(s["ks"]), "v": whole(s["vs"])}
        q = q.to(s["q"].dtype).double()                          # the rotated query is held in 16 bits as well
    out = torch.zeros((B, c["Hq"], d), dtype=torch.float64, device="cuda")
    lse = torch.full((B, c["Hq"]), -math.inf, dtype=torch.float64, device="cuda")
    plens, slens = s["plens"].tolist(), lens.tolist()
    for p in range(P):
        kp, vp = _wide(s["kp"][p, :, :plens[p]], s["kfac"]), _wide(s["vp"][p, :, :plens[p]], s["vfac"])
        for b in range(p * G, (p + 1) * G):
            if not act[b]:
                continue
            n = slens[b]
            if ps:
                pages = table[b, :-(-n // ps)]
                rows = lambda t: t[pages].transpose(0, 1).reshape(t.shape[1], -1, d)[:, :n]
                k, v = rows(s["ks"]), rows(s["vs"])
            else:
                k, v = s["ks"][b, :, :n], s["vs"][b, :, :n]
            out[b], lse[b] = _attend(q[b], [kp, _wide(k, s["kfac"])], [vp, _wide(v, s["vfac"])], scale)
    return {"out": out, "lse": lse, **more}


def _exact_tree(c, seed):
    s = _tree_inputs(c, seed)
    B, q = c["B"], s["q"].double()
    out, lse = torch.zeros_like(q), torch.zeros((B, c["Hq"]), dtype=torch.float64, device="cuda")
    slens, lens = s["slens"].tolist(), [lv[2].tolist() for lv in s["levels"]]
    for b in range(B):
        ks, vs = [], []
        for (k, v, _, group), ln in zip(s["levels"], lens):
            e = b // group
            ks.append(_wide(k[e, :, :ln[e]])), vs.append(_wide(v[e, :, :ln[e]]))
        ks.append(_wide(s["ks"][b, :, :slens[b]])), vs.append(_wide(s["vs"][b, :, :slens[b]]))
        out[b], lse[b] = _attend(q[b], ks, vs, 1.0 / math.sqrt(128))
    return {"out": out, "lse": lse}


def _exact_prefill(c, seed):
    s = _prepare_prefill(c, seed)
    P, Hq, Hkv, L = c["P"], c["Hq"], c["Hkv"], c["L"]
    r, scale = Hq // Hkv, 1.0 / math.sqrt(128)
    out = torch.zeros((P, L, Hq, 128), dtype=torch.float64, device="cuda")
    lse = torch.zeros((P, L, Hq), dtype=torch.float64, device="cuda")
    for p, n in enumerate(s["lens"].tolist()):
        future = torch.ones((n, n), dtype=torch.bool, device="cuda").triu(1)
        for j in range(Hkv):
            k, v = s["k"][p, j, :n].double().t().contiguous(), s["v"][p, j, :n].double()
            for h in range(j * r, (j + 1) * r):
                sc = torch.mm(s["q"][p, :n, h].double().contiguous(), k).mul_(scale).masked_fill_(future, -math.inf)
                l = torch.logsumexp(sc, -1)
                lse[p, :n, h] = l
                out[p, :n, h] = torch.mm(torch.exp(sc - l[:, None]), v)
    return {"out": out, "lse": lse}


def _exact_stats(c, seed):
    s = _prepare_stats(c, seed)
    got = {}
    for lo in range(0, c["rows"], 256):
        z, y = s["logits"][lo:lo + 256].double(), s["ids"][lo:lo + 256].long()[:, None]
        lp = torch.log_softmax(z, -1)
        p = lp.exp()
        part = {"logprob": lp.gather(1, y)[:, 0], "lse": torch.logsumexp(z, -1), "entropy": -(p * lp).sum(-1)}
        if c["ref"]:
            lr = torch.log_softmax(s["ref"][lo:lo + 256].double(), -1)
            part["ref_logprob"], part["kl"] = lr.gather(1, y)[:, 0], (p * (lp - lr)).sum(-1)
        for k, v in part.items():
            got.setdefault(k, []).append(v)
    return {k: torch.cat(v) for k, v in got.items()}


def _exact_loss(c, seed):
    s = _prepare_loss(c, seed)
    B, G, T = c["P"] * c["G"], c["G"], c["T"]
    r = (s["weights"].double()[:, None] * s["metrics"].double()).sum(0)
    g = r.view(-1, G)
    adv = ((g - g.mean(1, keepdim=True)) / (g.std(1, keepdim=True) + 1e-6)).reshape(B)
    lens = s["lens"].clamp(0, T)
    valid = torch.arange(T, device="cuda")[None] < lens[:, None]
    n = valid.sum().double()
    w = torch.full((B,), 1.0, dtype=torch.float64, device="cuda") / n
    if c["agg"] == "seq":
        w = torch.where(lens > 0, 1.0 / (lens.double() * (lens > 0).sum().double()), torch.zeros_like(w))
    wt = valid * w[:, None]
    lp, old = s["logprob"].double(), s["old"].double()
    rho, a = (lp - old).exp(), adv[:, None]
    lo, hi = float(np.float32(1) - np.float32(0.2)), float(np.float32(1) + np.float32(0.28))
    un, cl = rho * a, rho.clamp(lo, hi) * a
    term, flat = torch.minimum(un, cl), ~(un <= cl)
    tot = lambda x, weight: (x.double() * weight).sum()
    mean = valid / n
    pg = tot(term, wt)
    kl = tot(s["kl"], wt) if c["terms"] else torch.zeros_like(pg)
    ent = tot(s["entropy"], wt) if c["terms"] else torch.zeros_like(pg)
    stats = torch.stack([-pg + 0.01 * kl - 0.001 * ent, pg, kl, ent, tot(flat, mean), tot(rho, mean), tot(old - lp, mean), n])
    return {"rewards": r, "advantages": adv, "stats": stats, "grad": torch.where(flat, torch.zeros_like(un), -wt * un)}
