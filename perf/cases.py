"""What a decoding loop has this library do, as cases that can be timed and compared.

A case is a dict of plain values; `prepare` makes what a serving program holds before a call (KV pools, block
tables, queries, logits, token histories, workspaces and output buffers, all on the GPU), `run` makes the call
through the Python binding, and `exact` gives the attention outputs in 64-bit floating point from plain torch.

Kinds of case
  attention  one call of seer_verify_attention: chain or multi-path verification over a paged KV cache
  accept     one call of seer_accept, or of seer_accept_sampled where a temperature is given
  draft      one call of seer_draft over the token histories of prompt groups
  step       a whole step: drafts, attention of a few layers (the later ones on the first one's plan), acceptance,
             acceptance statistics, commit of the accepted path in every layer, append to the histories

Context lengths are the quantiles of the stated distribution, so a case has the same lengths whatever the seed;
which request has which length, the page order and all values come from the seed.  Keys and values are standard
normal, queries such that scaled scores have a standard deviation of 1.5 (some hundred tokens of a context
carry the weight).  Logits are standard normal with one entry per slot raised to 7.5 .. 8.5, the drafts agree
with those entries down to a random depth.
"""
from __future__ import annotations

import math
from statistics import NormalDist

import numpy as np
import torch

from paper_2511_14617_amd import binding, workloads

SCORE_STD = 1.5


def _attention(name, B, T, Hq, Hkv, Dqk, Dv, page, ctx, lo, mid, hi, paths=0, prefix=0, group=8):
    c = {"kind": "attention", "B": B, "T": T, "Hq": Hq, "Hkv": Hkv, "Dqk": Dqk, "Dv": Dv, "page": page, "ctx": ctx,
         "lo": lo, "mid": mid, "hi": hi, "paths": paths, "prefix": prefix, "group": group, "latent": Dqk == 576}
    return {"name": name, **c} if name else c


def listed():
    return [
        # a handful of short requests at the start of a rollout: the call is launches and latency
        _attention("chain_tiny", 4, 5, 8, 2, 128, 128, 16, "uniform", 64, 0, 512, group=4),
        # the bulk of a rollout on an 8B-class model: 8 groups of 8, one chain of 8 draft tokens each
        _attention("chain_grouped", 64, 9, 32, 8, 128, 128, 16, "lognormal", 512, 4096, 32768, prefix=512),
        # the end of a rollout: few stragglers with very long contexts and longer drafts
        _attention("chain_long_tail", 8, 17, 32, 8, 128, 128, 16, "uniform", 65536, 0, 131072),
        # one GPU's share of a dense 72B-class model under 8-way tensor parallelism
        _attention("chain_tp_share", 64, 9, 8, 1, 128, 128, 16, "lognormal", 512, 4096, 32768, prefix=512, group=16),
        # four candidate paths of eight tokens for every request of a large batch
        _attention("multipath_tree", 128, 33, 32, 8, 128, 128, 16, "lognormal", 1024, 8192, 32768, paths=4, prefix=512),
        # all 128 heads of a large MoE model over the shared latent, one GPU's requests
        _attention("latent_chain", 32, 5, 128, 1, 576, 512, 64, "uniform", 8192, 0, 24576),
        # a small model with 64-wide heads
        _attention("head64_chain", 16, 9, 16, 4, 64, 64, 16, "lognormal", 256, 2048, 16384),
        # few wide heads that share one KV head, 32-token pages
        _attention("head256_chain", 16, 5, 8, 1, 256, 256, 32, "lognormal", 256, 2048, 16384),
        # the vocabulary scan and acceptance walk that go with the grouped rollout, greedy
        {"name": "accept_greedy", "kind": "accept", "B": 64, "T": 9, "V": 152064, "paths": 0, "temperature": 0.0},
        # the same under sampling for a batch of draft trees
        {"name": "accept_sampled_tree", "kind": "accept", "B": 32, "T": 33, "V": 152064, "paths": 4, "temperature": 0.8},
        # drafts of four paths for every request of a large batch, from the histories of 16 groups
        {"name": "draft_multipath", "kind": "draft", "B": 128, "group": 8, "top_k": 4, "gamma": 8, "V": 152064,
         "lo": 1024, "mid": 8192, "hi": 32768},
        # one step of a small serving batch, drafts to appended tokens
        {"name": "decode_step", "kind": "step", "B": 16, "group": 8, "top_k": 1, "gamma": 8, "layers": 4, "Hq": 32, "Hkv": 8,
         "D": 128, "page": 16, "V": 152064, "lo": 512, "mid": 4096, "hi": 32768, "prefix": 512},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["d128", "d128", "d128", "latent", "other", "accept", "accept", "draft", "step"])
    if kind in ("d128", "latent", "other"):
        while True:
            if kind == "d128":
                dqk, dv, hkv, g = 128, 128, rng.choice([1, 2, 4, 8]), rng.choice([1, 2, 4, 4, 5, 8])
                page = rng.choice([16, 16, 16, 32, 64, 128])
                paths, length = rng.choice([(0, 0), (0, 0), (2, 4), (4, 8), (3, 5)])
                T = 1 + paths * length if paths else rng.randint(1, 17)
            elif kind == "latent":
                dqk, dv, hkv, g = 576, 512, 1, rng.choice([16, 32, 64, 128])
                page, paths, T = rng.choice([32, 64, 64, 128]), 0, rng.randint(1, 9)
            else:
                dqk, dv = rng.choice([(64, 64), (256, 256), (192, 128)])
                hkv, g = rng.choice([1, 2, 4]), rng.choice([1, 2, 4, 8])
                page = rng.choice([8, 16, 20, 32, 64])
                paths = rng.choice([0, 0, 2])
                T = 9 if paths else rng.randint(1, 17)
            B, mid = _log_int(rng, 1, 256), _log_int(rng, 64, 65536)
            ctx = rng.choice(["lognormal", "uniform"])
            lo = max(T, mid // 8 if ctx == "lognormal" else mid // 2)
            c = _attention("", B, T, g * hkv, hkv, dqk, dv, page, ctx, lo, mid if ctx == "lognormal" else 0,
                           max(mid * (8 if ctx == "lognormal" else 1), lo), paths=paths,
                           prefix=rng.choice([0, 512]) if lo >= 1024 else 0)
            tokens = int(_lengths(c).sum())
            bound = {"d128": 1.3e6 * 8, "latent": 0.5e6, "other": 60000}[kind]
            rows = T * g * hkv
            if tokens * hkv <= bound and tokens * rows <= {"d128": 1.3e6 * 1056, "latent": 0.5e6 * 640, "other": 6.4e6}[kind]:
                return c
    if kind == "accept":
        while True:
            paths = rng.choice([0, 0, 2, 4])
            c = {"kind": "accept", "B": _log_int(rng, 1, 256), "T": 1 + 8 * paths if paths else rng.randint(1, 17),
                 "V": rng.choice([1024, 32000, 50257, 128256, 151936, 152064, 163840]) + rng.choice([0, 0, 0, 3]),
                 "paths": paths, "temperature": rng.choice([0.0, 0.0, 0.8, 1.0])}
            if c["B"] * c["T"] * c["V"] <= 1056 * 152064:
                return c
    top_k = rng.choice([1, 2, 4])
    mid = _log_int(rng, 1024, 8192)
    c = {"kind": kind, "B": _log_int(rng, 1, 128 if kind == "draft" else 32), "group": rng.choice([4, 8, 16]),
         "top_k": top_k, "gamma": rng.randint(2, 8), "V": rng.choice([32000, 152064]), "lo": 64 + mid // 8, "mid": mid,
         "hi": 4 * mid}
    if kind == "step":
        c.update(layers=rng.randint(1, 6), Hkv=rng.choice([2, 4, 8]), D=128, page=rng.choice([16, 64]), prefix=0)
        c["Hq"] = c["Hkv"] * rng.choice([1, 4])
    return c


# ------------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------------
def _lengths(c):
    """Context lengths of a case, ascending: B quantiles of its distribution."""
    p = [(i + 0.5) / c["B"] for i in range(c["B"])]
    if c.get("ctx", "lognormal") == "uniform":
        n = [c["lo"] + x * (c["hi"] - c["lo"]) for x in p]
    else:
        n = [min(max(c["mid"] * math.exp(0.8 * NormalDist().inv_cdf(x)), c["lo"]), c["hi"]) for x in p]
    return np.maximum(np.rint(np.asarray(n)), _slots(c)).astype(np.int64)


def _slots(c):
    return 1 + c["top_k"] * c["gamma"] if "top_k" in c else c["T"]


def _pages(c, ctx, rng):
    """Block table (the pages of a group's common prompt shared, page order random) and the number of pages."""
    P, B, T = c["page"], c["B"], _slots(c)
    n_pages = -(-ctx // P)
    table = np.zeros((B, int(-(-max(c["hi"], int(ctx.max())) // P))), dtype=np.int32)
    shared, nxt = {}, 0
    for b in range(B):
        n_shared = int(min(c["prefix"], ctx[b] - T)) // P
        own = shared.setdefault(b // c["group"], [])
        while len(own) < n_shared:
            own.append(nxt)
            nxt += 1
        table[b, :n_shared] = own[:n_shared]
        rest = int(n_pages[b]) - n_shared
        table[b, n_shared:n_shared + rest] = np.arange(nxt, nxt + rest)
        nxt += rest
    total = nxt + max(2, nxt // 16)
    return rng.permutation(total).astype(np.int32)[table], total, nxt


def _tree(c, rng):
    """(parent, mask) of a batch of draft trees, None for chains."""
    if not c["paths"]:
        return None, None
    parent = workloads.multipath_parent(c["B"], c["paths"], (c["T"] - 1) // c["paths"], rng, dedup_fraction=0.25)
    return parent, workloads.ancestor_masks(parent)


def _normal(gen, shape, std=1.0, dtype=torch.bfloat16):
    x = torch.randn(shape, dtype=dtype, device="cuda", generator=gen)
    return x if std == 1.0 else x.mul_(std)


def _i32(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()


def _attention_state(c, rng, gen, layers=1):
    ctx = rng.permutation(_lengths(c))
    table, total, _ = _pages(c, ctx, rng)
    parent, mask = _tree(c, rng)
    scale = c["Dqk"] ** -0.5
    s = {"table": _i32(table), "ctx": _i32(ctx), "scale": scale, "Dv": c["Dv"], "parent": None if parent is None else _i32(parent),
         "mask": None if mask is None else torch.from_numpy(mask.view(np.int64)).cuda(), "layers": []}
    for _ in range(layers):
        s["layers"].append({
            "q": _normal(gen, (c["B"], c["T"], c["Hq"], c["Dqk"]), SCORE_STD),
            "k": _normal(gen, (total, c["Hkv"], c["page"], c["Dqk"])),
            "v": None if c["latent"] else _normal(gen, (total, c["Hkv"], c["page"], c["Dv"])),
            "out": torch.zeros((c["B"], c["T"], c["Hq"], c["Dv"]), dtype=torch.bfloat16, device="cuda")})
    x = s["layers"][0]
    p = binding.attn_params(x["q"], x["k"], x["v"], s["table"], scale, Dv=c["Dv"])
    s["workspace"] = torch.zeros(binding.seer_verify_attention_workspace(p), dtype=torch.uint8, device="cuda")
    return s


def _result_buffers(B, T):
    return tuple(torch.zeros(n, dtype=torch.int32, device="cuda") for n in ((B,), (B, T), (B,), (B, T)))


def _accept_state(c, rng, gen):
    B, T, V = c["B"], c["T"], c["V"]
    parent, _ = _tree(c, rng)
    par = workloads.chain_parent(B, T) if parent is None else parent
    target, draft = rng.integers(0, V, size=(B, T)), rng.integers(0, V, size=(B, T))
    depth = np.zeros((B, T), dtype=np.int64)
    agree = rng.integers(0, T if parent is None else 1 + (T - 1) // c["paths"], size=(B, T))   # a limit per slot and path
    rows = np.arange(B)
    for t in range(1, T):
        up = np.maximum(par[:, t], 0)
        depth[:, t] = depth[rows, up] + 1
        agree[:, t] = np.where(up > 0, agree[rows, up], agree[:, t])
        draft[:, t] = np.where((par[:, t] >= 0) & (depth[:, t] <= agree[:, t]), target[rows, up], draft[:, t])
    logits = _normal(gen, (B, T, V), dtype=torch.float32)
    logits.scatter_(2, torch.from_numpy(target[:, :, None]).cuda(), 7.5 + torch.rand((B, T, 1), device="cuda", generator=gen))
    return {"logits": logits, "draft": _i32(draft), "parent": None if parent is None else _i32(parent), "out": _result_buffers(B, T),
            "workspace": torch.zeros(max(16, binding.seer_accept_workspace(B, T, V)), dtype=torch.uint8, device="cuda")}


def _draft_config(c):
    return workloads.CONFIGS[2].scaled(B=c["B"], group_size=c["group"], T=_slots(c), V=c["V"], shared_prefix=c.get("prefix", 512),
                                       ctx=("fixed", tuple(int(x) for x in _lengths(c))))


def _draft_state(c, seed, spare=0):
    d = workloads.make_draft_inputs(_draft_config(c), seed, gamma_max=c["gamma"], top_k=c["top_k"], spare=spare)
    B, T, dev = c["B"], d.T, "cuda"
    p = binding.SeerDraftParams(B, len(d.group_first) - 1, len(d.seq_start), len(d.tokens), d.max_group_tokens + spare * c["group"],
                                c["gamma"], c["top_k"], d.p_min, d.p_max, c["V"], 0.0)
    i32 = lambda *n: torch.zeros(n, dtype=torch.int32, device=dev)  # noqa: E731
    return {"tokens": _i32(d.tokens), "seq_start": _i32(d.seq_start), "seq_len": _i32(d.seq_len), "capacity": _i32(d.seq_capacity),
            "group_first": _i32(d.group_first), "req_group": _i32(d.req_group), "req_seq": _i32(d.req_seq), "pattern": _i32(d.pattern),
            "pattern_len": _i32(d.pattern_len), "max_spec": _i32(d.max_spec_tokens), "gamma": c["gamma"], "top_k": c["top_k"],
            "p_min": d.p_min, "vocab": c["V"], "max_group_tokens": d.max_group_tokens + spare * c["group"], "future": d.future,
            "out": (i32(B, T), i32(B, T), torch.zeros((B, T), dtype=torch.int64, device=dev), i32(B, T), i32(B)),
            "workspace": torch.zeros(binding.seer_draft_workspace(p), dtype=torch.uint8, device=dev)}


def _step_case(c):
    """The attention call inside a step."""
    return {**c, "T": _slots(c), "Dqk": c["D"], "Dv": c["D"], "latent": False, "paths": 0}


def _step_state(c, rng, gen, seed):
    B, T, V = c["B"], _slots(c), c["V"]
    a = _attention_state(_step_case(c), rng, gen, c["layers"])
    d = _draft_state(c, seed, spare=64)
    # the model's logits: the token that really comes next, by depth of the slot, stands out
    level = np.asarray([0] + [1 + (t - 1) // c["top_k"] for t in range(1, T)])
    logits = _normal(gen, (B, T, V), dtype=torch.float32)
    logits.scatter_(2, torch.from_numpy(d["future"][:, level].astype(np.int64)[:, :, None]).cuda(),
                    7.5 + torch.rand((B, T, 1), device="cuda", generator=gen))
    return {"attention": a, "draft": d, "logits": logits, "accept": _result_buffers(B, T), "layers": c["layers"],
            "accept_workspace": torch.zeros(max(16, binding.seer_accept_workspace(B, T, V)), dtype=torch.uint8, device="cuda"),
            "counts": torch.zeros((3, T), dtype=torch.int64, device="cuda"), "tree": c["top_k"] > 1,
            "lens": torch.zeros((c["layers"], B), dtype=torch.int32, device="cuda"), "seq_len": d["seq_len"].clone()}


def prepare(case, seed):
    rng = np.random.default_rng([seed, 1])
    gen = torch.Generator(device="cuda").manual_seed(seed)
    state = {"attention": lambda: _attention_state(case, rng, gen), "accept": lambda: _accept_state(case, rng, gen),
             "draft": lambda: _draft_state(case, seed), "step": lambda: _step_state(case, rng, gen, seed)}[case["kind"]]()
    return {"kind": case["kind"], "temperature": case.get("temperature", 0.0), "seed": seed, **state}


# ------------------------------------------------------------------------------------------------
# the calls
# ------------------------------------------------------------------------------------------------
def _run_attention(s, mask, layer=0, flags=0):
    x = s["layers"][layer]
    return binding.seer_verify_attention(x["q"], x["k"], x["v"], s["table"], s["ctx"], mask, s["scale"], Dv=s["Dv"], flags=flags,
                                         out=x["out"], workspace=s["workspace"])


def _run_draft(s, seq_len):
    return binding.seer_draft(s["tokens"], s["seq_start"], seq_len, s["group_first"], s["req_group"], s["pattern"], s["pattern_len"],
                              s["max_spec"], gamma_max=s["gamma"], top_k=s["top_k"], pattern_lookup_min=s["p_min"],
                              vocab=s["vocab"], max_group_tokens=s["max_group_tokens"], workspace=s["workspace"], out=s["out"])


def _run_step(s):
    a, d = s["attention"], s["draft"]
    # the step works on copies of the lengths, so that it can be taken again from the same state
    s["lens"].copy_(a["ctx"].expand(s["layers"], -1))
    s["seq_len"].copy_(d["seq_len"])
    drafts = _run_draft(d, d["seq_len"])
    tokens, parent, mask = drafts[:3]
    outs = [_run_attention(a, mask, i, binding.SEER_ATTN_REUSE_PLAN if i else 0) for i in range(s["layers"])]
    alen, path, bonus, target = binding.seer_accept(s["logits"], tokens, parent, workspace=s["accept_workspace"], out=s["accept"])
    binding.seer_acceptance_stats(alen, path, parent, s["counts"])
    for i, x in enumerate(a["layers"]):
        emitted = binding.seer_kv_commit(x["k"], x["v"], a["table"], s["lens"][i], alen, path, draft_tokens=tokens, bonus_token=bonus)
    binding.seer_history_append(d["tokens"], d["seq_start"], s["seq_len"], d["capacity"], d["req_seq"], emitted[0], emitted[1])
    return {"attention": outs, "draft": list(drafts), "accept": [alen, path, bonus, target], "emitted": list(emitted),
            "lens": s["lens"], "seq_len": s["seq_len"], "counts": s["counts"]}


def run(state):
    kind = state["kind"]
    if kind == "attention":
        return _run_attention(state, state["mask"])
    if kind == "accept":
        if state["temperature"] > 0.0:
            return binding.seer_accept_sampled(state["logits"], state["draft"], state["parent"], state["temperature"],
                                               state["seed"], workspace=state["workspace"], out=state["out"])
        return binding.seer_accept(state["logits"], state["draft"], state["parent"], workspace=state["workspace"], out=state["out"])
    return _run_draft(state, state["seq_len"]) if kind == "draft" else _run_step(state)


# ------------------------------------------------------------------------------------------------
# what a pass cannot do without, how far results may be apart, and what they are in 64 bits
# ------------------------------------------------------------------------------------------------
def _attention_work(c):
    n = _lengths(c)
    _, _, unique = _pages(c, n, np.random.default_rng(0))
    per_page = c["Hkv"] * c["page"] * (c["Dqk"] + (0 if c["latent"] else c["Dv"])) * 2
    rows = c["B"] * c["T"] * c["Hq"]
    return {"bytes": unique * per_page + rows * (c["Dqk"] + c["Dv"]) * 2 + 4 * int(np.sum(-(-n // c["page"]))),
            "flops": 2 * (c["Dqk"] + c["Dv"]) * c["T"] * c["Hq"] * int(n.sum())}


def work(case):
    kind = case["kind"]
    if kind == "attention":
        return _attention_work(case)
    T = _slots(case)
    rows = case["B"] * T
    if kind == "accept":
        return {"bytes": 4 * rows * case["V"] + 16 * rows, "flops": rows * case["V"]}
    history = 4 * int(np.maximum(_lengths(case) - T - case.get("prefix", 512), 0).sum())
    draft = {"bytes": history + rows * 20, "flops": history // 4}
    if kind == "draft":
        return draft
    a = _attention_work(_step_case(case))
    return {"bytes": draft["bytes"] + case["layers"] * a["bytes"] + 4 * rows * case["V"],
            "flops": draft["flops"] + case["layers"] * a["flops"] + rows * case["V"]}


def tolerance(case):
    # bf16 outputs of sums in fp32; other cuts of the contexts, and so other orders of summation, gave outputs up to 3e-3
    # (largest element 0.022) apart where probabilities are rounded to bf16 for the matrix product, and up to 3e-5 (0.0065:
    # single roundings of the output) where they stay in fp32; whole numbers are exact
    if case["kind"] == "attention" and case["Dqk"] not in (128, 576):
        return {"rel": 5e-4, "max": 0.03}
    return {"rel": 1e-2, "max": 0.1} if case["kind"] in ("attention", "step") else "exact"


def _attention_exact(c, s, mask):
    outs = []
    T, G, D, V = c["T"], c["Hq"] // c["Hkv"], c["Dqk"], c["Dv"]
    for x in s["layers"]:
        out = torch.zeros((c["B"], T, c["Hq"], V), dtype=torch.float64, device="cuda")
        for b in range(c["B"]):
            n = int(s["ctx"][b])
            pages = s["table"][b, : -(-n // c["page"])].long()
            k = x["k"][pages].transpose(0, 1).reshape(c["Hkv"], -1, D)[:, :n].double()
            v = k[..., :V] if c["latent"] else x["v"][pages].transpose(0, 1).reshape(c["Hkv"], -1, V)[:, :n].double()
            q = x["q"][b].double().reshape(T, c["Hkv"], G, D).permute(1, 0, 2, 3)
            seen = torch.ones((T, n), dtype=torch.bool, device="cuda")
            slots = torch.arange(T, device="cuda")
            seen[:, n - T:] = (slots[None, :] <= slots[:, None]) if mask is None else ((mask[b][:, None] >> slots[None, :]) & 1).bool()
            for h in range(c["Hkv"]):
                sc = (q[h].reshape(T * G, D) @ k[h].T) * s["scale"]
                sc.view(T, G, n).masked_fill_(~seen[:, None, :], -math.inf)
                out[b].view(T, c["Hkv"], G, V)[:, h] = (torch.softmax(sc, dim=1) @ v[h]).view(T, G, V)
        outs.append(out)
    return outs


def exact(case, seed):
    if case["kind"] == "attention":
        s = prepare(case, seed)
        return _attention_exact(case, s, s["mask"])[0]
    if case["kind"] == "step":
        # the attention outputs, with the masks of the drafts (whole numbers, compared as such)
        s = prepare(case, seed)
        mask = _run_draft(s["draft"], s["draft"]["seq_len"])[2]
        return {"attention": _attention_exact(_step_case(case), s["attention"], mask), "draft": None, "accept": None,
                "emitted": None, "lens": None, "seq_len": None, "counts": None}
    return None
