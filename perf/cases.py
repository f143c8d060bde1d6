"""The work that users of this package have it do, case by case, for timing.

Every case is one pass through the public entry points of
``paper_2606_18394_amd``: the verification attention in its four cache
layouts, greedy and sampled tree acceptance, tree drafting (per-depth
candidates, then the best-first tree), the draft head's training mask, and a
whole serving step (attention, acceptance, commit).  Head shapes, tree sizes,
cache lengths and the vocabulary are those of ``synth.WORKLOADS``, of
``bench.py`` and of the tests; the odd sizes are generic.

  listed()             the cases
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  what a program has in hand before the call, on the GPU
  run(state)           one pass; its outputs, whole
  work(case)           bytes and flops a pass cannot do without
  tolerance(case)      how far another correct implementation may be off
  exact(case, seed)    the computed numbers in 64 bits, plain torch
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2606_18394_amd as tv
from paper_2606_18394_amd import synth

# (query heads, KV heads, head dim): the shapes of synth.WORKLOADS, and two
# small generic ones with D = 64 (one without grouped queries)
HEADS = [(4, 2, 64), (32, 8, 128), (32, 4, 128), (64, 8, 128), (16, 8, 64), (8, 8, 128)]
LAYOUTS = ["padded", "paged", "tail", "paged_tail"]
BLOCK = 64  # rows of a cache page


def _attend(name, B, Hq, Hkv, D, L, lo, N, depth, branching, layout):
    """Verification attention.  kv_len is drawn from [lo, L]; branching 0: no cap."""
    return {"name": name, "kind": "attend", "B": B, "Hq": Hq, "Hkv": Hkv, "D": D, "L": L,
            "lo": lo, "N": N, "depth": depth, "branching": branching, "layout": layout}


def listed():
    return [
        # the smallest call: a draft of 16 nodes on a short prompt of a small model
        _attend("attend_tiny", 1, 4, 2, 64, 256, 256, 16, 4, 0, "padded"),
        # one user, 8B-shaped target, 64-node tree, a few thousand tokens of context
        _attend("attend_8b", 1, 32, 8, 128, 4096, 4096, 64, 8, 4, "padded"),
        # one user, a long document: 32768 cached rows, 128-node tree
        _attend("attend_long", 1, 32, 8, 128, 32768, 32768, 128, 12, 4, "padded"),
        # the serving engine's layout at batch 16, root + 32 drafts, ragged
        # paged caches with the tree's rows behind the context
        _attend("attend_serving", 16, 32, 8, 128, 4096, 300, 33, 8, 4, "paged_tail"),
        # a loaded server: 16 sequences of very different lengths
        _attend("attend_batch", 16, 32, 4, 128, 16384, 1024, 64, 8, 4, "padded"),
        # the largest draft budget on the widest target
        _attend("attend_big_tree", 1, 64, 8, 128, 8192, 8192, 512, 16, 8, "padded"),
        # greedy acceptance over one user's 64-node tree
        {"name": "accept_8b", "kind": "accept", "B": 1, "N": 64, "V": 151936, "dtype": "bf16",
         "depth": 8, "branching": 4, "p": 0.6},
        # greedy acceptance of a batch whose logits come in fp32, with a
        # vocabulary that is no multiple of anything
        {"name": "accept_odd_batch", "kind": "accept", "B": 8, "N": 33, "V": 100003,
         "dtype": "f32", "depth": 8, "branching": 4, "p": 0.6},
        # temperature sampling: four users with 64-node trees
        {"name": "sampled", "kind": "sampled", "B": 4, "N": 64, "V": 151936, "dtype": "bf16",
         "depth": 8, "branching": 4, "T": 1.0},
        # drafting, first half: candidates of 16 draft depths of one user
        {"name": "draft_topw", "kind": "topw", "B": 1, "Nd": 16, "W": 8, "V": 151936,
         "dtype": "bf16"},
        # drafting, second half: four users' trees of 512 nodes
        {"name": "draft_tree", "kind": "tree", "B": 4, "Nd": 16, "W": 8, "budget": 512},
        # draft-head training: 512 sampled anchors, blocks of 16, forward
        {"name": "train_mask", "kind": "train", "B": 1, "A": 512, "S": 16, "Hq": 32, "Hkv": 8,
         "D": 128, "L": 4096},
    ]


def _log_int(rng, lo, hi):
    """An integer of [lo, hi], spread evenly over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _caps(rng):
    """Depth and branching caps of a drawn tree that leave room for 512 nodes."""
    depth = rng.randint(4, 16)
    return depth, rng.choice([0, 4 if depth > 5 else 8, 8])


def _draw_once(rng):
    kind = rng.choice(["attend", "attend", "attend", "accept", "accept", "sampled", "topw", "tree",
                       "train", "step"])
    if kind in ("attend", "step"):
        Hq, Hkv, D = rng.choice(HEADS if kind == "attend" else HEADS[1:4])
        N = _log_int(rng, 8, 512)
        L = _log_int(rng, 256, 32768)
        B = _log_int(rng, 1, 32)
        depth, branching = _caps(rng)
        c = {"kind": kind, "B": B, "Hq": Hq, "Hkv": Hkv, "D": D, "L": L, "lo": max(1, L // 16),
             "N": N, "depth": depth, "branching": branching,
             "layout": rng.choice(LAYOUTS)}
        if kind == "step":
            c["N"] = min(N, 128)
            c["V"] = rng.choice([32000, 151936])
            c["dtype"] = rng.choice(["bf16", "f32"])
            c["p"] = rng.choice([0.5, 0.6, 0.7])
            c["layout"] = rng.choice(["padded", "paged"])
        return c
    V = rng.choice([_log_int(rng, 1024, 160000), 32000, 151936])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    if kind in ("accept", "sampled"):
        depth, branching = _caps(rng)
        c = {"kind": kind, "B": _log_int(rng, 1, 32), "N": _log_int(rng, 8, 512), "V": V,
             "dtype": dtype, "depth": depth, "branching": branching}
        c.update({"p": rng.choice([0.5, 0.6, 0.7])} if kind == "accept" else
                 {"T": rng.choice([0.6, 0.8, 1.0, 1.3])})
        return c
    if kind == "topw":
        return {"kind": kind, "B": _log_int(rng, 1, 32), "Nd": rng.randint(4, 16),
                "W": rng.choice([2, 4, 8, 16]), "V": V, "dtype": dtype}
    if kind == "tree":
        return {"kind": kind, "B": _log_int(rng, 1, 64), "Nd": rng.randint(4, 16),
                "W": rng.choice([2, 4, 8, 16]), "budget": _log_int(rng, 16, 1024)}
    Hq, Hkv, D = rng.choice(HEADS[1:])
    return {"kind": kind, "B": rng.randint(1, 3), "A": _log_int(rng, 16, 512),
            "S": rng.choice([8, 16, 16, 32]), "Hq": Hq, "Hkv": Hkv, "D": D,
            "L": _log_int(rng, 256, 4096)}


def draw(rng):
    """One more case; redrawn while it would cost more than the largest listed
    ones (the training mask's flops, a quarter of a gigabyte of traffic)."""
    while True:
        c = _draw_once(rng)
        w = work(c)
        if w["flops"] > 1.3e11 or w["bytes"] > 2.5e8:
            continue
        if c["kind"] in ("attend", "step") and c["B"] * c["L"] * c["Hkv"] * c["D"] > 1.5e8:
            continue
        return c


# ------------------------------------------------------------------ inputs


def _rng(seed, salt=0):
    return np.random.default_rng([seed, salt])


def _gen(seed, salt=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1000003 + salt)
    return g


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32).to(torch.bfloat16)


def _i32(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()


def _trees(case, seed):
    r = _rng(seed, 1)
    return np.stack([synth.random_tree(r, case["N"], case["depth"], case["branching"] or None)
                     for _ in range(case["B"])])


def _room(case):
    """Cache rows of a sequence: the context, the tree's rows in the tail
    layouts, the committed rows of a step; whole pages in the paged ones."""
    rows = case["L"]
    if case["layout"].endswith("tail"):
        rows += case["N"]
    if case["kind"] == "step":
        rows += case["depth"] + 1
    if case["layout"].startswith("paged"):
        rows = (rows + BLOCK - 1) // BLOCK * BLOCK
    return rows


def _logits(case, g, rows):
    """Target or draft logits with the spread of a language model's: N(0, 2)."""
    x = torch.randn(case["B"], rows, case["V"], generator=g, device="cuda") * 2.0
    return x if case["dtype"] == "f32" else x.to(torch.bfloat16)


def _draft(case, logits, parent, g):
    """Draft tokens: the target's choice at the parent with probability p."""
    B, N, V = logits.shape
    tgt = logits.float().argmax(-1)
    up = tgt.gather(1, parent.long().clamp(min=0))
    other = torch.randint(0, V, (B, N), generator=g, device="cuda")
    hit = torch.rand(B, N, generator=g, device="cuda") < case.get("p", 0.6)
    return torch.where(hit, up, other).to(torch.int32)


def _attention_state(case, seed):
    g = _gen(seed)
    B, N, Hq, Hkv, D = (case[k] for k in ("B", "N", "Hq", "Hkv", "D"))
    rows = _room(case)
    kv = _rng(seed, 2).integers(case["lo"], case["L"] + 1, size=B)
    s = {"case": case, "parent": _i32(_trees(case, seed)), "kv_len": _i32(kv),
         "q": _normal(g, B, N, Hq, D), "out": torch.empty(B, N, Hq, D, dtype=torch.bfloat16,
                                                          device="cuda")}
    if case["layout"].startswith("paged"):
        per = rows // BLOCK
        bt, _ = synth.block_table(_rng(seed, 3), B, per)
        s["table"] = _i32(bt)
        s["k"] = _normal(g, B * per, BLOCK, Hkv, D)
        s["v"] = _normal(g, B * per, BLOCK, Hkv, D)
    else:
        s["k"] = _normal(g, B, rows, Hkv, D)
        s["v"] = _normal(g, B, rows, Hkv, D)
    tail = case["layout"].endswith("tail")
    s["kt"] = None if tail else _normal(g, B, N, Hkv, D)
    s["vt"] = None if tail else _normal(g, B, N, Hkv, D)
    return s


def prepare(case, seed):
    kind = case["kind"]
    g = _gen(seed, 7)
    if kind == "attend":
        return _attention_state(case, seed)
    if kind in ("accept", "sampled", "step"):
        s = _attention_state(case, seed) if kind == "step" else {"case": case}
        parent = s["parent"] if kind == "step" else _i32(_trees(case, seed))
        lg = _logits(case, g, case["N"])
        s.update(parent=parent, logits=lg, draft=_draft(case, lg, parent, g))
        if kind == "sampled":
            s["u"] = torch.rand(case["B"], case["N"], generator=g, device="cuda")
            s["seed"] = 12345 + seed
        if kind == "step":
            s["kv0"] = s["kv_len"].clone()
        return s
    if kind == "topw":
        return {"case": case, "logits": _logits(case, g, case["Nd"])}
    if kind == "tree":
        # candidates as the first half of drafting makes them: per depth the
        # W best log-probabilities, decreasing
        B, Nd, W = case["B"], case["Nd"], case["W"]
        x = torch.randn(B, Nd, 4096, generator=g, device="cuda") * 2.0
        lp, tok = torch.log_softmax(x, -1).topk(W, dim=-1)
        return {"case": case, "tok": tok.to(torch.int32).contiguous(), "logp": lp.contiguous(),
                "root": torch.randint(0, 4096, (B,), generator=g, device="cuda").to(torch.int32)}
    B, A, S, Hq, Hkv, D, L = (case[k] for k in ("B", "A", "S", "Hq", "Hkv", "D", "L"))
    return {"case": case, "q": _normal(g, B, A, S, Hq, D), "k": _normal(g, B, L, Hkv, D),
            "v": _normal(g, B, L, Hkv, D), "kb": _normal(g, B, A, S, Hkv, D),
            "vb": _normal(g, B, A, S, Hkv, D),
            "anchors": _i32(_rng(seed, 4).integers(0, L + 1, size=(B, A))),
            "out": torch.empty(B, A, S, Hq, D, dtype=torch.bfloat16, device="cuda")}


# ------------------------------------------------------------------ a pass


def _verify(s):
    if "table" in s:
        return tv.tree_verify_attention_paged(s["q"], s["k"], s["v"], s["table"], s["kt"], s["vt"],
                                              s["parent"], s["out"], kv_len=s["kv_len"])
    return tv.tree_verify_attention(s["q"], s["k"], s["v"], s["kt"], s["vt"], s["parent"],
                                    s["out"], kv_len=s["kv_len"])


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "attend":
        return _verify(s)
    if kind == "accept":
        return tv.tree_accept(s["logits"], s["draft"], s["parent"], case["depth"] + 1)
    if kind == "sampled":
        return tv.tree_accept_sampled(s["logits"], s["draft"], s["parent"], s["u"], s["seed"],
                                      case["T"], case["depth"] + 1)
    if kind == "topw":
        return tv.draft_topw(s["logits"], case["W"])
    if kind == "tree":
        return tv.build_tree(s["tok"], s["logp"], case["budget"], root_tok=s["root"])
    if kind == "train":
        return tv.block_causal_attention(s["q"], s["k"], s["v"], s["kb"], s["vb"], s["anchors"],
                                         s["out"])
    # a serving step: verify, accept, commit.  The cache starts each pass at
    # the same length, so every pass commits the same rows.
    s["kv_len"].copy_(s["kv0"])
    out = _verify(s)
    n, path, tgt = tv.tree_accept(s["logits"], s["draft"], s["parent"], case["depth"] + 1)
    if "table" in s:
        tv.commit_path_paged(s["kt"], s["vt"], path, n, s["k"], s["v"], s["table"], s["kv_len"])
    else:
        tv.commit_path(s["kt"], s["vt"], path, n, s["k"], s["v"], s["kv_len"])
    return out, n, path, tgt, s["kv_len"], s["k"], s["v"]


# ------------------------------------------------------------------ accounts


def _mean_kv(case):
    return (case["lo"] + case["L"]) / 2


def work(case):
    kind = case["kind"]
    if kind in ("attend", "step"):
        B, N, Hq, Hkv, D = (case[k] for k in ("B", "N", "Hq", "Hkv", "D"))
        keys = _mean_kv(case)
        nbytes = 4 * B * D * (Hkv * (keys + N) + Hq * N) + 4 * B * N
        flops = 4 * D * Hq * B * N * (keys + case["depth"] / 2 + 1)
        if kind == "step":
            nbytes += B * N * case["V"] * (4 if case["dtype"] == "f32" else 2)
            nbytes += 8 * B * case["depth"] / 2 * Hkv * D
        return {"bytes": nbytes, "flops": flops}
    if kind in ("accept", "sampled"):
        e = 4 if case["dtype"] == "f32" else 2
        return {"bytes": case["B"] * case["N"] * (case["V"] * e + 12), "flops": 0}
    if kind == "topw":
        e = 4 if case["dtype"] == "f32" else 2
        return {"bytes": case["B"] * case["Nd"] * (case["V"] * e + 8 * case["W"]), "flops": 0}
    if kind == "tree":
        return {"bytes": case["B"] * (8 * case["Nd"] * case["W"] + 16 * case["budget"]),
                "flops": 0}
    B, A, S, Hq, Hkv, D, L = (case[k] for k in ("B", "A", "S", "Hq", "Hkv", "D", "L"))
    return {"bytes": 4 * B * D * (Hkv * L + Hkv * A * S + Hq * A * S),
            "flops": 4 * D * Hq * B * A * S * (L / 2 + (S + 1) / 2)}


def tolerance(case):
    kind = case["kind"]
    if kind in ("attend", "train", "step"):
        # bf16 weights and bf16 outputs: the outputs are 2.0e-3 to 2.3e-3 off
        # their 64-bit values
        return {"rel": 9e-3, "max": 0.2}
    if kind == "topw":
        # fp32 log-sum-exps of up to 160000 terms (7e-8 off their 64-bit
        # values); the tokens are exact
        return {"rel": 5e-7, "max": 4e-6}
    if kind == "sampled":
        # tests and races in fp32: one within 1e-6 of its threshold may go either way
        return {"rel": 0.0, "differ": 0.005}
    return "exact"  # acceptance and trees are comparisons of given numbers


# ------------------------------------------------------------------ 64 bits


def _masked(q, k, v, vis, scale):
    """softmax(q k^T scale, where vis) v in fp64; q [M, D], k, v [T, D], vis [M, T]."""
    sc = (q.double() @ k.double().t()) * scale
    return torch.softmax(sc.masked_fill(~vis, -math.inf), -1) @ v.double()


def _exact_attention(s):
    case = s["case"]
    B, N, Hq, Hkv, D = (case[k] for k in ("B", "N", "Hq", "Hkv", "D"))
    G = Hq // Hkv
    parent, kv = s["parent"].cpu().numpy(), s["kv_len"].cpu().numpy()
    out = torch.empty(B, N, Hq, D, dtype=torch.float64, device="cuda")
    for b in range(B):
        anc = np.zeros((N, N), dtype=bool)
        for i in range(N):
            if i:
                anc[i] = anc[parent[b, i]]
            anc[i, i] = True
        n = int(kv[b])
        if "table" in s:
            kc, vc = (s[x][s["table"][b].long()].reshape(-1, Hkv, D) for x in "kv")
        else:
            kc, vc = s["k"][b], s["v"][b]
        if s["kt"] is None:
            k, v = kc[:n + N], vc[:n + N]
        else:
            k, v = torch.cat([kc[:n], s["kt"][b]]), torch.cat([vc[:n], s["vt"][b]])
        vis = torch.ones(N, n + N, dtype=torch.bool, device="cuda")
        vis[:, n:] = torch.from_numpy(anc).cuda()
        vis = vis.repeat_interleave(G, 0)
        for h in range(Hkv):
            q = s["q"][b, :, h * G:(h + 1) * G].reshape(N * G, D)
            out[b, :, h * G:(h + 1) * G] = _masked(q, k[:, h], v[:, h], vis,
                                                   D ** -0.5).reshape(N, G, D)
    return out


def _exact_train(s):
    case = s["case"]
    B, A, S, Hq, Hkv, D, L = (case[k] for k in ("B", "A", "S", "Hq", "Hkv", "D", "L"))
    G = Hq // Hkv
    out = torch.empty(B, A, S, Hq, D, dtype=torch.float64, device="cuda")
    own = torch.ones(S, S, dtype=torch.bool, device="cuda").tril().repeat_interleave(G, 0)
    pos = torch.arange(L, device="cuda")
    step = max(1, 4096 // (S * G))
    for b in range(B):
        for h in range(Hkv):
            hs = slice(h * G, (h + 1) * G)
            kc, vc = s["k"][b, :, h].double(), s["v"][b, :, h].double()
            for a0 in range(0, A, step):
                a1 = min(A, a0 + step)
                n = a1 - a0
                q = s["q"][b, a0:a1, :, hs].reshape(n, S * G, D).double() * D ** -0.5
                ctx = q.reshape(-1, D) @ kc.t()
                ctx = ctx.reshape(n, S * G, L)
                ctx = ctx.masked_fill(pos >= s["anchors"][b, a0:a1, None, None], -math.inf)
                kb, vb = s["kb"][b, a0:a1, :, h].double(), s["vb"][b, a0:a1, :, h].double()
                blk = torch.bmm(q, kb.transpose(1, 2).contiguous()).masked_fill(~own, -math.inf)
                w = torch.softmax(torch.cat([ctx, blk], -1), -1)
                o = (w[..., :L].reshape(-1, L) @ vc).reshape(n, S * G, D)
                o = o + torch.bmm(w[..., L:].contiguous(), vb)
                out[b, a0:a1, :, hs] = o.reshape(n, S, G, D)
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "attend":
        return _exact_attention(prepare(case, seed))
    if kind == "step":
        return _exact_attention(prepare(case, seed)), None, None, None, None, None, None
    if kind == "train":
        return _exact_train(prepare(case, seed))
    if kind == "topw":
        lg = prepare(case, seed)["logits"]
        logp = torch.stack([(r.topk(case["W"], dim=-1).values - torch.logsumexp(r, -1, True))
                            for r in (x.double() for x in lg)])
        return None, logp
    return None  # whole numbers, and sums that the tree's rule takes in fp32
