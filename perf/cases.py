"""Workloads of one decoding step, as a serving program runs them through the Python binding.

Three kinds of call:

- ``verify``: one verification step of a batch of draft trees (the fused LM head, the margin
  rule, the walk and, with ``policy``, the draft confidence and the per-request state). A serving
  loop keeps its outputs and workspace, so they are allocated in ``prepare``.
- ``draft``: the drafting phase of a step: ``nsteps`` draft LM-head passes with tree growth, then
  the pruning to the verification budget.
- ``around``: what sits on either side of the target forward: tree-attention positions and masks
  before it, the commit of the accepted rows' hidden states after it.

Inputs follow ``workloads/``: weights N(0, 0.02) and hidden states N(0, 1) in bf16, drafted
tokens that are the target's top-1, one of its top-8 or any id in the proportions of a drafter
that agrees about half of the time, draft logits N(0, 2), a margin threshold of 0.05 to 0.3.
"""

import math
import random

import torch

import paper_2609_02897_amd as asv

LLAMA_V, QWEN_V, DRAFT_V, H8B = 128256, 151936, 32000, 4096


def _verify(name, H, V, B, N, layout, policy):
    return dict(name=name, op="verify", H=H, V=V, B=B, N=N, layout=layout, policy=policy)


def _draft(name, H, V, B, nsteps, topk, ndt):
    return dict(name=name, op="draft", H=H, V=V, B=B, nsteps=nsteps, topk=topk, ndt=ndt)


def listed():
    return [
        # One user, the deep narrow tree of the adaptive policy (7 drafted tokens and the root),
        # with the draft's confidence and the policy state: the most frequent call of all.
        _verify("llama_b1_chain8", H8B, LLAMA_V, 1, 8, "packed", True),
        # One user, a wide 60-node tree: the headline of bench.py.
        _verify("llama_b1_tree60", H8B, LLAMA_V, 1, 60, "packed", False),
        # A few users with small trees and a weight left in the checkpoint's row-major layout.
        _verify("qwen_b4_rowmajor", H8B, QWEN_V, 4, 29, "row_major", False),
        # A small batch on a target with a 32000-id vocabulary.
        _verify("vocab32k_b8", H8B, DRAFT_V, 8, 57, "packed", False),
        # A few users with ragged trees, policy on.
        _verify("qwen_b4_ragged", H8B, QWEN_V, 4, 190, "packed", True),
        # Eight users with ragged trees of 8 to 96 nodes, policy on.
        _verify("qwen_b8_ragged", H8B, QWEN_V, 8, 378, "packed", True),
        # The MFMA-bound batch: 32 users with 64 nodes each.
        _verify("llama_b32x64", H8B, LLAMA_V, 32, 2048, "packed", False),
        # The largest batch: 64 users with chains and wide trees.
        _verify("qwen_b64_mixed", H8B, QWEN_V, 64, 3048, "packed", True),
        # The drafting phase at one user (wide shallow trees), an ordinary and the largest batch.
        _draft("draft_b1", H8B, DRAFT_V, 1, 3, 4, 4),
        _draft("draft_b32", H8B, DRAFT_V, 32, 3, 4, 4),
        _draft("draft_b64", H8B, DRAFT_V, 64, 7, 1, 8),
        # Metadata and commit around the target forward: kilobytes to a few megabytes, where
        # launches and the latency of a call count.
        dict(name="around_b64", op="around", H=H8B, B=64, N=509),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["verify"] * 6 + ["draft"] * 3 + ["around"])
    if op == "verify":
        H = 64 * rng.randint(16, 80)                    # 1024 .. 5120
        V = rng.choice([DRAFT_V, LLAMA_V, QWEN_V, _log_int(rng, 32000, 152000)])
        N = min(_log_int(rng, 3, 3048), int(3048 * H8B * QWEN_V / (H * V)))
        B = max(1, min(64, N // rng.randint(3, 64)))
        return dict(op=op, H=H, V=V, B=B, N=N,
                    layout=rng.choice(["packed", "packed", "packed", "row_major"]),
                    policy=rng.random() < 0.5)
    if op == "draft":
        H = 64 * rng.randint(32, 64)                    # 2048 .. 4096
        nsteps, topk, ndt = rng.choice([(3, 4, 4), (4, 3, 5), (5, 2, 6), (6, 2, 7), (7, 1, 8)])
        return dict(op=op, H=H, V=rng.choice([DRAFT_V, _log_int(rng, 16000, 64000)]),
                    B=_log_int(rng, 1, 64), nsteps=nsteps, topk=topk, ndt=ndt)
    B = _log_int(rng, 1, 64)
    return dict(op=op, H=64 * rng.randint(16, 80), B=B, N=B * rng.randint(4, 60) + rng.randint(0, 3))


# ---- inputs

def _sizes(B, N):
    """Nodes of each request: ragged, at least one each, N in all, the same for every seed."""
    rng = random.Random(1000003 * B + N)
    w = [rng.uniform(0.3, 1.7) for _ in range(B)]
    n = [1 + int((N - B) * x / sum(w)) for x in w]
    for k in range(N - sum(n)):
        n[k % B] += 1
    return n


def _trees(B, N, rng):
    """(parent, depth, offsets) of a packed batch: chains, and trees whose nodes hang under one
    of the four nodes before them."""
    parent, depth, off = [], [], [0]
    for b, n in enumerate(_sizes(B, N)):
        lo, chain = off[-1], b % 3 == 0 and n <= 17
        for c in range(n):
            p = -1 if c == 0 else lo + (c - 1 if chain else max(0, c - rng.randint(1, 4)))
            parent.append(p)
            depth.append(0 if c == 0 else depth[p] + 1)
        off.append(lo + n)
    return parent, depth, off


def _i32(x):
    return torch.tensor(x, dtype=torch.int32, device="cuda")


def _normal(gen, shape, std, dtype=torch.bfloat16):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=gen)


def _chunks(V):
    return [(v, min(v + 16384, V)) for v in range(0, V, 16384)]


def _top8(hidden, w):
    """The 8 best ids of every row, best first."""
    h, val, ids = hidden.float(), None, None
    for lo, hi in _chunks(w.shape[0]):
        v, i = (h @ w[lo:hi].float().T).topk(min(8, hi - lo), dim=1)
        val, ids = (v, i + lo) if val is None else (torch.cat([val, v], 1),
                                                    torch.cat([ids, i + lo], 1))
    return ids.gather(1, val.topk(8, dim=1)[1]).cpu().tolist()


def _verify_inputs(case, seed):
    H, V, B, N = case["H"], case["V"], case["B"], case["N"]
    rng, gen = random.Random(seed), torch.Generator(device="cuda")
    gen.manual_seed(seed)
    hidden, w = _normal(gen, (N, H), 1.0), _normal(gen, (V, H), 0.02)
    parent, depth, off = _trees(B, N, rng)
    top8, tok = _top8(hidden, w), []
    for c in range(N):
        u = rng.random()
        if parent[c] < 0:
            tok.append(0)
        elif u < 0.5:
            tok.append(top8[parent[c]][0])
        else:
            tok.append(top8[parent[c]][rng.randrange(8)] if u < 0.8 else rng.randrange(V))
    logits = _normal(gen, (N, V), 2.0, torch.float32) if case["policy"] else None
    tau = [rng.choice([0.05, 0.1, 0.2, 0.3]) for _ in range(B)]
    return hidden, w, parent, tok, off, tau, logits


def _draft_inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    H, V, B = case["H"], case["V"], case["B"]
    w = _normal(gen, (V, H), 0.02)
    hidden = [_normal(gen, (4 * B, H), 1.0) for _ in range(case["nsteps"])]
    ids = torch.randperm(4 * V, generator=gen, device="cuda")[:V].sort()[0].to(torch.int32)
    root = _i32([(seed * 31 + b * 7919) % (4 * V) for b in range(B)])
    return w, hidden, ids, root


def _prepare_verify(case, seed):
    hidden, w, parent, tok, off, tau, logits = _verify_inputs(case, seed)
    B, N, H, V, dev = case["B"], case["N"], case["H"], case["V"], hidden.device
    s = dict(op="verify", hidden=hidden, tok=_i32(tok), parent=_i32(parent), off=_i32(off),
             tau=torch.tensor(tau, dtype=torch.float32, device=dev), logits=logits, state=None,
             w=asv.pack_lm_head(w) if case["layout"] == "packed" else w,
             out=asv.alloc_outputs(B, N, dev, case["policy"]),
             ws=asv.alloc_workspace(B, N, H, V, dev))
    s["out"].drafted_logit.zero_()      # the roots' entries are not written by the call
    ret = {f: getattr(s["out"], f) for f in s["out"]._fields if getattr(s["out"], f) is not None}
    if case["policy"]:
        s["state"] = asv.state_init(B, device=dev)
        f, i = s["state"].view(torch.float32), s["state"].view(torch.int32)
        # rar, the history ring | head, count, streak, breaker, steps | mean, confidence, score |
        # the next tree's shape
        ret.update(rar_hist=f[:, :17], counters=i[:, 17:22], scores=f[:, 22:25], shape=i[:, 25:])
    s["ret"] = ret
    return s


def _prepare_draft(case, seed):
    w, hidden, ids, root = _draft_inputs(case, seed)
    B, H, V = case["B"], case["H"], case["V"]
    R, dev = 4 * B, w.device
    outs = [asv.DraftOut(torch.empty((R, 4), dtype=torch.int32, device=dev),
                         torch.empty((R, 4), dtype=torch.float32, device=dev),
                         torch.empty(R, dtype=torch.float32, device=dev),
                         torch.empty((B, 4), dtype=torch.int32, device=dev),
                         torch.empty(B, dtype=torch.float32, device=dev) if k == 0 else None)
            for k in range(case["nsteps"])]
    pool = case["topk"] + (case["nsteps"] - 1) * case["topk"] ** 2
    return dict(op="draft", w=asv.pack_draft_head(w), hidden=hidden, ids=ids, root=root,
                shape=(case["nsteps"], case["topk"], case["ndt"]), outs=outs,
                n=B * (1 + min(case["ndt"] - 1, pool)), trees=asv.alloc_draft_trees(B, dev),
                ws=torch.empty(max(asv.draft_workspace_bytes(B, H, V), 256), dtype=torch.uint8,
                               device=dev))


def _prepare_around(case, seed):
    H, B, N = case["H"], case["B"], case["N"]
    rng, gen = random.Random(seed), torch.Generator(device="cuda")
    gen.manual_seed(seed)
    parent, depth, off = _trees(B, N, rng)
    # the accepted nodes, the first ones of the last node's path from the root: up to four, the
    # same number for every seed (a tree of n nodes is at least (n - 1) / 4 deep)
    path, length, fixed = [-1] * N, [], random.Random(B)
    for lo, hi in zip(off, off[1:]):
        c, chain = hi - 1, []
        while c != lo:
            chain.append(c)
            c = parent[c]
        length.append(min(fixed.randint(0, 4), (hi - lo + 2) // 4))
        path[lo:lo + length[-1]] = chain[::-1][:length[-1]]
    ids = lambda n: _i32([rng.randrange(QWEN_V) for _ in range(n)])  # noqa: E731
    widest = max(hi - lo for lo, hi in zip(off, off[1:]))
    return dict(op="around", parent=_i32(parent), off=_i32(off),
                base=_i32([rng.randrange(4096) for _ in range(B)]), words=-(-widest // 32),
                tok=ids(N), length=_i32(length), path=_i32(path), bonus=ids(B),
                hidden=_normal(gen, (N, H), 1.0), total=sum(length) + B)


def prepare(case, seed):
    return {"verify": _prepare_verify, "draft": _prepare_draft,
            "around": _prepare_around}[case["op"]](case, seed)


# ---- one pass

def run(s):
    if s["op"] == "verify":
        asv.verify(s["hidden"], s["w"], s["tok"], s["parent"], s["off"], s["tau"], s["logits"],
                   state=s["state"], out=s["out"], workspace=s["ws"])
        return s["ret"]
    if s["op"] == "draft":
        for k, out in enumerate(s["outs"]):
            asv.draft_step(s["hidden"][k], s["w"], s["trees"], k, shape=s["shape"],
                           vocab_map=s["ids"], out=out, workspace=s["ws"])
        return {"steps": [list(o) for o in s["outs"]],
                "tree": asv.draft_prune(s["trees"], s["n"], s["root"])}
    pos, mask, st1 = asv.tree_meta(s["parent"], s["off"], s["base"], s["words"])
    off, tok, row, dst, st2 = asv.commit(s["off"], s["tok"], s["length"], s["path"], s["bonus"],
                                         s["hidden"])
    n = s["total"]                      # entries past the committed ones are not written
    return [pos, mask, st1, off, tok[:n], row[:n], dst[:n], st2]


# ---- what a pass cannot do without, and how far two right answers may be apart

def work(case):
    B, H = case["B"], case["H"]
    if case["op"] == "verify":
        N, V = case["N"], case["V"]
        conf = 4 * B * V + 2 * 112 * B if case["policy"] else 0
        return {"bytes": 2 * V * H + 2 * N * H + 29 * N + 20 * B + conf, "flops": 2 * N * V * H}
    if case["op"] == "draft":
        R, V, n = 4 * B, case["V"], case["nsteps"]
        return {"bytes": n * (2 * V * H + 2 * R * H + 40 * R), "flops": n * 2 * R * V * H}
    # metadata and ids, and the committed rows once in and once out (about four a request)
    return {"bytes": 32 * case["N"] + 2 * 2 * 4 * B * H, "flops": 0}


def tolerance(case):
    if case["op"] == "around":
        return "exact"
    # sums of H bf16 products in float32: 2e-7 to 4e-7 off the float64 values; the draft's
    # confidence is the exponential of such a sum, 4e-6 off
    return {"rel": 1.6e-5 if case["op"] == "draft" else 2e-6, "max": 4e-5, "differ": 1e-3}


# ---- the computed outputs in float64

def _logits64(hidden, w):
    h = hidden.double()
    return torch.cat([h @ w[lo:hi].double().T for lo, hi in _chunks(w.shape[0])], 1)


def exact(case, seed):
    if case["op"] == "around":
        return None
    if case["op"] == "draft":
        w, hidden, _, _ = _draft_inputs(case, seed)
        steps = []
        for k, h in enumerate(hidden):
            z = _logits64(h, w)
            lse = torch.logsumexp(z, 1)
            lp = z.topk(4, dim=1)[0] - lse[:, None]
            steps.append([None, lp, lse, None, lp[0::4, 0].exp() if k == 0 else None])
        return {"steps": steps, "tree": [None] * 4}
    hidden, w, parent, tok, off, _, logits = _verify_inputs(case, seed)
    z = _logits64(hidden, w)
    ret = {"row_max": z.max(1)[0], "row_lse": torch.logsumexp(z, 1)}
    par, ids = torch.tensor(parent, device="cuda"), torch.tensor(tok, device="cuda")
    ret["drafted_logit"] = torch.where(par < 0, 0.0, z[par.clamp(min=0), ids])
    if logits is not None:
        q = logits[torch.tensor(off[:-1], device="cuda")].double()
        ret["draft_conf"] = torch.softmax(q, 1).max(1)[0]
    return ret
