"""Performance cases: the calls that one speculative decoding iteration makes.

An iteration of tree-based speculative decoding builds a draft tree
(`tree_build`), runs the target model with one `tree_verify_attention` per
layer, reduces the final hidden states to greedy tokens with
`tree_lm_head_argmax_accept` (or `tree_argmax_accept` where the program has the
logits), keeps the accepted rows with `kv_compact_accepted` and re-samples a
tree from the logits it did not use (`tree_resample`). The listed cases take
each call at the sizes of this repository's own presets and between them; the
drawn ones spread over the same ranges. Workspaces and output buffers are kept
between calls, as a serving loop keeps them.
"""
import math

import numpy as np
import torch

import paper_2602_21224_amd as T
from paper_2602_21224_amd import workloads as W

BF16 = torch.bfloat16


def listed():
    return [
        # A whole verification step of one short sequence: attention, acceptance
        # from logits and compaction. Launches and the host path count.
        dict(name="step_tiny", kind="step", B=1, N=16, Hq=8, Hkv=8, D=64, P=16, lo=128, hi=128,
             tree="forest", ragged=False, V=1000),
        # Multi-head attention with the narrow depth-3 trees of 12 tokens that the
        # method verifies, two requests.
        dict(name="attn_mha_b2", kind="attn", B=2, N=12, Hq=32, Hkv=32, D=128, P=16, lo=256,
             hi=2048, tree="frontier", ragged=False),
        # Fused verification (a new tree and a re-sampled one per sequence: node
        # counts differ) with head size 64, one-token pages, odd sizes, three heads per group.
        dict(name="attn_fused_d64", kind="attn", B=5, N=45, Hq=24, Hkv=8, D=64, P=1, lo=300,
             hi=2500, tree="fused", ragged=True),
        # Grouped-query attention of an 8B-shaped layer, 16 requests in 16-token pages.
        dict(name="attn_gqa_b16", kind="attn", B=16, N=64, Hq=32, Hkv=8, D=128, P=16, lo=1024,
             hi=4096, tree="capped", ragged=False),
        # The same of a 70B-shaped layer: 1024 query rows per KV head.
        dict(name="attn_gqa70_b8", kind="attn", B=8, N=128, Hq=64, Hkv=8, D=128, P=16, lo=8192,
             hi=8192, tree="capped", ragged=False),
        # Long prefixes and the widest trees.
        dict(name="attn_long_b4", kind="attn", B=4, N=256, Hq=32, Hkv=8, D=128, P=16, lo=32768,
             hi=32768, tree="capped", ragged=False),
        # The end of a step that has its logits: acceptance, then compaction of the
        # accepted rows into an 8B-shaped layer's cache.
        dict(name="accept_b16", kind="accept", B=16, N=64, Hq=32, Hkv=8, D=128, P=16, lo=1024,
             hi=4096, tree="capped", ragged=False, V=128256),
        # LM head and acceptance: two requests with 12-token trees over a 32000-token
        # vocabulary, one request with a 64-token tree, a full batch.
        dict(name="lm_b2", kind="lm", B=2, N=12, V=32000, d=4096),
        dict(name="lm_b1", kind="lm", B=1, N=64, V=128256, d=4096),
        dict(name="lm_b16", kind="lm", B=16, N=64, V=128256, d=4096),
        # Draft trees of a batch, 7 steps of 8 branches, 32768 hot tokens.
        dict(name="build_b16", kind="build", B=16, S=7, V=128256, H=32768, k=8, budget=64),
        # Re-sampled trees of a small batch over a vocabulary that is hot as a whole.
        dict(name="resample_b3", kind="resample", B=3, S=5, V=32000, H=32000, k=4, budget=12),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_attn(rng, kind):
    while True:
        D = rng.choice([64, 128, 128])
        Hkv = rng.choice([2, 4, 8, 8, 16, 32])
        G = rng.choice([1, 2, 3, 4, 4, 5, 7, 8])
        N = _log_int(rng, 1, 256)
        B = _log_int(rng, 1, 16)
        hi = _log_int(rng, 64, 32768)
        lo = rng.choice([hi, hi // 2, hi // 4])
        c = dict(kind=kind, B=B, N=N, Hq=Hkv * G, Hkv=Hkv, D=D,
                 P=rng.choice([1, 2, 8, 16, 16, 16, 32, 64, 256]), lo=lo, hi=hi,
                 tree=rng.choice(["forest", "capped", "capped"]), ragged=False)
        if N >= 12 and rng.random() < 0.3:
            c.update(tree="fused", ragged=True)
        if G * N <= 2048 and _attn_work(c)[1] < 5e11 and B * hi * Hkv * D < 1.6e8:
            return c


def draw(rng):
    kind = rng.choice(["attn"] * 5 + ["step", "accept"] + ["lm"] * 3 + ["build"] * 2 + ["resample"])
    if kind == "attn":
        return _draw_attn(rng, "attn")
    if kind in ("step", "accept"):
        while True:
            c = _draw_attn(rng, kind)
            c["V"] = rng.choice([1000, 32000, 32000, 50257, 128256])
            if c["B"] * c["N"] * c["V"] < 1.3e8:
                return c
    if kind == "lm":
        while True:
            c = dict(kind="lm", B=_log_int(rng, 1, 16), N=_log_int(rng, 1, 64),
                     V=rng.choice([32000, 50257, 128256, 151936, _log_int(rng, 4000, 128000)]),
                     d=64 * _log_int(rng, 16, 128))
            if c["V"] * c["d"] < 5.3e8 and c["B"] * c["N"] * c["V"] * c["d"] < 5.3e11:
                return c
    V = rng.choice([32000, 32000, 50257, 128256, _log_int(rng, 4000, 128000)])
    return dict(kind=kind, B=_log_int(rng, 1, 16), S=rng.randint(2, 8), V=V,
                H=V if V <= 40000 else rng.choice([0, 32768, 32768, 20001]),
                k=rng.randint(2, 10), budget=_log_int(rng, 8, 64))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _trees(case, rng):
    """Parent links [B, N] (padding -1), node counts [B] and one child per node
    that an acceptable draft would continue with ([B, N], -1: none)."""
    B, N = case["B"], case["N"]
    kind = case.get("tree", "capped")
    parent = np.full((B, N), -1, dtype=np.int32)
    pick = np.full((B, N), -1, dtype=np.int64)
    counts = np.full(B, N, dtype=np.int32)
    for b in range(B):
        if kind == "forest":
            t = W.tree_uniform_forest(rng, N)
        elif kind == "frontier":
            t = W.tree_frontier_expansion(rng, 4, 3, N)
        elif kind == "fused":
            t = W.fusion_forest(rng, (max(1, N // 2), N - N // 4), (0, N // 4), 8)
        else:
            t = W.tree_random_depth_capped(rng, N, 10)
        counts[b] = len(t)
        parent[b, :len(t)] = t
        for i in range(len(t)):          # the last child of each node, with probability 0.6
            if t[i] >= 0 and rng.random() < 0.6:
                pick[b, t[i]] = i
    return parent, counts, pick


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _randn(shape, g):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)


def _draft_tokens(rng, B, N, V):
    return rng.integers(0, V, size=(B, N)).astype(np.int32)


def _int32(*shape):
    return torch.empty(shape, dtype=torch.int32, device="cuda")


def _accept_buffers(B, N):
    return dict(argmax_out=_int32(B, N), accept_len=_int32(B), accept_idx=_int32(B, N),
                bonus_token=_int32(B))


def _pages(rng, case, lens):
    """A pool with room for every sequence at its longest; each takes the pages
    of its prefix and its tree in a random order of the pool."""
    B, N, P = case["B"], case["N"], case["P"]
    per = -(-(case["hi"] + N) // P)
    perm = rng.permutation(B * per).astype(np.int32)
    table = np.full((B, per), -1, dtype=np.int32)
    for b in range(B):
        n = -(-(int(lens[b]) + N) // P)
        table[b, :n] = perm[b * per:b * per + n]
    return table, B * per


def _prepare_attn(case, seed):
    B, N, Hq, Hkv, D, P = (case[k] for k in ("B", "N", "Hq", "Hkv", "D", "P"))
    rng, g = np.random.default_rng(seed), _gen(seed)
    parent, counts, pick = _trees(case, rng)
    lens = rng.integers(case["lo"], case["hi"] + 1, size=B).astype(np.int32)
    page_table, num_pages = _pages(rng, case, lens)
    bf = lambda *shape: torch.randn(shape, generator=g, device="cuda", dtype=BF16)  # noqa: E731
    s = dict(case=case, q=bf(B, N, Hq, D), k_tree=bf(B, N, Hkv, D), v_tree=bf(B, N, Hkv, D),
             k_cache=bf(num_pages, P, Hkv, D), v_cache=bf(num_pages, P, Hkv, D),
             page_table=_dev(page_table), kv_len=_dev(lens), parent=_dev(parent),
             num_nodes=_dev(counts) if case["ragged"] else None, max_kv_len=int(lens.max()),
             out=torch.empty((B, N, Hq, D), dtype=BF16, device="cuda"),
             lse=torch.empty((B, N, Hq), dtype=torch.float32, device="cuda"),
             attn_ws=torch.empty(T.attention_workspace_size(B, N, Hq, Hkv, D),
                                 dtype=torch.uint8, device="cuda"))
    if case["kind"] != "attn":
        V = case["V"]
        draft = _draft_tokens(rng, B, N, V)
        logits = _randn((B, N, V), g)
        b, i = np.nonzero(pick >= 0)     # a node's picked child wins its argmax more often than not
        logits[_dev(b), _dev(i), _dev(draft[b, pick[b, i]].astype(np.int64))] += 5.0
        s.update(draft=_dev(draft), logits=logits, accept=_accept_buffers(B, N),
                 accept_ws=torch.empty(T.argmax_workspace_size(B, N, V), dtype=torch.uint8,
                                       device="cuda"))
    return s


def _prepare_lm(case, seed):
    B, N, V, d = (case[k] for k in ("B", "N", "V", "d"))
    rng, g = np.random.default_rng(seed), _gen(seed)
    parent, _, pick = _trees(case, rng)
    draft = _draft_tokens(rng, B, N, V)
    w = torch.randn((V, d), generator=g, device="cuda", dtype=BF16).mul_(0.02)
    h = _randn((B, N, d), g)
    b, i = np.nonzero(pick >= 0)         # the picked child's logit rises by 6
    wt = w[_dev(draft[b, pick[b, i]].astype(np.int64))].float()
    h[_dev(b), _dev(i)] += wt * (6.0 / wt.square().sum(-1, keepdim=True))
    return dict(case=case, hidden=h.to(BF16), w=w, draft=_dev(draft), parent=_dev(parent),
                accept=_accept_buffers(B, N),
                ws=torch.empty(T.lm_head_workspace_size(B, N, V, d), dtype=torch.uint8,
                               device="cuda"))


def _prepare_build(case, seed):
    B, S, V, H, k, budget = (case[x] for x in ("B", "S", "V", "H", "k", "budget"))
    rng, g = np.random.default_rng(seed), _gen(seed)
    hot_vocab = torch.randperm(V, generator=g, device="cuda")[:H].to(torch.int32)
    hot_index = torch.full((V,), -1, dtype=torch.int32, device="cuda")
    hot_index[hot_vocab.long()] = torch.arange(H, dtype=torch.int32, device="cuda")
    logits = _randn((B, S, V), g).mul_(2.5)
    table = torch.randn((H, H), generator=g, device="cuda", dtype=BF16) if H else None
    roots = rng.integers(0, V, size=B).astype(np.int32)
    if H:                                # three roots of four are hot tokens
        hot = rng.random(B) < 0.75
        roots[hot] = hot_vocab.cpu().numpy()[rng.integers(0, H, size=int(hot.sum()))]
    s = dict(case=case, logits=logits, roots=_dev(roots), table=table,
             hot_vocab=hot_vocab if H else None, hot_index=hot_index if H else None,
             outs=dict(parent=_int32(B, budget), token=_int32(B, budget),
                       joint=torch.empty((B, budget), dtype=torch.float32, device="cuda"),
                       num_nodes=_int32(B)),
             ws=torch.empty(T.tree_build_workspace_size(B, S, V, H, k), dtype=torch.uint8,
                            device="cuda"))
    if case["kind"] == "resample":       # the root and up to three accepted drafts
        s["accept_len"] = _dev(rng.integers(1, min(4, S) + 1, size=B).astype(np.int32))
    return s


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("attn", "step", "accept"):
        return _prepare_attn(case, seed)
    return _prepare_lm(case, seed) if kind == "lm" else _prepare_build(case, seed)


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def _attend(s):
    return T.tree_verify_attention(s["q"], s["k_tree"], s["v_tree"], s["k_cache"], s["v_cache"],
                                   s["page_table"], s["kv_len"], s["parent"],
                                   max_kv_len=s["max_kv_len"], num_nodes=s["num_nodes"],
                                   out=s["out"], lse=s["lse"], workspace=s["attn_ws"])


def _accept_and_compact(s):
    am, alen, aidx, bonus = T.tree_argmax_accept(s["logits"], s["draft"], s["parent"],
                                                 num_nodes=s["num_nodes"],
                                                 workspace=s["accept_ws"], **s["accept"])
    kc, vc = T.kv_compact_accepted(s["k_tree"], s["v_tree"], s["k_cache"], s["v_cache"],
                                   s["page_table"], s["kv_len"], aidx, alen)
    return dict(argmax=am, accept_len=alen, accept_idx=aidx, bonus=bonus, k_cache=kc, v_cache=vc)


def run(s):
    kind, case = s["case"]["kind"], s["case"]
    if kind == "attn":
        out, lse = _attend(s)
        return dict(out=out, lse=lse)
    if kind == "step":
        out, lse = _attend(s)
        return dict(out=out, lse=lse, **_accept_and_compact(s))
    if kind == "accept":
        return _accept_and_compact(s)
    if kind == "lm":
        am, alen, aidx, bonus = T.tree_lm_head_argmax_accept(
            s["hidden"], s["w"], s["draft"], s["parent"], workspace=s["ws"], **s["accept"])
        return dict(argmax=am, accept_len=alen, accept_idx=aidx, bonus=bonus)
    args = dict(k=case["k"], budget=case["budget"], workspace=s["ws"], **s["outs"])
    if kind == "build":
        par, tok, joint, nn = T.tree_build(s["logits"], s["roots"], s["table"], s["hot_vocab"],
                                           s["hot_index"], **args)
    else:
        par, tok, joint, nn = T.tree_resample(s["logits"], s["roots"], s["accept_len"],
                                              s["table"], s["hot_vocab"], s["hot_index"], r=1,
                                              **args)
    return dict(parent=par, token=tok, joint=joint, num_nodes=nn)


# ---------------------------------------------------------------------------
# necessary work, tolerances
# ---------------------------------------------------------------------------

def _attn_work(c):
    row = c["Hkv"] * c["D"] * 2
    L = c["B"] * (c["lo"] + c["hi"]) / 2          # prefix tokens, mean over the draws
    nodes = c["B"] * c["N"] * (0.75 if c["ragged"] else 1.0)
    keys = (c["lo"] + c["hi"]) / 2 + min(c["N"], 6)
    return (2 * row * (L + nodes) + nodes * c["Hq"] * (4 * c["D"] + 4) + 4 * L / c["P"] + 4 * nodes,
            4 * nodes * c["Hq"] * c["D"] * keys)


def _accept_work(c):
    nodes = c["B"] * c["N"] * (0.75 if c["ragged"] else 1.0)
    return 4 * nodes * c["V"] + 16 * nodes + 3 * c["B"] * c["Hkv"] * c["D"] * 8


def work(case):
    kind = case["kind"]
    by = fl = 0.0
    if kind in ("attn", "step"):
        by, fl = _attn_work(case)
    if kind in ("accept", "step"):
        by += _accept_work(case)
    if kind == "lm":
        R, V, d = case["B"] * case["N"], case["V"], case["d"]
        by, fl = 2 * d * (R + V) + 20 * R, 2.0 * R * V * d
    if kind in ("build", "resample"):
        B, S, V, H, k = (case[x] for x in ("B", "S", "V", "H", "k"))
        steps = [S] if kind == "build" else [S - a if S - a > 1 else 0
                                             for a in range(1, min(4, S) + 1)]
        rows = B * sum(steps) / len(steps)
        expanded = B * sum(1 + (n - 1) * k if n else 0 for n in steps) / len(steps)
        by = 4 * V * rows + (4 * V + 4 * H if H else 0) + 2 * H * expanded + 12 * B * case["budget"]
    return {"bytes": by, "flops": fl}


def tolerance(case):
    kind = case["kind"]
    if kind in ("attn", "step"):
        # bf16 probabilities and outputs, split sums in bf16 units of their result;
        # accepted tokens and copied rows stay the same
        return {"rel": 1.2e-2, "max": 0.1}
    if kind in ("build", "resample"):
        return {"rel": 1e-8, "max": 4e-7}      # fp64 decisions and sums, joint rounded to fp32
    if kind == "lm":
        # fp32 sums in another order: only logits within that rounding of each other may swap
        return {"rel": 0.0, "differ": 0.002}
    return "exact"


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

def _exact_attention(s):
    c = s["case"]
    B, N, Hq, Hkv, D, P = (c[k] for k in ("B", "N", "Hq", "Hkv", "D", "P"))
    G = Hq // Hkv
    out = torch.zeros((B, N, Hq, D), dtype=torch.float64, device="cuda")
    lse = torch.full((B, N, Hq), -math.inf, dtype=torch.float64, device="cuda")
    parent = s["parent"].cpu().numpy()
    lens = s["kv_len"].cpu().numpy()
    counts = s["num_nodes"].cpu().numpy() if s["num_nodes"] is not None else np.full(B, N)
    for b in range(B):
        n, L = int(counts[b]), int(lens[b])
        if n == 0:
            continue
        see = np.zeros((n, n), dtype=bool)
        for i in range(n):
            if parent[b, i] >= 0:
                see[i] = see[parent[b, i]]
            see[i, i] = True
        bias = torch.zeros((n, 1, L + n), dtype=torch.float64, device="cuda")
        bias[:, 0, L:].masked_fill_(~_dev(see), -math.inf)
        t = torch.arange(L, device="cuda")
        at = (s["page_table"][b].long()[t // P], t % P)
        for g in range(Hkv):
            k = torch.cat([s["k_cache"][at[0], at[1], g], s["k_tree"][b, :n, g]]).double()
            v = torch.cat([s["v_cache"][at[0], at[1], g], s["v_tree"][b, :n, g]]).double()
            q = s["q"][b, :n, g * G:(g + 1) * G].double().reshape(n * G, D)
            x = (q @ k.T).div_(math.sqrt(D)).view(n, G, L + n).add_(bias).view(n * G, L + n)
            m = x.amax(-1, keepdim=True)
            x.sub_(m).exp_()
            z = x.sum(-1, keepdim=True)
            out[b, :n, g * G:(g + 1) * G] = (x @ v).div_(z).view(n, G, D)
            lse[b, :n, g * G:(g + 1) * G] = (m + z.log()).view(n, G)
    return out, lse


def _exact_joint(s):
    """Joint probabilities of the kept nodes, in creation order, one expansion at a time."""
    c = s["case"]
    B, S, V, H, k, budget = (c[x] for x in ("B", "S", "V", "H", "k", "budget"))
    joint = torch.zeros((B, budget), dtype=torch.float64, device="cuda")
    roots = s["roots"].cpu().numpy()
    first = s["accept_len"].cpu().numpy() if c["kind"] == "resample" else np.zeros(B, dtype=int)
    hot_index = s["hot_index"].cpu().numpy() if H else None
    cols = s["hot_vocab"].long() if H else None
    for b in range(B):
        probs, frontier = [1.0], [(int(roots[b]), 1.0)]
        steps = range(first[b], S)
        if c["kind"] == "resample" and len(steps) <= 1:
            steps = []
        for i in steps:
            x = s["logits"][b, i].repeat(len(frontier), 1)
            for j, (tok, _) in enumerate(frontier):
                if H and hot_index[tok] >= 0:
                    x[j, cols] += s["table"][int(hot_index[tok])].float()
            top, ids = torch.sort(x, dim=-1, descending=True, stable=True)   # ties: lower id first
            x = x.double()
            lse = torch.logsumexp(x, dim=-1, keepdim=True)
            p = (top[:, :k].double() - lse).exp().cpu().numpy()
            ids = ids[:, :k].cpu().numpy()
            kids = [(int(ids[j, r]), frontier[j][1] * float(p[j, r]))
                    for j in range(len(frontier)) for r in range(k)]
            probs += [q for _, q in kids]
            frontier = sorted(kids, key=lambda t: -t[1])[:k]
        order = sorted(range(len(probs)), key=lambda i: (-probs[i], i))[:budget]
        kept = [probs[i] for i in sorted(order)]
        joint[b, :len(kept)] = torch.tensor(kept, dtype=torch.float64, device="cuda")
    return joint


def exact(case, seed):
    kind = case["kind"]
    if kind in ("accept", "lm"):
        return None                    # whole numbers and copied rows
    s = prepare(case, seed)
    if kind in ("build", "resample"):
        return dict(parent=None, token=None, joint=_exact_joint(s), num_nodes=None)
    out, lse = _exact_attention(s)
    r = dict(out=out, lse=lse)
    if kind == "step":
        r.update(argmax=None, accept_len=None, accept_idx=None, bonus=None, k_cache=None,
                 v_cache=None)
    return r
