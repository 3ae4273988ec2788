"""Performance cases of the draft-and-verify path, through its Python entry points.

A case is one call (or one short sequence of calls) that a decoding loop makes
per iteration, on seeded synthetic inputs that already live on the GPU:

  step     adapld_step, the whole iteration: lexical match, rerank or
           hidden-state fallback, draft tree, tree-masked verify attention
  verify   tree_verify_attn alone, the call of a loop that drafts elsewhere
  embed    semantic_topk_embed, the token-embedding fallback and its rerank
  paper    build_draft_tree_paper, branch tokens from the target's top tokens
           with reranked successors (embedding backoff for absent tokens)
  accept   accept_greedy, acceptance of the verified tree and K/V compaction
  lexical  lexical_match alone on long contexts
  ngram    the n-gram index of a batch of prompts: built, then 16 decoding
           iterations that each append 4 tokens and match

Contexts are Zipf draws with copied spans, hidden rows N(0, 1) with noisy
copies, attention tensors N(0, 1), as in ``paper_2606_05742_amd.synth`` (drawn
here on the GPU, since a case's inputs are made many times).  ``miss`` is the
number of sequences whose last token is new to the context, so that the
semantic fallback runs for exactly those.  Buffers start at zero, so entries
that a call leaves alone compare equal.
"""
import math

import numpy as np
import torch

import paper_2606_05742_amd as adapld
from paper_2606_05742_amd.binding import (OP_BUILD_DRAFT_TREE_PAPER, OP_SEMANTIC_TOPK_EMBED, OP_TREE_VERIFY_ATTN)

ZIPF_A = 1.1
D = 128   # head dimension


def _step(name, B, L, V, d, Hq, Hkv, n_max, k, W, S, miss, ragged=False, preceding=False, tau=None):
    c = dict(kind="step", B=B, L=L, V=V, d=d, Hq=Hq, Hkv=Hkv, n_max=n_max, k=k, W=W, S=S, miss=miss,
             ragged=ragged, preceding=preceding, tau=tau)
    return dict(c, name=name) if name else c


def listed():
    return [
        # One short chat turn on a 7B-class model with full multi-head
        # attention: launches and memory round trips are all that counts.
        _step("step_b1_l512_mha32", 1, 512, 32000, 4096, 32, 32, 3, 4, 4, 8, 1),
        # One user, a few thousand tokens, an 8B-class model with grouped heads.
        _step("step_b1_l4096_gqa32x8", 1, 4096, 128256, 4096, 32, 8, 4, 8, 4, 10, 1),
        # The benchmark's workload: a served batch of 16 at 8k tokens.
        _step("step_b16_l8192_gqa32x8", 16, 8192, 128256, 4096, 32, 8, 4, 8, 4, 12, 6),
        # Many short conversations on a 14B-class model, wide trees (136 nodes).
        _step("step_b64_l2048_gqa40x8", 64, 2048, 152064, 5120, 40, 8, 5, 8, 8, 16, 32),
        # Long-document batch on a 70B-class model: the largest sizes.
        _step("step_b8_l32768_gqa64x8", 8, 32768, 128256, 8192, 64, 8, 4, 16, 8, 8, 4),
        # A live server's batch: every sequence at another length, an odd
        # capacity, 7 query heads per kv head, Eq. (6) as printed, a threshold.
        _step("step_b24_l6007_ragged_gqa28x4", 24, 6007, 50000, 3584, 28, 4, 3, 10, 5, 6, 8, True, True, 0.05),
        # Verification of a single copied chain (prompt lookup): small trees,
        # so the call is one pass over the K/V cache.
        dict(name="verify_b32_l4096_chain16_gqa32x8", kind="verify", B=32, L=4096, Hq=32, Hkv=8, W=1, S=15,
             ragged=False),
        # The token-embedding fallback in place of the hidden-state one.
        dict(name="embed_b16_l8192_v128256", kind="embed", B=16, L=8192, V=128256, d=4096, n_max=4, k=8, miss=6,
             ragged=False),
        # The paper's draft construction on the same batch, a successor after
        # every branch token.
        dict(name="paper_tree_b16_l8192_w4", kind="paper", B=16, L=8192, V=128256, d=4096, n_max=4, k=8, W=4, S=12,
             miss=6, ragged=False),
        # The end of an iteration: acceptance, kept K/V moved into the cache.
        dict(name="accept_b16_l4096_t52", kind="accept", B=16, L=4096, Hkv=8, W=4, S=12),
        # Lexical match alone over contexts of 128k tokens.
        dict(name="lexical_b4_l131072", kind="lexical", B=4, L=131072, V=128256, n_max=4, miss=1, ragged=True),
        # A batch of prompts enters: its n-gram index is built and then used
        # for 16 decoding iterations.
        dict(name="ngram_b16_l8192_n4", kind="ngram", B=16, L=8192, V=128256, n_max=4),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# Largest work of a drawn case: bytes and flops of the largest listed step.
_MAX_BYTES, _MAX_FLOPS = 3.2e9, 3.4e11


def draw(rng):
    while True:
        kind = rng.choice(["step"] * 5 + ["verify", "verify", "embed", "paper", "accept", "lexical", "ngram"])
        B, L = _log_int(rng, 1, 64), _log_int(rng, 512, 32768)
        V = rng.choice([32000, 50000, 128256, 152064])
        d = rng.choice([1024, 2048, 3584, 4096, 5120, 8192])
        Hq, Hkv = rng.choice([(32, 32), (32, 8), (40, 8), (64, 8), (28, 4), (16, 16), (8, 2)])
        n_max, k, W, S = rng.randint(1, 8), rng.choice([4, 8, 10, 16]), rng.randint(1, 8), rng.randint(3, 16)
        ragged = rng.random() < 0.6
        miss = rng.randint(0, B)
        if kind == "step":
            c = _step(None, B, L, V, d, Hq, Hkv, n_max, k, W, S, miss, ragged, rng.random() < 0.4,
                      rng.choice([None, 0.05]))
        elif kind == "verify":
            c = dict(kind=kind, B=B, L=L, Hq=Hq, Hkv=Hkv, W=W, S=S, ragged=ragged)
        elif kind == "embed":
            c = dict(kind=kind, B=B, L=L, V=V, d=d, n_max=n_max, k=k, miss=miss, ragged=ragged)
        elif kind == "paper":
            c = dict(kind=kind, B=B, L=L, V=V, d=d, n_max=n_max, k=k, W=W, S=S, miss=miss, ragged=ragged)
        elif kind == "accept":
            c = dict(kind=kind, B=B, L=min(L, 8192), Hkv=Hkv, W=W, S=S)
        elif kind == "lexical":
            c = dict(kind=kind, B=B, L=_log_int(rng, 512, 131072), V=V, n_max=n_max, miss=miss, ragged=ragged)
        else:
            c = dict(kind=kind, B=min(B, 16), L=min(L, 8192), V=V, n_max=min(n_max, 4))
        w = work(c)
        bank = 2 * B * L * c["d"] if "d" in c else 0
        if w["bytes"] <= _MAX_BYTES and w["flops"] <= _MAX_FLOPS and bank <= 4.4e9:
            return c


# ---------------------------------------------------------------------- inputs

def _misses(c, b):
    return (b + 1) * c["miss"] // c["B"] > b * c["miss"] // c["B"]


def _lens(c, rng):
    B, L = c["B"], c["L"]
    if not c["ragged"]:
        return np.full(B, L, np.int32)
    return rng.integers(max(L // 3, 64), L + 1, B).astype(np.int32)


def _tokens(c, lens, rng, L_stride, misses):
    """Zipf draws with 40 % of the positions copied from earlier spans of 4 to
    64 tokens; a missing sequence ends on a token absent from it, any other on
    a copy of an earlier span of 1 to 2*n_max tokens.  Also returns, per
    position, the position whose hidden row it repeats."""
    cdf = np.cumsum(np.arange(1, c["V"] + 1, dtype=np.float64) ** -ZIPF_A)
    cdf /= cdf[-1]
    B = len(lens)
    tok = np.zeros((B, L_stride), np.int32)
    root = np.tile(np.arange(L_stride, dtype=np.int64), (B, 1))
    for b in range(B):
        L = int(lens[b])
        t, r = tok[b], root[b]
        t[:L] = np.searchsorted(cdf, rng.random(L), side="right").clip(max=c["V"] - 1)
        n = int(0.4 * L / 34) + 1
        ln = rng.integers(4, 65, n).clip(max=L // 4)
        for l, u, v in zip(ln, rng.random(n), rng.random(n)):
            at = int(l + u * (L - 2 * l))
            s = int(v * (at - l + 1))
            t[at:at + l] = t[s:s + l]
            r[at:at + l] = r[s:s + l]
        if misses[b]:
            seen = np.zeros(L + 1, bool)
            seen[t[:L - 1][t[:L - 1] <= L]] = True
            t[L - 1] = int(np.flatnonzero(~seen)[0])
            r[L - 1] = r[int(rng.integers(0, L - 1))]
        else:
            l = int(rng.integers(1, 2 * c["n_max"] + 1))
            s = int(rng.integers(0, L - 2 * l))
            t[L - l:L] = t[s:s + l]
            r[L - l:L] = r[s:s + l]
    return tok, root


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _randn(g, *shape):
    """bf16 N(0, 1), drawn in slices of the first axis."""
    out = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    for x in out:
        x.normal_(generator=g)
    return out


def _bank(g, root, d):
    """Hidden rows: N(0, 1), a copied position its source's row + 0.1 N(0, 1)."""
    B, L = root.shape
    bank = _randn(g, B, L, d)
    for b in range(B):
        src = torch.from_numpy(root[b])
        at = torch.nonzero(src != torch.arange(L)).flatten().cuda()
        rows = bank[b, src.cuda()[at]].float()
        bank[b, at] = (rows + 0.1 * torch.randn(rows.shape, generator=g, device="cuda")).bfloat16()
    return bank


def _zeros(dtype, *shape):
    return torch.zeros(shape, dtype=dtype, device="cuda")


def _i32(*shape):
    return _zeros(torch.int32, *shape)


def _chains(B, W, S, counts):
    """W chains of S+1 nodes, the first counts[b] nodes of them: parent, depth
    and ancestor-or-self mask rows, as numpy arrays."""
    T_max = W * (S + 1)
    nw = (T_max + 63) // 64
    u = np.arange(T_max)
    depth = (u % (S + 1)).astype(np.int32)
    parent = np.where(depth == 0, -1, u - 1).astype(np.int32)
    rows = np.zeros((T_max, nw * 64), bool)
    for i in range(T_max):
        rows[i, i - depth[i]:i + 1] = True
    mask = np.packbits(rows, axis=1, bitorder="little").view(np.int64)
    live = u[None, :] < np.asarray(counts)[:, None]
    return (np.where(live, parent, 0).astype(np.int32), np.where(live, depth, 0).astype(np.int32),
            np.where(live[:, :, None], mask[None], 0).astype(np.int64))


def _attention(c, g, B, L, T_max):
    Hq, Hkv = c["Hq"], c["Hkv"]
    return dict(q=_randn(g, B, T_max, Hq, D), k_ctx=_randn(g, B, Hkv, L, D), v_ctx=_randn(g, B, Hkv, L, D),
                k_tree=_randn(g, B, T_max, Hkv, D), v_tree=_randn(g, B, T_max, Hkv, D))


def _retrieval(c, seed):
    """Contexts, hidden bank and the lexical result of a step's retrieval."""
    rng = np.random.default_rng(seed)
    lens = _lens(c, rng)
    tok, root = _tokens(c, lens, rng, c["L"], [_misses(c, b) for b in range(c["B"])])
    s = dict(tokens=torch.from_numpy(tok).cuda(), lens=torch.from_numpy(lens).cuda())
    s["bank"] = _bank(_gen(seed), root, c["d"])
    return s


def _embeddings(V, d):
    """One model's embedding table: clusters of rows with cosine about 0.9
    inside a cluster and about 0 between clusters."""
    g = _gen(1234)
    centers = torch.randn((1024, d), generator=g, device="cuda")
    emb = torch.empty((V, d), dtype=torch.bfloat16, device="cuda")
    for lo in range(0, V, 32768):
        i = torch.arange(lo, min(lo + 32768, V), device="cuda")
        emb[i] = (centers[i % 1024] + 0.35 * torch.randn((len(i), d), generator=g, device="cuda")).bfloat16()
    return emb


EMB_TAU = 0.5


def prepare(case, seed):
    c = case
    kind, B, L = c["kind"], c["B"], c["L"]
    if kind == "step":
        s = _retrieval(c, seed)
        T_max = c["W"] * (c["S"] + 1)
        att = _attention(c, _gen(seed + 1), B, L, T_max)
        buf = adapld.StepBuffers.allocate(B, L, c["d"], c["k"], T_max, c["Hq"], c["Hkv"], D)
        for t in vars(buf).values():
            t.zero_()
        s["call"] = adapld.StepCall(s["tokens"], s["lens"], s["bank"], *att.values(), n_max=c["n_max"], k=c["k"],
                                    W=c["W"], S=c["S"], tau=c["tau"], preceding=c["preceding"], buffers=buf)
        s["att"] = att
        return dict(s, case=c)
    rng = np.random.default_rng(seed)
    if kind == "verify":
        T_max = c["W"] * (c["S"] + 1)
        lens = _lens(c, rng)
        # every sequence keeps its first branch, most keep all of them
        counts = np.array([(c["S"] + 1) * (c["W"] if rng.random() < 0.7 else 1) for _ in range(B)], np.int32)
        _, _, mask = _chains(B, c["W"], c["S"], counts)
        s = _attention(c, _gen(seed), B, L, T_max)
        need = adapld.workspace_bytes(OP_TREE_VERIFY_ATTN, B, L, 0, 0, T_max, c["Hq"], c["Hkv"], D)
        return dict(s, case=c, lens=torch.from_numpy(lens).cuda(), counts=torch.from_numpy(counts).cuda(),
                    mask=torch.from_numpy(mask).cuda(), out=_zeros(torch.bfloat16, B, T_max, c["Hq"], D),
                    lse=_zeros(torch.float32, B, c["Hq"], T_max), ws=_zeros(torch.uint8, max(need, 16)))
    if kind in ("embed", "paper"):
        s = _retrieval(c, seed)
        s["emb"] = _embeddings(c["V"], c["d"])
        k = c["k"]
        s["cand"] = (_i32(B, L), _i32(B), _i32(B))
        adapld.lexical_match(s["tokens"], s["lens"], c["n_max"], cand_pos=s["cand"][0], cand_count=s["cand"][1],
                             match_n=s["cand"][2])
        top = dict(topk_pos=_i32(B, k), topk_score=_zeros(torch.float32, B, k), topk_count=_i32(B), kind=_i32(B))
        if kind == "embed":
            need = adapld.workspace_bytes(OP_SEMANTIC_TOPK_EMBED, B, L, c["d"], k)
        else:
            adapld.semantic_topk(s["bank"], s["lens"], s["cand"][0], s["cand"][1], k, **top)
            W, T_max = c["W"], c["S"] + 1 + 2 * c["W"]
            # the target's top tokens: slot 0 the copy token, the others
            # tokens of the context, the last one (W > 1) often absent from it
            tok = s["tokens"]
            g = _gen(seed + 2)
            idx = torch.rand((B, L, W), generator=g, device="cuda") * (s["lens"].view(B, 1, 1) - 1)
            table = torch.gather(tok.view(B, L, 1).expand(B, L, W), 1, idx.long())
            table[:, :-1, 0] = tok[:, 1:]
            if W > 1:
                table[:, :, W - 1] = torch.randint(0, c["V"], (B, L), generator=g, device="cuda")
            s["table"] = table.to(torch.int32).contiguous()
            s["tree"] = dict(node_token=_i32(B, T_max), node_parent=_i32(B, T_max), node_depth=_i32(B, T_max),
                             node_src=_i32(B, T_max), node_count=_i32(B),
                             tree_mask=_zeros(torch.int64, B, T_max, (T_max + 63) // 64))
            need = adapld.workspace_bytes(OP_BUILD_DRAFT_TREE_PAPER, B, L, c["d"], W)
        return dict(s, case=c, top=top, ws=_zeros(torch.uint8, max(need, 16)))
    if kind == "accept":
        W, S, Hkv = c["W"], c["S"], c["Hkv"]
        T = W * (S + 1)
        parent, depth, mask = _chains(B, W, S, np.full(B, T))
        token = np.stack([rng.permutation(T) + 100 for _ in range(B)]).astype(np.int32)
        # the target agrees with a random prefix of a random branch
        nxt = rng.integers(0, 100, (B, T + 1)).astype(np.int32)
        for b in range(B):
            at, keep = int(rng.integers(0, W)) * (S + 1), int(rng.integers(0, S + 2))
            if keep:
                nxt[b, 0] = token[b, at]
                nxt[b, at + 1:at + keep] = token[b, at + 1:at + keep]
        g = _gen(seed)
        up = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
        return dict(case=c, token=up(token), parent=up(parent), depth=up(depth), mask=up(mask),
                    count=up(np.full(B, T, np.int32)), nxt=up(nxt),
                    lens=up(rng.integers(L // 2, L + 1, B).astype(np.int32)),
                    k_tree=_randn(g, B, T, Hkv, D), v_tree=_randn(g, B, T, Hkv, D),
                    k_ctx=_zeros(torch.bfloat16, B, Hkv, L + T + 1, D),
                    v_ctx=_zeros(torch.bfloat16, B, Hkv, L + T + 1, D),
                    out=dict(accept_len=_i32(B), accept_nodes=_i32(B, T), out_tokens=_i32(B, T + 1)))
    if kind == "lexical":
        lens = _lens(c, rng)
        tok, _ = _tokens(c, lens, rng, L, [_misses(c, b) for b in range(B)])
        return dict(case=c, tokens=torch.from_numpy(tok).cuda(), lens=torch.from_numpy(lens).cuda(),
                    out=dict(cand_pos=_i32(B, L), cand_count=_i32(B), match_n=_i32(B)))
    if kind == "ngram":
        iters, m = 16, 4
        cap = L + iters * m
        lens = np.full(B, cap, np.int32)
        tok, _ = _tokens(c, lens, rng, cap, [False] * B)
        for b in range(B):   # each iteration appends tokens copied from earlier
            for at in range(L, cap, m):
                src = int(rng.integers(0, at - m))
                tok[b, at:at + m] = tok[b, src:src + m]
        return dict(case=c, tokens=torch.from_numpy(tok).cuda(), index=adapld.NgramIndex(B, cap, c["n_max"]),
                    lens=[torch.full((B,), L + m * i, dtype=torch.int32, device="cuda") for i in range(iters + 1)],
                    cand_pos=_i32(B, cap), count=_i32(iters, B), n=_i32(iters, B))
    raise ValueError(kind)


# ------------------------------------------------------------------------ run

def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "step":
        o = s["call"]()
        return dict(cand_pos=o.cand_pos, cand_count=o.cand_count, match_n=o.match_n, topk_pos=o.topk_pos,
                    topk_score=o.topk_score, topk_count=o.topk_count, kind=o.kind, node_token=o.node_token,
                    node_parent=o.node_parent, node_depth=o.node_depth, node_src=o.node_src, node_count=o.node_count,
                    tree_mask=o.tree_mask, out=o.out, lse=o.lse)
    if kind == "verify":
        return adapld.tree_verify_attn(s["q"], s["k_ctx"], s["v_ctx"], s["k_tree"], s["v_tree"], s["lens"],
                                       s["counts"], s["mask"], out=s["out"], lse=s["lse"], ws=s["ws"])
    if kind == "embed":
        return adapld.semantic_topk_embed(s["bank"], s["tokens"], s["lens"], s["cand"][0], s["cand"][1], s["emb"],
                                          c["k"], EMB_TAU, ws=s["ws"], **s["top"])
    if kind == "paper":
        t = s["top"]
        return adapld.build_draft_tree_paper(s["tokens"], s["lens"], s["bank"], t["topk_pos"], t["topk_count"],
                                             t["kind"], s["table"], c["S"], emb=s["emb"], tau=EMB_TAU, ws=s["ws"],
                                             **s["tree"])
    if kind == "accept":
        got = adapld.accept_greedy(s["token"], s["parent"], s["depth"], s["count"], s["mask"], s["nxt"], s["lens"],
                                   k_tree=s["k_tree"], v_tree=s["v_tree"], k_ctx=s["k_ctx"], v_ctx=s["v_ctx"],
                                   **s["out"])
        return [*got, s["k_ctx"], s["v_ctx"]]
    if kind == "lexical":
        return adapld.lexical_match(s["tokens"], s["lens"], c["n_max"], **s["out"])
    s["index"].build(s["tokens"], s["lens"][0])
    for i in range(len(s["lens"]) - 1):
        s["index"].append_match(s["tokens"], s["lens"][i + 1], cand_pos=s["cand_pos"], cand_count=s["count"][i],
                                match_n=s["n"][i])
    return [s["cand_pos"], s["count"], s["n"]]


# ----------------------------------------------------------------------- work

def _attention_work(B, L, T_list, Hq, Hkv, S):
    byts = sum(4 * Hkv * D * (L + T) + 4 * Hq * D * T + 4 * Hq * T for T in T_list)
    flops = sum(4 * Hq * D * T * (L + (S + 2) / 2) for T in T_list)
    return byts, flops


def work(case):
    """Each input read once, each output written once.  A ragged batch counts
    two thirds of its capacity; a missing sequence drafts a full tree, any
    other at least one branch and one scored row."""
    c = case
    kind, B = c["kind"], c["B"]
    L = c["L"] * 2 // 3 if c.get("ragged") else c["L"]
    if kind in ("step", "verify"):
        W, S = c["W"], c["S"]
        if kind == "step":
            T_list = [(S + 1) * (W if _misses(c, b) else 1) for b in range(B)]
        else:
            T_list = [int((S + 1) * (0.7 * W + 0.3))] * B
        byts, flops = _attention_work(B, L, T_list, c["Hq"], c["Hkv"], S)
        if kind == "step":
            byts += 4 * B * L + 2 * c["d"] * (c["miss"] * L + 2 * (B - c["miss"]))
            flops += 4 * c["d"] * c["miss"] * L
        return {"bytes": byts, "flops": flops}
    if kind == "embed":
        # tokens read, one embedding row per distinct token (about a fifth of
        # the positions of a Zipf context), the candidates' ranking
        rows = c["miss"] * L // 5
        return {"bytes": 4 * B * L + 2 * c["d"] * (rows + 2 * B), "flops": 4 * c["d"] * rows}
    if kind == "paper":
        # tokens read once; per sequence at least the anchor's row and one
        # occurrence row per branch; an absent branch token reads one embedding
        # row per distinct token of its context
        rows = B * (1 + c["W"]) + (B * L // 5 if c["W"] > 1 else 0)
        return {"bytes": 4 * B * L + 2 * c["d"] * rows, "flops": 4 * c["d"] * rows}
    if kind == "accept":
        T = c["W"] * (c["S"] + 1)
        kept = (c["S"] + 1) // 2
        return {"bytes": B * (16 * T + 8 * T * ((T + 63) // 64) + 8 * kept + kept * c["Hkv"] * D * 2 * 4), "flops": 0}
    if kind == "lexical":
        return {"bytes": 4 * B * L, "flops": 0}
    # ngram: the tokens read once, one slot and one position per n-gram written
    return {"bytes": B * L * 4 + B * c["n_max"] * L * 20, "flops": 0}


def tolerance(case):
    if case["kind"] in ("step", "verify"):
        # bf16 outputs with bf16 probabilities; ranks may swap between ties
        return {"rel": 1.2e-2, "max": 0.1, "differ": 2e-3}
    if case["kind"] in ("embed", "paper"):
        return {"rel": 1e-5, "max": 1e-4, "differ": 2e-3}   # fp32 cosines
    return "exact"


# ---------------------------------------------------------------------- exact

def _suffix_matches(tok, L, n_max):
    """Candidate ends of the longest matching suffix, and its length."""
    t = tok[:L]
    ok = torch.ones(max(L - 1, 0), dtype=torch.bool, device=t.device)
    best, n_star = ok[:0], 0
    for n in range(min(n_max, L - 1)):
        eq = t[:L - 1] == t[L - 1 - n]
        ok = ok & torch.cat([torch.zeros(n, dtype=torch.bool, device=t.device), eq[:L - 1 - n]])
        if not bool(ok.any()):
            break
        best, n_star = torch.nonzero(ok).flatten(), n + 1
    return best, n_star


def _cosines(rows, q):
    out = []
    for r in rows.split(4096):
        r = r.double()
        out.append((r @ q) / (r.norm(dim=1) * q.norm()))
    return torch.cat(out) if out else torch.zeros(0, dtype=torch.float64, device=q.device)


def _rank(score, pos, k):
    """Indices of the k best: score descending, then position ascending."""
    order = torch.argsort(pos, stable=True)
    order = order[torch.argsort(score[order], descending=True, stable=True)]
    return order[:k]


def _attend(q, kc, vc, kt, vt, L, T, rows, Hkv, out, lse):
    """fp64 attention of one sequence's first T nodes; rows[u, v]: v visible to u."""
    G = q.shape[1] // Hkv
    for g in range(Hkv):
        K = torch.cat([kc[g, :L], kt[:T, g]]).double()
        Vv = torch.cat([vc[g, :L], vt[:T, g]]).double()
        for h in range(g * G, (g + 1) * G):
            s = (q[:T, h].double() @ K.t().contiguous()) / math.sqrt(D)
            s[:, L:] = s[:, L:].masked_fill(~rows, -math.inf)
            m = torch.logsumexp(s, dim=1)
            out[:T, h] = torch.exp(s - m[:, None]) @ Vv
            lse[h, :T] = m


def _visible(mask, T):
    """Boolean [T, T] from mask rows of 64-bit words."""
    bits = (mask[:T, :, None] >> torch.arange(64, device=mask.device)) & 1
    return bits.reshape(T, -1)[:, :T].bool()


def exact(case, seed):
    """The floating outputs in 64 bits (integers have one right answer and are
    None)."""
    c = case
    if c["kind"] not in ("step", "verify", "embed"):
        return None
    s = prepare(c, seed)
    B = c["B"]
    if c["kind"] == "verify":
        out = _zeros(torch.float64, *s["out"].shape)
        lse = _zeros(torch.float64, *s["lse"].shape)
        for b in range(B):
            T = int(s["counts"][b])
            _attend(s["q"][b], s["k_ctx"][b], s["v_ctx"][b], s["k_tree"][b], s["v_tree"][b], int(s["lens"][b]), T,
                    _visible(s["mask"][b], T), c["Hkv"], out[b], lse[b])
        return [out, lse]
    k = c["k"]
    score = _zeros(torch.float64, B, k)
    pre = 1 if c.get("preceding") else 0
    if c["kind"] == "step":
        W, S = c["W"], c["S"]
        T_max = W * (S + 1)
        a = s["att"]
        out = _zeros(torch.float64, B, T_max, c["Hq"], D)
        lse = _zeros(torch.float64, B, c["Hq"], T_max)
    for b in range(B):
        L = int(s["lens"][b])
        tok, bank = s["tokens"][b], s["bank"][b]
        cand, _ = _suffix_matches(tok, L, c["n_max"])
        hit = len(cand) > 0
        if not hit and c["kind"] == "embed":
            t = tok[:L - 1].long()
            uniq, inv = torch.unique(t, return_inverse=True)
            near = _cosines(s["emb"][uniq], s["emb"][tok[L - 1].long()].double())
            cand = torch.nonzero(near[inv] >= EMB_TAU).flatten()
        elif not hit:
            cand = torch.arange(L - 1, device=tok.device)
        cand = cand[cand >= pre]
        sc = _cosines(bank[cand - pre], bank[L - 1 - pre].double())
        best = _rank(sc, cand, k)
        if not hit and c["kind"] == "step" and c["tau"] is not None:
            best = best[sc[best] >= c["tau"]]
        score[b, :len(best)] = sc[best]
        if c["kind"] != "step":
            continue
        starts, heads = [], []
        for r in cand[best].tolist():
            head = int(tok[r + 1])
            if r <= L - 2 and head not in heads and len(heads) < W:
                heads.append(head)
                starts.append(min(S + 1, L - 1 - r))
        T = sum(starts)
        rows = torch.zeros((T, T), dtype=torch.bool, device="cuda")
        at = 0
        for n in starts:
            rows[at:at + n, at:at + n] = torch.tril(torch.ones((n, n), dtype=torch.bool, device="cuda"))
            at += n
        if T:
            _attend(a["q"][b], a["k_ctx"][b], a["v_ctx"][b], a["k_tree"][b], a["v_tree"][b], L, T, rows, c["Hkv"],
                    out[b], lse[b])
    if c["kind"] == "embed":
        return [None, score, None, None]
    names = ("cand_pos", "cand_count", "match_n", "topk_pos", "topk_score", "topk_count", "kind", "node_token",
             "node_parent", "node_depth", "node_src", "node_count", "tree_mask", "out", "lse")
    return {n: {"topk_score": score, "out": out, "lse": lse}.get(n) for n in names}
