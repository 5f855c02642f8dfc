"""The work a user of this library has it do, as cases that can be timed and compared.

A case is one call (or one step of a serving loop) over a paged K/V cache: some prefill chunks, some speculative
verify segments and some decodes, with a head shape and a page size.  The lengths of its sequences are drawn,
log-uniformly, from the bounds the case states; ``lengths`` is the seed they are drawn with.

Fields: heads_q, heads_kv, page (tokens per block-table entry);
prefills, prefill_lo .. prefill_hi (new tokens), cached_lo .. cached_hi (tokens already in the cache), share (prefills
come in pairs with the same cached prefix, as behind a prefix-cache hit); verifies, draft_lo .. draft_hi,
verify_ctx_lo .. verify_ctx_hi, tree (a token tree with its corner mask, else a chain); decodes,
decode_ctx_lo .. decode_ctx_hi; layers (calls over the same plan, each with its own cache, as the layers of a model's
step are); from_qkv (the call starts from the fused projection output: this step's K and V rows are written into the
cache first); replan (the step plans its batch, as every step of a serving loop does, and runs a copy-on-write copy
of a partly reused block).
"""
import math
import random

import numpy as np
import torch

from paper_2412_18106_amd import binding as X
from paper_2412_18106_amd import workloads as W

D = 128

BASE = {"heads_q": 32, "heads_kv": 8, "page": 128,
        "prefills": 0, "prefill_lo": 1, "prefill_hi": 1, "cached_lo": 0, "cached_hi": 0, "share": False,
        "verifies": 0, "draft_lo": 1, "draft_hi": 1, "verify_ctx_lo": 1, "verify_ctx_hi": 1, "tree": True,
        "decodes": 0, "decode_ctx_lo": 1, "decode_ctx_hi": 1,
        "layers": 1, "from_qkv": False, "replan": False, "lengths": 1}


def listed():
    return [
        # one user's chat: a single decode, one layer; nothing but latency
        dict(BASE, name="single_decode", page=16, decodes=1, decode_ctx_lo=900, decode_ctx_hi=1900, from_qkv=True),
        # the smallest batch with everything in it, at a small model's head shape
        dict(BASE, name="tiny_hybrid", heads_q=8, heads_kv=2, prefills=1, prefill_lo=128, prefill_hi=128,
             verifies=1, draft_lo=4, draft_hi=4, verify_ctx_lo=192, verify_ctx_hi=192,
             decodes=2, decode_ctx_lo=256, decode_ctx_hi=256),
        # a step of a lightly loaded server: a prompt's suffix behind a cached prefix, two dozen decodes, small
        # pages, planned anew, eight layers
        dict(BASE, name="serving_step", page=16, prefills=1, prefill_lo=150, prefill_hi=250, cached_lo=500, cached_hi=1000,
             decodes=24, decode_ctx_lo=100, decode_ctx_hi=2000, layers=8, from_qkv=True, replan=True),
        # several prompts of all lengths prefilled from nothing
        dict(BASE, name="prompts", page=16, prefills=8, prefill_lo=60, prefill_hi=4000, from_qkv=True),
        # one chunk of a long prompt, alone on the GPU
        dict(BASE, name="prefill_chunk", page=64, prefills=1, prefill_lo=1024, prefill_hi=1024,
             cached_lo=20000, cached_hi=24000, from_qkv=True),
        # speculative decoding with large token trees on long contexts, small batch
        dict(BASE, name="verify_long_trees", verifies=4, draft_lo=31, draft_hi=31,
             verify_ctx_lo=10000, verify_ctx_hi=20000),
        # decodes at a multi-head shape (no K/V sharing between heads)
        dict(BASE, name="decode_multi_head", heads_kv=32, decodes=8, decode_ctx_lo=2000, decode_ctx_hi=6000),
        # speculative decoding, large batch of small trees
        dict(BASE, name="verify_heavy", verifies=128, draft_lo=1, draft_hi=8, verify_ctx_lo=512, verify_ctx_hi=4096),
        # a prefill chunk riding along a batch of decodes, from the projection output
        dict(BASE, name="splitfuse", prefills=1, prefill_lo=512, prefill_hi=512, cached_lo=2048, cached_hi=2048,
             decodes=64, decode_ctx_lo=1024, decode_ctx_hi=8192, from_qkv=True),
        # prefix-cache hits: eight suffixes of 1024 tokens on four shared prefixes
        dict(BASE, name="prefix_prefill", prefills=8, prefill_lo=1024, prefill_hi=1024, cached_lo=4096, cached_hi=16384,
             share=True),
        # a large batch of decodes on long contexts
        dict(BASE, name="decode_large", page=32, decodes=128, decode_ctx_lo=2048, decode_ctx_hi=16384),
        # the largest: long prefill chunks, verify chains and decodes of a large model in one call
        dict(BASE, name="long_mixed", heads_q=64, prefills=2, prefill_lo=2048, prefill_hi=2048,
             cached_lo=32768, cached_hi=32768, verifies=16, draft_lo=4, draft_hi=4, verify_ctx_lo=256,
             verify_ctx_hi=32768, tree=False, decodes=256, decode_ctx_lo=256, decode_ctx_hi=32768),
    ]


def _log(rng, lo, hi):
    """An integer of [lo, hi], uniform over its logarithm."""
    return min(hi, max(lo, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def _span(rng, lo, hi):
    """Two such integers in order."""
    return sorted((_log(rng, lo, hi), _log(rng, lo, hi)))


def draw(rng):
    largest = work(listed()[-1])
    while True:
        c = dict(BASE)
        c["heads_q"], c["heads_kv"] = rng.choice([(32, 8), (32, 8), (32, 8), (64, 8), (32, 32), (8, 2)])
        c["page"] = rng.choice([16, 32, 64, 128])
        c["from_qkv"] = rng.random() < 0.5
        c["lengths"] = rng.randrange(1, 1 << 20)
        kind = rng.choice(["decode", "verify", "prompts", "cached", "mixed", "step"])
        if kind in ("decode", "mixed", "step"):
            c["decodes"] = _log(rng, 1, 256) if kind != "step" else _log(rng, 4, 64)
            c["decode_ctx_lo"], c["decode_ctx_hi"] = _span(rng, 64, 32768 if kind != "step" else 4096)
        if kind == "verify" or (kind == "mixed" and rng.random() < 0.5):
            c["verifies"] = _log(rng, 1, 128)
            c["draft_lo"], c["draft_hi"] = _span(rng, 1, 31)
            c["verify_ctx_lo"], c["verify_ctx_hi"] = _span(rng, 64, 32768)
            c["tree"] = rng.random() < 0.6
        if kind in ("prompts", "cached", "mixed", "step"):
            c["prefills"] = _log(rng, 1, 8) if kind != "step" else 1
            c["prefill_lo"], c["prefill_hi"] = _span(rng, 16, 4096 if kind != "step" else 512)
            if kind == "cached" or (kind != "prompts" and rng.random() < 0.6):
                c["cached_lo"], c["cached_hi"] = _span(rng, 64, 32768 if kind != "step" else 2048)
                c["share"] = kind == "cached" and rng.random() < 0.5
        if kind == "step":
            c["from_qkv"] = c["replan"] = True
            c["layers"] = _log(rng, 1, 8)
        w = work(c)
        if w["bytes"] <= largest["bytes"] and w["flops"] <= largest["flops"]:
            return c


def _specs(case):
    """The sequences of a case: workloads.SeqSpec entries, prefills first."""
    rng = random.Random(case["lengths"])
    tree_rng = np.random.default_rng(case["lengths"])
    specs = []
    for i in range(case["prefills"]):
        q = _log(rng, case["prefill_lo"], case["prefill_hi"])
        c = _log(rng, case["cached_lo"], case["cached_hi"]) if case["cached_hi"] else 0
        if case["share"] and i % 2:
            specs.append(W.SeqSpec(q, specs[-1].context_len, W.PREFILL, share_prefix_with=i - 1))
        else:
            specs.append(W.SeqSpec(q, c, W.PREFILL))
    for _ in range(case["verifies"]):
        q = _log(rng, case["draft_lo"], case["draft_hi"])
        c = _log(rng, case["verify_ctx_lo"], case["verify_ctx_hi"])
        if case["tree"]:
            specs.append(W.SeqSpec(q, c, W.VERIFY, W.MASK_TREE, W.random_tree(tree_rng, q)))
        else:
            specs.append(W.SeqSpec(q, c, W.VERIFY))
    for _ in range(case["decodes"]):
        specs.append(W.SeqSpec(1, _log(rng, case["decode_ctx_lo"], case["decode_ctx_hi"]), W.DECODE))
    return specs


def _layout(case, specs, rng):
    """Block table on a shuffled pool of blocks, the number of blocks, and the partly filled prefix blocks that a
    sequence shares by copy: (source block, destination block, rows)."""
    page = case["page"]
    need = [-(-(s.context_len + s.query_len) // page) for s in specs]
    shared = [s.context_len // page if s.share_prefix_with is not None else 0 for s in specs]
    used = sum(need) - sum(shared)
    blocks = used + max(2, used // 16)
    perm = rng.permutation(blocks).astype(np.int32)
    table = np.full((len(specs), max(need)), perm[used], dtype=np.int32)
    copies, cursor = [], 0
    for i, s in enumerate(specs):
        if shared[i]:
            table[i, :shared[i]] = table[s.share_prefix_with, :shared[i]]
        own = need[i] - shared[i]
        table[i, shared[i]:need[i]] = perm[cursor:cursor + own]
        cursor += own
        if s.share_prefix_with is not None and s.context_len % page:
            copies.append((int(table[s.share_prefix_with, shared[i]]), int(table[i, shared[i]]), s.context_len % page))
    # a block that stands in for the source of the step's copy-on-write copy: nobody else reads it
    return table, blocks, copies, int(perm[used + 1])


class _Plan:
    """A plan handle that is freed with the state."""

    def __init__(self, cfg, seqs):
        self.handle = X.xy_attn_plan_create(cfg, seqs)

    def __del__(self):
        X.xy_attn_plan_destroy(self.handle)


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    rng = np.random.default_rng(seed)
    hq, hkv, page, layers = case["heads_q"], case["heads_kv"], case["page"], case["layers"]
    specs = _specs(case)
    table, blocks, copies, spare = _layout(case, specs, rng)
    seqs, masks = W.specs_to_seqs(specs)
    tokens = sum(s.query_len for s in specs)

    # Q, K and V of unit variance: scores of unit variance behind the 1 / sqrt(D) scale
    def noise(*shape):
        return torch.empty(shape, dtype=torch.bfloat16, device=dev).normal_(generator=gen)

    st = {"layers": [], "seqs": seqs, "scale": 1.0 / math.sqrt(D), "hkv": hkv, "replan": case["replan"],
          "from_qkv": case["from_qkv"], "copies": []}
    for _ in range(layers):
        k, v = noise(blocks, hkv, page, D), noise(blocks, hkv, page, D)
        for src, dst, rows in copies:
            k[dst, :, :rows] = k[src, :, :rows]
            v[dst, :, :rows] = v[src, :, :rows]
        q = noise(tokens, hq + 2 * hkv, D) if case["from_qkv"] else noise(tokens, hq, D)
        st["layers"].append((q, k, v, torch.empty(tokens, hq, D, dtype=torch.bfloat16, device=dev)))
    if case["replan"] and specs[0].context_len:
        # the first sequence was admitted with a partial match: half of a page of its context is copied
        st["copies"] = [(spare, int(table[0, (specs[0].context_len - 1) // page]), max(1, page // 2))]
    st["table"] = torch.from_numpy(table).to(dev)
    st["masks"] = torch.from_numpy(masks.view(np.int32)).to(dev)
    st["cfg"] = X.xy_attn_default_config(hq, hkv, table.shape[1], block_size=page)
    st["plan"] = _Plan(st["cfg"], seqs)
    X.xy_attn_plan_upload(st["plan"].handle)
    st["workspace"] = torch.empty(max(16, X.xy_attn_plan_workspace_bytes(st["plan"].handle)), dtype=torch.uint8, device=dev)
    return st


def run(state):
    plan, table, masks, ws, scale = state["plan"].handle, state["table"], state["masks"], state["workspace"], state["scale"]
    if state["replan"]:
        X.xy_attn_plan_rebuild(plan, state["cfg"], state["seqs"])
        X.xy_attn_plan_upload_async(plan)
    for q, k, v, out in state["layers"]:
        X.xy_attn_copy_block_rows(state["copies"], state["hkv"], k, v)
        if state["from_qkv"]:
            X.xy_attn_run_fused_qkv(plan, q, k, v, table, masks, out, ws, scale)
        else:
            X.xy_attn_run(plan, q, k, v, table, masks, out, ws, scale)
    if state["from_qkv"]:       # the caches are written too
        return [(out, k, v) for _, k, v, out in state["layers"]]
    return [out for _, _, _, out in state["layers"]]


def work(case):
    specs = _specs(case)
    hq, hkv = case["heads_q"], case["heads_kv"]
    pairs = tokens = cached = entries = 0
    for s in specs:
        q, c = s.query_len, s.context_len
        if s.parents is not None:
            corner = sum(bin(int(w)).count("1") for w in W.pack_tree_mask(s.parents))
        else:
            corner = q * (q + 1) // 2
        pairs += q * c + corner
        tokens += q
        if s.share_prefix_with is None:
            cached += c
        entries += -(-(c + q) // case["page"])
    row = D * 2                                                     # bytes of one head of one token
    nbytes = 2 * tokens * hq * row + 2 * cached * hkv * row         # Q in, O out; K and V of the cached tokens
    nbytes += 2 * tokens * hkv * row * (2 if case["from_qkv"] else 1)   # this step's K and V: read, and written
    nbytes += 4 * entries
    if case["replan"] and specs[0].context_len:
        nbytes += 2 * 2 * max(1, case["page"] // 2) * hkv * row     # the copied rows, read and written
    return {"bytes": case["layers"] * nbytes, "flops": case["layers"] * 4 * D * hq * pairs}


def tolerance(case):
    # bf16 inputs and outputs, probabilities rounded to bf16, 32-bit sums: against the same in 64 bits, rel is
    # 1.7e-3 to 2.9e-3 over the cases (1.6e-3 of it the rounding of the outputs) and max up to 5.1e-2 (prompts
    # from nothing, where a row sees few keys); four times that
    return {"rel": 1.2e-2, "max": 0.2}
