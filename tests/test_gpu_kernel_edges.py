"""Small cases at the edges of single kernels and of the branches that choose between their variants, against the fp64
oracle.  Tolerance as for the parity tests: bf16 outputs of order one (half an ulp is 2^-9 relative), probabilities
rounded to bf16 (2^-9 relative, averaging down over the keys), fp32 sums: max-abs <= 2e-2, mean-abs <= 2e-3."""
import numpy as np
import pytest

from oracle import attention as A
from paper_2412_18106_amd import workloads as W

pytestmark = pytest.mark.gpu

MAX_ABS, MEAN_ABS = 2e-2, 2e-3
P, D_, V = W.PREFILL, W.DECODE, W.VERIFY


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("these tests need a GPU (run with -m gpu on an MI355X box)")
    from paper_2412_18106_amd import runner
    return runner


def assert_layout(db, **want):
    """The way the launches of a batch take (fields of xy_probe_layout; halved=True: any units handed out as halves)."""
    from paper_2412_18106_amd import binding as X
    layout = X.xy_probe_plan_layout(db.plan, db.cfg.num_workers)[0]
    for field, value in want.items():
        got = getattr(layout, field)
        assert (got > 0 if value is True else got == value), (field, got, value)


def run_and_check(gpu, b, what, plan_check=None, layout=None, **cfg):
    db = gpu.DeviceBatch(b, **cfg)
    try:
        assert_layout(db, **(layout or {}))
        if plan_check is not None:
            from paper_2412_18106_amd import binding as X
            plan_check(*X.xy_attn_plan_get(db.plan))
        got = db.run_numpy()
    finally:
        db.close()
    ref = A.attention_oracle(b.seqs, b.q, b.k_cache, b.v_cache, b.block_table, b.tree_masks,
                             num_q_heads=b.num_q_heads, num_kv_heads=b.num_kv_heads, block_size=b.block_size, scale=b.scale)
    assert not np.isnan(got).any(), f"{what}: NaN in output (row never written?)"
    err = np.abs(got.astype(np.float64) - ref)
    assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, f"{what}: max {err.max():.3e} mean {err.mean():.3e}"


@pytest.mark.parametrize("pieces", [2, 3, 4, 5, 8, 9, 12, 13, 17])
def test_merge_pass_over_the_number_of_pieces_and_rows(gpu, pieces):
    """The merge pass takes pieces in batches of eight, four or two and rows in groups of eight per workgroup: every
    remainder of either, one-row families and families of one row more than a group."""
    ctx = 128 * pieces - 5
    for hq, hkv, specs in ((1, 1, [W.SeqSpec(1, ctx, D_)]),
                           (6, 2, [W.SeqSpec(3, ctx - 3, V), W.SeqSpec(1, ctx, D_), W.SeqSpec(5, ctx - 7, V)]),
                           (4, 2, [W.SeqSpec(17, ctx - 20, V), W.SeqSpec(128, 128 * pieces - 128, V)])):
        b = W.make_custom(specs, hq, hkv, 900 + pieces)

        def plan_check(units, _offs, merges):
            assert pieces in set(merges["num_splits"].tolist())
        run_and_check(gpu, b, f"{pieces} pieces, {hq}/{hkv} heads", plan_check, split_kv_blocks=1,
                      verify_tile_tokens=128 if hq == 4 else 5)


@pytest.mark.parametrize("workers,wide,narrow", [(4, 4, 3), (4, 4, 40), (4, 5, 4), (4, 1, 3), (4, 1, 12), (4, 1, 13),
                                                 (4, 3, 50), (16, 3, 1), (16, 15, 70), (1, 1, 9)])
@pytest.mark.parametrize("heads,tokens,row_tiles", [(4, 32, 1), (3, 85, 2)])
def test_first_draws_from_the_shared_list(gpu, heads, tokens, row_tiles, workers, wide, narrow):
    """Entries of the shared list are reserved for workers without wide units; the others draw four at once.  No free
    worker, one, most; fewer entries than reserved, exactly as many, one more; three launches (the last workgroup
    puts the counters back).  Wide units of 128 rows and of 85 x 3, neither of which is ever halved; narrow ones that are too
    short for teams where these could take them."""
    import torch
    from paper_2412_18106_amd import binding as X
    ctx = (100, 37) if narrow > 2 * (workers - wide) else (30, 20)
    specs = [W.SeqSpec(tokens, 40 + 30 * i, P) for i in range(wide)] + [W.SeqSpec(1, ctx[0] + ctx[1] * i, D_) for i in range(narrow)]
    b = W.make_custom(specs, heads, 1, 77)
    ref = A.attention_oracle(b.seqs, b.q, b.k_cache, b.v_cache, b.block_table, b.tree_masks, num_q_heads=heads,
                             num_kv_heads=1, block_size=b.block_size, scale=b.scale)
    db = gpu.DeviceBatch(b, num_workers=workers, split_kv_blocks=0)
    try:
        units, offs, _ = X.plan_arrays(db.plan, workers)
        assert len(units) == wide + narrow and offs[workers] == wide
        assert_layout(db, row_tiles=row_tiles, halved=0, narrow_team=0)
        first = db.run_numpy()
        err = np.abs(first.astype(np.float64) - ref)
        assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS
        for _ in range(2):
            assert np.array_equal(db.run_numpy(), first)
        torch.cuda.synchronize()
    finally:
        db.close()


def two_halves(g):
    """Most tokens of g heads that make a unit of at most 256 rows which goes out as halves of at most 128."""
    return max(t for t in range(1, 256 // g + 1) if -(-t // 2) * g <= 128)


# where every large unit finds an idle worker, it is handed out as two halves to wavefronts of one row tile; with one
# worker none is idle and the wavefronts hold two
WAYS = [(256, dict(row_tiles=1, halved=True)), (1, dict(row_tiles=2, halved=0))]


@pytest.mark.parametrize("workers,layout", WAYS)
@pytest.mark.parametrize("hq,hkv", [(1, 1), (3, 1), (5, 1), (14, 2), (24, 1)])
def test_wide_units_row_mapping_through_lds(gpu, hq, hkv, workers, layout):
    """Q enters and O leaves a wide unit in groups of four rows (row = token x heads + head): group sizes that are no
    power of two, row counts that end inside a group of four, inside a 32-row tile and at a wavefront's first row;
    split (partial results) and whole; one and two row tiles."""
    g = hq // hkv
    most = two_halves(g) if workers > 1 else 256 // g
    tokens = [max(33, 33 // g), -(-65 // g), most, most + 3]
    b = W.make_custom([W.SeqSpec(t, 30 + 70 * i, P) for i, t in enumerate(tokens)], hq, hkv, 31 + hq)
    run_and_check(gpu, b, f"{hq}/{hkv} heads, whole", layout=layout, split_kv_blocks=0, num_workers=workers, prefill_tile_tokens=most)
    b = W.make_custom([W.SeqSpec(t, 300 + 70 * i, V) for i, t in enumerate(tokens)], hq, hkv, 41 + hq)
    run_and_check(gpu, b, f"{hq}/{hkv} heads, split", layout=layout, split_kv_blocks=1, num_workers=workers, verify_tile_tokens=most)


@pytest.mark.parametrize("workers,tokens,layout", [(256, 37, dict(row_tiles=1, halved=0))] +
                         [(workers, 70, layout) for workers, layout in WAYS])
@pytest.mark.parametrize("dim", ["token", "head"])
def test_wide_units_far_strides_of_q_and_out(gpu, dim, workers, tokens, layout):
    """Row offsets of Q and O are 32-bit while the strides stay below 2^21 elements, 64-bit from there on."""
    import torch
    from paper_2412_18106_amd import binding as X
    b = W.make_custom([W.SeqSpec(tokens, 150, P), W.SeqSpec(1, 90, D_)], 2, 1, 5)
    db = gpu.DeviceBatch(b, num_workers=workers, split_kv_blocks=0)
    try:
        assert_layout(db, **layout)
        want = db.run_numpy()
        t = b.total_q
        for stride in ((1 << 21) - 8, 1 << 21):
            ts, hs = (stride, 128) if dim == "token" else (128, stride)
            size = (t - 1) * ts + hs + 128
            q, out = (torch.zeros(size, dtype=torch.bfloat16, device="cuda").as_strided((t, 2, 128), (ts, hs, 1)) for _ in range(2))
            q.copy_(db.q)
            X.xy_attn_run(db.plan, q, db.k_cache, db.v_cache, db.block_table, db.tree_masks, out, db.workspace, b.scale)
            assert np.array_equal(out.float().cpu().numpy(), want), stride
    finally:
        db.close()


@pytest.mark.parametrize("hq,hkv,tokens", [(1, 1, 1), (4, 1, 1), (3, 1, 2), (5, 1, 6), (8, 1, 4), (31, 1, 1), (32, 1, 1), (4, 2, 3)])
def test_narrow_units_of_few_slices(gpu, hq, hkv, tokens):
    """Narrow units of one, two, three and more 32-key slices, ends inside a slice and right at one, rows from one to 32 in
    groups of four; whole, cut, and three times as many through one worker (the ways a launch can take are in
    test_ways_of_processing_narrow_units)."""
    specs = [W.SeqSpec(tokens, max(0, keys - tokens), V) for keys in (tokens, 31, 32, 33, 63, 64, 65, 95, 96, 97, 129, 200, 300)]
    run_and_check(gpu, W.make_custom(specs, hq, hkv, 11 * hq + tokens), f"{hq}/{hkv} heads, {tokens} tokens", split_kv_blocks=0)
    run_and_check(gpu, W.make_custom(specs, hq, hkv, 12 * hq + tokens), f"{hq}/{hkv} heads, {tokens} tokens, split", split_kv_blocks=1)
    run_and_check(gpu, W.make_custom(specs * 3, hq, hkv, 13 * hq + tokens), f"{hq}/{hkv} heads, {tokens} tokens, one worker",
                  split_kv_blocks=0, num_workers=1)


def _poison(b):
    """NaN and infinities in every slot of the caches that no sequence of the batch owns."""
    patterns = np.array([0x7FC0, 0x7F80, 0xFF80, 0xFFC1], dtype=np.uint16)
    bs = b.block_size
    owned = np.zeros((b.k_cache.shape[0], bs), dtype=bool)
    for i, (q, c, *_rest) in enumerate(b.seqs):
        for j in range(c + q):
            owned[b.block_table[i, j // bs], j % bs] = True
    blk, slot = np.nonzero(~owned)
    fill = patterns[(blk + slot)[:, None, None] % 4]
    b.k_cache[blk, :, slot] = fill
    b.v_cache[blk, :, slot] = fill[::-1]


@pytest.mark.parametrize("workers,layout", WAYS)
@pytest.mark.parametrize("bs", [16, 32, 128])
@pytest.mark.parametrize("hq", [4, 8])
def test_wide_units_of_less_than_one_step_ignore_what_lies_behind_them(gpu, bs, hq, workers, layout):
    """A wide unit of fewer than 32 keys has one step, which is its first and its last: V rows behind the last key must
    not meet the zero probabilities of the step before the first (0 x NaN).  Prompts from nothing, a tree of 20 tokens,
    the last piece of a cut family with 1, 17 and 31 keys; one step and one key more."""
    tree20 = W.random_tree(np.random.default_rng(3), 20)
    whole = [W.SeqSpec(n, 0, P) for n in (9, 20, 31, 32, 33)] + [W.SeqSpec(20, 0, V, W.MASK_TREE, tree20), W.SeqSpec(20, 5, V)]
    cut = [W.SeqSpec(20, 128 + last - 20, V) for last in (1, 17, 31, 32, 33)] + [W.SeqSpec(40, 128 + 17 - 40, V)]
    for name, specs, cfg in (("whole", whole, dict(verify_tile_tokens=256 // hq, split_kv_blocks=0)),
                             ("cut", cut, dict(verify_tile_tokens=256 // hq, split_kv_blocks=1))):
        b = W.make_custom(specs, hq, 1, 60 + hq, block_size=bs)
        cfg["num_workers"] = workers
        db = gpu.DeviceBatch(b, **cfg)
        base = db.run_numpy()
        db.close()
        _poison(b)

        def plan_check(units, _offs, _merges):
            rows = units["q_count"] * units["head_count"]
            keys = np.array([min(128 * u["kv_block_end"], b.seqs[u["seq"]][0] + b.seqs[u["seq"]][1]) - 128 * u["kv_block_begin"] for u in units])
            assert ((rows > 32) & (keys < 32)).sum() >= 3
        run_and_check(gpu, b, f"{name}, {hq} heads, pages of {bs}", plan_check, layout, **cfg)
        db = gpu.DeviceBatch(b, **cfg)
        assert np.array_equal(db.run_numpy(), base), name
        db.close()


@pytest.mark.parametrize("pieces", [2, 3, 4, 5, 6, 7, 8, 9, 11, 13])
def test_merge_pass_keeps_an_infinity_of_the_last_piece(gpu, pieces):
    """The merge pass fills its batches of two, four or eight pieces up: what stands in for a piece must not turn an
    infinite accumulator into a NaN (0 x Inf).  One decode row, an infinite V element at its last key."""
    b = W.make_custom([W.SeqSpec(1, 128 * pieces - 2, D_)], 1, 1, 300 + pieces)
    last = b.seqs[0][1]
    b.v_cache[b.block_table[0, last // 128], 0, last % 128, 5] = 0x7F80
    db = gpu.DeviceBatch(b, split_kv_blocks=1)
    try:
        got = db.run_numpy()
    finally:
        db.close()
    ref = A.attention_oracle(b.seqs, b.q, b.k_cache, b.v_cache, b.block_table, b.tree_masks, num_q_heads=1, num_kv_heads=1,
                             block_size=b.block_size, scale=b.scale)
    assert np.isposinf(ref[0, 0, 5]) and np.isposinf(got[0, 0, 5])
    others = np.arange(128) != 5
    assert np.abs(got[0, 0, others] - ref[0, 0, others]).max() <= MAX_ABS


def test_merge_pass_of_more_workgroups_than_one_launch_takes(gpu):
    """A launch has fewer than 2^32 threads, 2^24 workgroups of the merge pass: 257 decodes of 65536 heads on two tiles
    each are 2^24 + 65536 families of one row.  Every head reads the same K/V and every token has the same Q rows (strides
    of zero), so that the result is the same for every token."""
    import torch
    from paper_2412_18106_amd import binding as X
    heads, n, keys = 65536, 257, 129
    cfg = X.xy_attn_default_config(heads, heads, 2, split_kv_blocks=1, assign_policy=X.XY_ASSIGN_SNAKE)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    q1 = torch.empty(heads, 128, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    k1, v1 = (torch.empty(2, 1, 128, 128, dtype=torch.bfloat16, device="cuda").normal_(generator=gen) for _ in range(2))
    out = torch.full((n, heads, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    table = torch.tensor([[1, 0]] * n, dtype=torch.int32, device="cuda")
    plan = X.xy_attn_plan_create(cfg, [(1, keys - 1, X.XY_DECODE, 0, 0)] * n)
    try:
        ws = torch.empty(X.xy_attn_plan_workspace_bytes(plan), dtype=torch.uint8, device="cuda")
        X.xy_attn_run(plan, q1.expand(n, heads, 128), k1.expand(2, heads, 128, 128), v1.expand(2, heads, 128, 128), table, None,
                      out, ws, 128 ** -0.5)
        torch.cuda.synchronize()
    finally:
        X.xy_attn_plan_destroy(plan)
    k, v = (torch.cat([x[1, 0], x[0, 0, :1]]).float() for x in (k1, v1))
    ref = torch.softmax((q1.float() @ k.t().contiguous()) * 128 ** -0.5, -1) @ v
    err = (out[0].float() - ref).abs()
    assert float(err.max()) <= MAX_ABS and float(err.mean()) <= MEAN_ABS      # (a NaN fails both)
    assert all(torch.equal(out[i], out[0]) for i in range(1, n))


@pytest.mark.parametrize("hq,hkv,tokens", [(1, 1, 1), (4, 1, 1), (5, 1, 6), (8, 1, 4), (4, 2, 8), (32, 1, 1)])
@pytest.mark.parametrize("way", ["short", "two slices", "one slice"])
def test_ways_of_processing_narrow_units(gpu, way, hq, hkv, tokens):
    """Units of at most 32 rows that a wavefront has to itself are processed in one of three ways, by the average slices (32 keys) of a unit, the number of
    units and their tiles (128 keys) per wavefront: up to four slices (eight where units outnumber the wavefronts, two
    where they have more than 16 rows) short, else two slices in flight up to ten tiles a wavefront, else one.  Chains and trees that end inside a slice and right
    at one, with a few long ones that move the averages; through the shared list and through the workers' own lists.  Few enough
    workers that no team shares a unit."""
    tree = W.random_tree(np.random.default_rng(tokens), tokens)
    most = 70 if way == "short" and tokens * (hq // hkv) > 16 else 200
    specs = [W.SeqSpec(tokens, max(0, keys - tokens), V) for keys in (tokens, 31, 32, 33, 64, 95, 96, 97, 129, 200) if keys <= most]
    specs += [W.SeqSpec(tokens, keys - tokens, V, W.MASK_TREE, tree) for keys in (40, 64, 97, 160) if keys <= most]
    if way != "short":
        specs += [W.SeqSpec(tokens, keys - tokens, V) for keys in (1500, 1600, 1679, 1697)]
    units = len(specs) * hkv * -(-tokens // (32 // (hq // hkv)))
    workers = 1 if way == "one slice" else (units - 1) // 2
    b = W.make_custom(specs, hq, hkv, 17 * hq + tokens)

    def plan_check(units, _offs, _merges):
        n = len(units)
        assert int((units["q_count"] * units["head_count"]).max()) <= 32
        ends = [sum(b.seqs[u["seq"]][:2]) if b.seqs[u["seq"]][3] else b.seqs[u["seq"]][1] + u["q_begin"] + u["q_count"] for u in units]
        slices = sum(-(-(min(128 * u["kv_block_end"], e) - 128 * u["kv_block_begin"]) // 32) for u, e in zip(units, ends))
        tiles = int((units["kv_block_end"] - units["kv_block_begin"]).sum())
        many_rows = int((units["q_count"] * units["head_count"]).sum()) > 16 * n
        if slices <= (2 if many_rows else 8 if n > 4 * workers else 4) * n:
            assert way == "short"
        else:
            assert way == ("two slices" if tiles <= 40 * workers else "one slice")
    layout = dict(narrow_team=0, narrow_short=int(way == "short"), **({} if way == "short" else dict(narrow_depth=1 + (way == "two slices"))))
    for policy in (1, 2):
        run_and_check(gpu, b, f"{way}, policy {policy}", plan_check, layout, split_kv_blocks=0, num_workers=workers, assign_policy=policy)


@pytest.mark.parametrize("scale", [None, 1.0])
@pytest.mark.parametrize("hq,hkv", [(4, 1), (6, 2), (1, 1)])
def test_units_of_more_than_32_rows_on_one_and_on_two_row_tiles(gpu, hq, hkv, scale):
    """A wavefront holds one row tile where no unit of a launch has more than 128 rows, and units of more are handed out
    as two halves where there are idle workers for the second ones; else it holds two.  Rows at the edges of tiles,
    wavefronts and halves; a last piece of which the first half sees nothing; a tree; scores far above a row's first
    reference (second pass) and, with scale 1, a factor that is not folded into Q; padded cache rows.  A row is computed
    the same way either way: 256 workers (halves) and one worker (none idle) agree bit for bit."""
    import torch
    from paper_2412_18106_amd import binding as X
    g = hq // hkv
    rows = [33, 64, 65, 97, 128, 129, 192, 193, 255, 256]
    tokens = sorted({max(33 // g + 1, min(two_halves(g), r // g)) for r in rows})
    tree = W.random_tree(np.random.default_rng(3), 40)
    specs = [W.SeqSpec(t, 70 + 31 * i, V) for i, t in enumerate(tokens)] + [W.SeqSpec(40, 75, V, W.MASK_TREE, tree)]
    specs += [W.SeqSpec(64, c, V) for c in (0, 70, 134)]              # 64 tokens: the first 32 see no key of the last tile
    b = W.make_custom(specs, hq, hkv, 50 + hq, **({} if scale is None else dict(scale=scale)))
    k = W.bf16_bits_to_f32(b.k_cache)
    for i, s in enumerate(specs[:4]):                                   # 300 log2 units above what its row has seen so far
        pos, t0 = s.context_len - 3, sum(x.query_len for x in specs[:i])
        q = W.bf16_bits_to_f32(b.q[t0 + s.query_len - 1, 0])
        k[b.block_table[i, pos // 128], 0, pos % 128] = q * (300 / (b.scale * np.log2(np.e) * np.dot(q, q)))
    if scale is not None:         # (folded into Q, the factor costs a score of 300 log2 units more than the tolerance)
        b.k_cache[:] = W.f32_to_bf16_bits(k)
    ref = A.attention_oracle(b.seqs, b.q, b.k_cache, b.v_cache, b.block_table, b.tree_masks, num_q_heads=hq,
                             num_kv_heads=hkv, block_size=b.block_size, scale=b.scale)
    for split in (0, 1):
        outs = []
        for workers in (256, 1):
            db = gpu.DeviceBatch(b, num_workers=workers, split_kv_blocks=split, verify_tile_tokens=256 // g)
            try:
                assert_layout(db, **dict(WAYS)[workers])
                outs.append(db.run_numpy())
                views = []
                for src in (db.k_cache, db.v_cache):
                    views.append(torch.full((*src.shape[:3], 256), 3.0e4, dtype=torch.bfloat16, device="cuda")[..., :128])
                    views[-1].copy_(src)
                X.xy_attn_run(db.plan, db.q, *views, db.block_table, db.tree_masks, db.out, db.workspace, b.scale)
                outs.append(db.out.float().cpu().numpy())
            finally:
                db.close()
        err = np.abs(outs[0].astype(np.float64) - ref)
        assert err.max() <= MAX_ABS and err.mean() <= MEAN_ABS, (split, err.max(), err.mean())
        assert all(np.array_equal(o, outs[0]) for o in outs[1:]), split


@pytest.mark.parametrize("hq,hkv,tokens", [(1, 1, 1), (4, 1, 1), (5, 1, 6), (8, 1, 4), (4, 2, 8), (31, 1, 1)])
@pytest.mark.parametrize("team,wide", [(4, False), (4, True), (2, False), (2, True)])
def test_teams_of_wavefronts_on_narrow_units(gpu, team, wide, hq, hkv, tokens):
    """Several wavefronts share a narrow unit where there are fewer of them than workers without wide units (four each) or
    than twice as many (two), every wavefront with every fourth or second slice: units of fewer slices than members (the
    others come with nothing), ends inside a slice and right at one, trees, one to 32 rows, whole and cut, beside a wide
    unit and without, NaN and infinities in the slots nobody owns, three launches alike."""
    tree = W.random_tree(np.random.default_rng(tokens), tokens)
    specs = [W.SeqSpec(tokens, max(0, keys - tokens), V) for keys in (tokens, 31, 32, 33, 64, 95, 97, 129, 200, 700, 1055, 1100)]
    specs += [W.SeqSpec(tokens, keys - tokens, V, W.MASK_TREE, tree) for keys in (40, 97, 160, 1500)]
    if wide:
        specs.insert(5, W.SeqSpec(128 // (hq // hkv), 77, P))
    b = W.make_custom(specs, hq, hkv, 23 * hq + tokens)
    g, seqs = hq // hkv, len(specs) - wide
    for split in (0, 8):
        units = sum(-(-tokens // max(1, 32 // g)) * hkv * (-(-(-(-(s.context_len + s.query_len) // 128)) // split) if split else 1)
                    for s in specs if s.query_len == tokens and s.kind != P)
        workers = (units if team == 4 else (units + 1) // 2) + wide * hkv
        cfg = dict(split_kv_blocks=split, num_workers=workers)

        def plan_check(u, _offs, _merges):
            narrow = u[u["q_count"] * u["head_count"] <= 32]
            slices = 0
            for x in narrow:
                q, c, _kind, mask, _off = b.seqs[x["seq"]]
                end = c + q if mask else c + x["q_begin"] + x["q_count"]
                slices += -(-(min(128 * x["kv_block_end"], end) - 128 * x["kv_block_begin"]) // 32)
            free = workers - (len(u) - len(narrow))
            assert (free if team == 2 else 0) < len(narrow) <= (free if team == 4 else 2 * free)
            assert slices >= (3 if team == 4 else 8) * len(narrow)
        db = gpu.DeviceBatch(b, **cfg)
        try:
            assert_layout(db, narrow_team=team, row_tiles=1, halved=0)
            first = db.run_numpy()
            assert all(np.array_equal(db.run_numpy(), first) for _ in range(2))
        finally:
            db.close()
        saved = b.k_cache.copy(), b.v_cache.copy()
        _poison(b)
        db = gpu.DeviceBatch(b, **cfg)
        try:
            assert np.array_equal(db.run_numpy(), first)
        finally:
            db.close()
        b.k_cache[:], b.v_cache[:] = saved
        run_and_check(gpu, b, f"team of {team}, split {split}", plan_check, **cfg)


@pytest.mark.parametrize("workers, row_tiles", [(8, 2), (256, 1)])
@pytest.mark.parametrize("group", [1, 2, 4, 8, 16, 3, 12, 32])
def test_rows_of_a_wide_unit_leave_by_steps_of_sixteen(gpu, group, workers, row_tiles):
    """Results of whole wavefronts whose heads divide sixteen are stored by steps of sixteen rows, all others row by row: both
    for each group size, on two row tiles a wavefront and on one (as halves: an even number of tokens, or those of 3 and 12 heads are
    not divided), in units that end at, one token before and one token behind a wavefront's rows, with a padded output."""
    import torch
    from paper_2412_18106_amd import binding as X
    tile = 256 // group if row_tiles == 2 else 256 // group // 2 * 2
    lens = [tile, tile - 1, max(33 // group + 1, tile // 2), max(33 // group + 1, tile // 2 - 1), tile // 2 + 1, max(33 // group + 1, tile // 4 + 1)]
    b = W.make_custom([W.SeqSpec(n, 40 + n, P) for n in lens], 2 * group, 2, 7000 + group)
    db = gpu.DeviceBatch(b, num_workers=workers, split_kv_blocks=0)
    try:
        assert_layout(db, row_tiles=row_tiles)
        out = torch.full((b.total_q, 2 * group + 1, 136), float("nan"), dtype=torch.bfloat16, device="cuda")
        X.xy_attn_run(db.plan, db.q, db.k_cache, db.v_cache, db.block_table, db.tree_masks, out[:, :2 * group, :128], db.workspace, b.scale)
        torch.cuda.synchronize()
        assert torch.isnan(out[:, 2 * group]).all() and torch.isnan(out[..., 128:]).all()       # nothing beside the rows
        got = out[:, :2 * group, :128].float().cpu().numpy()
    finally:
        db.close()
    ref = A.attention_oracle(b.seqs, b.q, b.k_cache, b.v_cache, b.block_table, b.tree_masks,
                             num_q_heads=b.num_q_heads, num_kv_heads=b.num_kv_heads, block_size=b.block_size, scale=b.scale)
    err = np.abs(got.astype(np.float64) - ref)
    assert not np.isnan(got).any() and err.max() <= MAX_ABS and err.mean() <= MEAN_ABS
