"""How the units of a plan are handed out to the GPU (host only): the rule restated from the plan, and the tables checked
against the plan row by row."""
import numpy as np
import pytest

from paper_2412_18106_amd import binding as X

CHIPLETS, WAVEFRONTS = 8, 4


def expected(seqs, units, offs, workers):
    """(row_tiles, halved, team, short, depth) from the units and lists a caller sees."""
    rows = units["q_count"] * units["head_count"]
    narrow = rows <= 32
    n, slices, tiles = int(narrow.sum()), 0, 0
    for u in units[narrow]:
        q, c, _kind, mask, _off = seqs[u["seq"]]
        end = c + q if mask else c + u["q_begin"] + u["q_count"]
        slices += -(-(min(128 * u["kv_block_end"], end) - 128 * u["kv_block_begin"]) // 32)
        tiles += u["kv_block_end"] - u["kv_block_begin"]
    wavefronts = WAVEFRONTS * workers
    short = n > 0 and slices <= n * (2 if rows[narrow].sum() > 16 * n else 8 if n > wavefronts else 4)
    depth = 2 if tiles <= 10 * wavefronts else 1
    lists = [list(range(offs[w], offs[w + 1])) for w in range(workers)]
    idle = sum(not x for x in lists)
    free = sum(not any(rows[i] > 32 for i in x) for x in lists)
    large = [i for x in lists for i in x if rows[i] > 128]
    if large and (len(large) > idle or n > WAVEFRONTS * (idle - len(large)) or
                  any(-(-int(units["q_count"][i]) // 2) * units["head_count"][i] > 128 for i in large)):
        return 2, 0, 0, short, depth
    free -= len(large)
    team = 0
    if 0 < n <= free:
        team = 4 if slices >= 3 * n else 0
    elif 0 < n <= 2 * free:
        team = 2 if slices >= 8 * n else 0
    return 1, len(large), team, short, 2 if team else depth


def check(cfg, seqs):
    """The layout and tables of a plan; returns the layout, the records, the offsets and the ranks."""
    workers = cfg.num_workers
    plan = X.xy_attn_plan_create(cfg, seqs)
    try:
        units, offs, _ = X.plan_arrays(plan, workers)
        layout, rec, lists, ranks = X.xy_probe_plan_layout(plan, workers)
        again = X.plan_arrays(plan, workers)
        assert units.tobytes() == again[0].tobytes() and offs.tolist() == again[1].tolist()     # what a caller sees stays
    finally:
        X.xy_attn_plan_destroy(plan)
    assert (layout.row_tiles, layout.halved, layout.narrow_team, bool(layout.narrow_short), layout.narrow_depth) == \
        expected(seqs, units, offs, workers)
    assert layout.records == len(rec) == len(units) + layout.halved
    # every row of every unit once, by (family piece, token), with the unit's own sequence fields
    starts = np.concatenate([[0], np.cumsum([s[0] for s in seqs])]).astype(int)
    group = cfg.num_q_heads // cfg.num_kv_heads
    key = ("seq", "head_begin", "head_count", "kv_block_begin", "kv_block_end", "ws_offset")
    want = sorted((*(int(u[k]) for k in key), t) for u in units for t in range(u["q_begin"], u["q_begin"] + u["q_count"]))
    got = sorted((*(int(r[k]) for k in key), t) for r in rec for t in range(r["q_begin"], r["q_begin"] + r["q_count"]))
    assert got == want
    by_row = {(*(int(u[k]) for k in key), t): u for u in units for t in range(u["q_begin"], u["q_begin"] + u["q_count"])}
    wide = rec["q_count"] * rec["head_count"] > 32
    for i, r in enumerate(rec):
        u = by_row[(*(int(r[k]) for k in key), int(r["q_begin"]))]
        q, c, kind, mask, off = seqs[r["seq"]]
        assert (r["query_len"], r["context_len"], r["mask_word_offset"], r["token_start"]) == (q, c, off, starts[r["seq"]])
        assert r["kv_head"] == r["head_begin"] // group and (r["flags"] & 255) == (kind | mask << 2)
        if layout.row_tiles == 1 and (wide[i] or layout.narrow_team):
            assert r["q_count"] * r["head_count"] <= 128
            assert r["flags"] >> 8 & 0xfff == u["q_count"] * u["head_count"]
            assert r["flags"] >> 20 == (r["q_begin"] - u["q_begin"]) * u["head_count"]
    assert lists[0] == 0 and (np.diff(lists) >= 0).all() and lists[workers] <= len(rec)
    assert not wide[lists[workers]:].any()                      # the shared list
    if layout.narrow_team:
        assert not (~wide[:lists[workers]]).any()
    own = np.diff(lists) > 0
    assert (ranks[own] == -1).all() and sorted(ranks[~own]) == list(range(int((~own).sum())))
    if layout.halved:
        # a second half is the only unit of a worker that has none in the plan, on the first half's chiplet if one is left there
        chiplet = (lambda w: w * CHIPLETS // workers) if workers % CHIPLETS == 0 else (lambda w: 0)
        owner = {(*(int(u[k]) for k in key), int(u["q_begin"])): w for w in range(workers) for u in units[offs[w]:offs[w + 1]]}
        second = [(w, r) for w in range(workers) for r in rec[lists[w]:lists[w + 1]] if int(r["flags"]) >> 20]
        assert len(second) == layout.halved
        for w, r in second:
            assert offs[w] == offs[w + 1] and lists[w + 1] - lists[w] == 1
            first = owner[(*(int(r[k]) for k in key), int(by_row[(*(int(r[k]) for k in key), int(r["q_begin"]))]["q_begin"]))]
            assert chiplet(w) == chiplet(first) or all(offs[x] < offs[x + 1] or own[x] for x in range(workers)
                                                              if chiplet(x) == chiplet(first))
    return layout, rec, lists, ranks


P, D, V = X.XY_PREFILL, X.XY_DECODE, X.XY_VERIFY


def decodes(n, ctx):
    return [(1, ctx + 31 * i, D, 0, 0) for i in range(n)]


# (heads, KV heads, config, sequences, (row tiles, halved, team))
CASES = {
    "a prompt of 256 rows alone": (4, 1, {}, [(64, 0, P, 0, 0)], (1, 1, 0)),
    "as many idle workers as large units": (4, 1, dict(num_workers=4), [(64, 0, P, 0, 0)] * 2, (1, 2, 0)),
    "one idle worker too few": (4, 1, dict(num_workers=3), [(64, 0, P, 0, 0)] * 2, (2, 0, 0)),
    "no idle worker, 128 rows": (4, 1, dict(num_workers=1), [(32, 0, P, 0, 0)] * 2, (1, 0, 0)),
    "three heads: 85 tokens, a first half of 129 rows": (6, 2, {}, [(200, 0, P, 0, 0)], (2, 0, 0)),
    "three heads in tiles of 84 tokens": (6, 2, dict(prefill_tile_tokens=84), [(84, 0, P, 0, 0)], (1, 2, 0)),
    "five heads: 51 tokens, a first half of 130 rows": (5, 1, {}, [(51, 0, P, 0, 0), *decodes(3, 500)], (2, 0, 0)),
    "a wavefront for every narrow unit": (4, 1, dict(num_workers=3), [(64, 0, P, 0, 0), *decodes(4, 40)], (1, 1, 0)),
    "one narrow unit more": (4, 1, dict(num_workers=3), [(64, 0, P, 0, 0), *decodes(5, 40)], (2, 0, 0)),
    "a worker for every narrow unit, three slices": (4, 1, dict(num_workers=6), [(1, 95, D, 0, 0)] * 6, (1, 0, 4)),
    "two slices": (4, 1, dict(num_workers=6), [(1, 63, D, 0, 0)] * 6, (1, 0, 0)),
    "half a worker for every narrow unit, eight slices": (4, 1, dict(num_workers=6, split_kv_blocks=0), [(1, 255, D, 0, 0)] * 12, (1, 0, 2)),
    "seven slices": (4, 1, dict(num_workers=6, split_kv_blocks=0), [(1, 223, D, 0, 0)] * 12, (1, 0, 0)),
    "one narrow unit too many": (4, 1, dict(num_workers=6, split_kv_blocks=0), [(1, 255, D, 0, 0)] * 13, (1, 0, 0)),
    "halves and a team": (4, 1, dict(num_workers=16, split_kv_blocks=0), [(64, 100, P, 0, 0), *decodes(9, 300)], (1, 1, 4)),
    "one worker has units of its own beside a team": (4, 1, dict(num_workers=256), [(32, 100, P, 0, 0), *decodes(31, 300)], (1, 0, 4)),
    "nothing": (4, 1, {}, [], (1, 0, 0)),
}


@pytest.mark.parametrize("name", CASES)
def test_layout_rule_at_its_edges(name):
    hq, hkv, cfg, seqs, want = CASES[name]
    layout, *_ = check(X.xy_attn_default_config(hq, hkv, 64, **cfg), seqs)
    assert (layout.row_tiles, layout.halved, layout.narrow_team) == want


def test_layout_of_random_plans():
    rng = np.random.default_rng(5)
    seen = set()
    for _ in range(150):
        hkv, group = int(rng.choice([1, 2, 8])), int(rng.choice([1, 2, 3, 4, 5, 8, 12]))
        seqs, words = [], 0
        for _i in range(int(rng.integers(0, 12))):
            kind, ctx = int(rng.integers(0, 3)), int(rng.integers(0, rng.choice([100, 3000])))
            q = 1 if kind == D else int(rng.integers(1, 200 if kind == P else 65))
            tree = int(kind == V and rng.random() < 0.5)
            seqs.append((q, ctx, kind, tree, words if tree else 0))
            words += tree * q * -(-q // 32)
        cfg = X.xy_attn_default_config(hkv * group, hkv, 32, num_workers=int(rng.choice([1, 7, 8, 64, 256, 304])),
                                       split_kv_blocks=int(rng.choice([-1, -1, 0, 1])), assign_policy=int(rng.choice([2, 2, 1, 0])))
        layout, *_ = check(cfg, seqs)
        seen.add((layout.row_tiles, layout.halved > 0, layout.narrow_team))
    assert {(2, False, 0), (1, False, 0), (1, True, 0), (1, False, 4), (1, True, 4)} <= seen


@pytest.mark.parametrize("workers,wide,narrow", [(256, 1, 31), (256, 9, 200), (64, 20, 30), (64, 60, 4), (16, 3, 12), (12, 3, 9)])
def test_teams_beside_wide_units_go_round_the_chiplets(workers, wide, narrow):
    """Team i is the worker of rank i: among the first n of them no chiplet has two more than another, unless that one has no
    worker without units left (one chiplet's L2 and path to memory would carry a short launch else)."""
    cfg = X.xy_attn_default_config(4, 1, 64, num_workers=workers, split_kv_blocks=0)
    layout, _, lists, ranks = check(cfg, [(32, 100 + 128 * i, P, 0, 0) for i in range(wide)] + decodes(narrow, 300))
    assert layout.narrow_team
    chiplets = CHIPLETS if workers % CHIPLETS == 0 else 1
    left = [sum(ranks[w] >= 0 for w in range(workers) if w * chiplets // workers == x) for x in range(chiplets)]
    taken = [0] * chiplets
    for w in np.argsort(ranks)[(ranks < 0).sum():]:
        x = w * chiplets // workers
        assert all(taken[x] <= taken[y] or taken[y] == left[y] for y in range(chiplets)), (w, taken)
        taken[x] += 1


def test_probe_refuses_what_it_cannot_fill():
    import ctypes
    plan = X.xy_attn_plan_create(X.xy_attn_default_config(4, 1, 64, num_workers=2), [(64, 0, P, 0, 0)])
    try:
        out, room = X.xy_probe_layout(), np.zeros(128, np.uint8)
        lists = np.zeros(5, np.int32)
        call = X._lib.xy_probe_plan_layout
        assert call(None, ctypes.byref(out), None, 0, None) == X.XY_ERR_ARG and call(plan, None, None, 0, None) == X.XY_ERR_ARG
        assert call(plan, ctypes.byref(out), room.ctypes.data, 2, None) == X.XY_ERR_ARG
        assert call(plan, ctypes.byref(out), room.ctypes.data, 1, lists.ctypes.data) == X.XY_ERR_CAPACITY
        assert out.records == 2 and not room.any() and not lists.any()
        assert call(plan, ctypes.byref(out), room.ctypes.data, 2, lists.ctypes.data) == X.XY_OK and lists.tolist() == [0, 1, 2, -1, -1]
    finally:
        X.xy_attn_plan_destroy(plan)
