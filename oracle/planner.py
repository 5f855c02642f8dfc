"""Integer work-unit plan, written out rule by rule (TEST INFRASTRUCTURE ONLY).

Follows the paper's section 3.2.1 (Token-Table -> tiling blocks x heads =
tiling units) and section 3.3.1 (load = tileSize x kvLen, sort descending,
symmetric round-robin onto cores -> Task-Table).  Where the paper leaves a
choice open (tile sizes, tie-breaks, blocks vs tokens in the load, K/V
splitting across cores) the rules below are the written contract that the
C++ planner must reproduce bit for bit.

Rules
-----
1. Sequences in input order; ``token_start`` is the running sum of query_len.
   PREFILL uses token tiles of ``prefill_tile_tokens`` and head groups of
   ``prefill_heads_per_unit``; DECODE and VERIFY use token tiles of
   ``verify_tile_tokens`` and head groups of ``G = Hq / Hkv`` (one unit per KV
   head).  Families are enumerated sequence-major, then token tile, then head
   group.  K/V is visited in tiles of ``T = 128`` keys whatever the page size
   (a tile is ``128 / block_size`` consecutive block-table entries; the unit
   fields called ``kv_block_*`` count these tiles).  A causal family visits
   tiles ``[0, ceil((c + q_begin + q_count) / T))`` (tiles wholly past the
   tile's last visible key are never visited, section 4.2.2); a tree-masked
   family visits ``[0, ceil((c + q) / T))``.
   1a. ``verify_tile_tokens = -1`` (automatic): a DECODE / VERIFY sequence is
   tiled in ``max(1, 32 // G)`` tokens unless ``q`` exceeds that and
   ``ceil((c + q) / 128) >= 32``: then in ``min(q, max(1, 256 // G))`` tokens.
2. A non-PREFILL family with ``nb`` blocks and ``split_kv_blocks = S > 0`` and
   ``nb > S`` is cut into ``k = ceil(nb / S)`` units, unit ``p`` covering blocks
   ``[floor(p nb / k), floor((p + 1) nb / k))``.
   ``split_kv_blocks = -1`` (automatic) sizes S to the batch.  Narrow
   families are those of at most 32 rows; PREFILL ones (the last tokens of a
   prompt) count, and are cut like the others, if they visit more tiles than
   ``floor((2 t + 5 U) / (4 W))``, ``t`` the
   tiles of all families of the batch, ``U`` those of more than 32 rows; where
   the partial results of the whole batch would then exceed
   XY_STATIC_WORKSPACE_BYTES and would not without, no PREFILL one counts or
   is cut; ``F`` their
   number (token tiles times head groups), ``L = 4 W`` the wavefront slots.  If all of
   them have the same ``nb``: ``S = ceil(nb / k)`` for the ``k`` that minimises
   ``ceil(F k / L) * (ceil(nb / k) + 1)`` over ``k = 1 .. nb``, smallest ``k``
   on ties (the ``+ 1`` is what a piece costs beyond its tiles).  Otherwise
   ``S = min(max(s, 2), max(16, min(64, floor(2 s / 5))))`` with
   ``s = ceil(B / L)`` and ``B`` the sum of their ``nb``; where ``s <= 16`` and
   the batch has no other families, the smallest ``S`` from ``max(s, 2)`` to
   ``max(s + 1, floor(5 s / 4))`` that makes at most ``L`` pieces, if there is one.
   Wide families (more than 32 rows) of a DECODE / VERIFY sequence use ``S =
   16``, PREFILL ones are whole, unless a cut size ``T`` for all wide families,
   PREFILL too, is found.  ``U`` is the number of wide families:
   - ``2 U <= W`` and little else to do - ``2 N < M (W - U)`` with ``N`` the
     summed load ``max(rows, cost_row_floor) * nb`` of the families of at most
     32 rows and ``M`` the largest such load of a wide family: ``T`` is the
     smallest size from ``ceil(B / (W R))`` on (``R`` the largest ``max(rows,
     cost_row_floor)`` of a wide family, ``B = R sum nb + floor(N / 2)``) at
     which all together make at most ``ceil((W + ceil(W R sum nb / B)) / 2)``
     pieces, a family being cut at ``max(T, m)``,
     ``m = min(8, max(2, ceil(nb / 4)))`` or ``nb`` where ``nb <= 4``; then
     ``T`` is raised to the longest family that stays whole.
   - ``2 U > W`` and the longest family costs more than a quarter of the mean
     load of a worker (in half tiles: a piece ``2 nb + 5``, a narrow tile 2):
     candidates are, for ``r = ceil(U / W)`` and the next two, the smallest
     ``T >= max(2, ceil(sum nb / (r W)))`` with at most ``r W`` pieces; the one
     with the smallest estimated time (longest piece first to the least loaded
     worker, + 4 for the merge pass, at least the mean load) if that is at most
     ``floor(4 / 5)`` of the estimate without ``T``.
   Sizes that would need more workspace than XY_STATIC_WORKSPACE_BYTES, narrow
   partials included, are doubled until they do not (first kind) or left out
   (second kind).
3. ``rows = q_count * head_count``; ``cost = max(rows, cost_row_floor) * blocks``
   (``cost_row_floor = 1`` is the paper's tileSize x kvLen in block units).
4. Stable sort by cost descending, ties by (seq, head_begin, q_begin,
   split_index) ascending.
5. ``assign_policy`` 0 (the paper's symmetric round-robin): sorted position
   ``p`` has round ``p // W`` and lane ``p % W``; worker = lane on even rounds,
   ``W - 1 - lane`` on odd rounds.  ``assign_policy`` 1 (least loaded): walking
   the same sorted list, each unit goes to the worker whose summed cost so far
   is smallest, the lowest index among equals.  Units are emitted grouped by
   worker in assignment order, with ``worker_offsets[W + 1]``.
   5a. With policies 1 and 2, when 8 divides W, units of more than 32 rows
   are placed chiplet by chiplet: those of one (sequence, KV head) form a
   group; the groups, by summed cost descending (ties by sequence, KV head),
   go to the chiplet whose load so far is smallest (lowest index among
   equals); a unit then goes to the least-loaded worker among the W / 8 of its
   group's chiplet.  If the heaviest chiplet exceeds 1.03 times the mean
   (``max * 8 * 100 > total * 103``), no grouping is used; nor, with at most
   ``2 W`` units of more than 32 rows, if the largest load of a worker with it
   exceeds 1.03 times the largest without.
   ``assign_policy`` 2 (dynamic): units of more than 32 rows are assigned as
   with policy 1 among themselves, where ``cost_row_floor >= 128`` with
   ``2 * blocks + 5`` (a unit's time, whatever its rows) instead of the cost, in
   the sort as well; units of at most 32 rows are
   emitted behind all workers' lists, in sorted order, as one shared list that
   starts at ``worker_offsets[W]``.  When no unit has more than 32 rows and
   either all costs are equal or no unit visits more than 2 K/V tiles, policy
   2 gives the plan of policy 1.
6. A partial result is ``slab = rows * (D + 2)`` fp32 elements rounded up to a
   multiple of 4.  Split families, in enumeration order, get consecutive
   workspace regions of ``num_splits * slab``; a unit's ``ws_offset`` is its
   family base plus ``split_index * slab``; unsplit units carry -1.  One merge
   item per split family.
"""
from __future__ import annotations

import heapq

import numpy as np

PREFILL, DECODE, VERIFY = 0, 1, 2
MASK_CAUSAL, MASK_TREE = 0, 1
KV_TILE = 128
SPLIT_AUTO = -1          # split_kv_blocks value that sizes the K/V split to the batch
STATIC_WORKSPACE_FLOATS = 64 * 1024 * 1024 // 4      # what the library's own workspace holds
TILE_AUTO = -1           # verify_tile_tokens value that picks the token tile per sequence
NEVER = 1 << 62          # a number of tiles no family visits
NARROW_ROWS = 32         # units of at most this many rows are processed one per wavefront
CHIPLETS = 8             # L2 domains of the GPU: workers [x W / 8, (x + 1) W / 8) run on domain x when 8 divides W

UNIT_DTYPE = np.dtype([
    ("seq", "<i4"), ("head_begin", "<i4"), ("head_count", "<i4"),
    ("q_begin", "<i4"), ("q_count", "<i4"),
    ("kv_block_begin", "<i4"), ("kv_block_end", "<i4"),
    ("split_index", "<i4"), ("num_splits", "<i4"), ("kind_flags", "<i4"),
    ("cost", "<i8"), ("ws_offset", "<i8"),
])

MERGE_DTYPE = np.dtype([
    ("seq", "<i4"), ("head_begin", "<i4"), ("head_count", "<i4"),
    ("q_begin", "<i4"), ("q_count", "<i4"), ("num_splits", "<i4"),
    ("ws_offset", "<i8"),
])


def _verify_tile(cfg, ql, c, group):
    """Token tile of a DECODE / VERIFY sequence (rule 1a)."""
    t = cfg["verify_tile_tokens"]
    if t != TILE_AUTO:
        return t
    narrow = max(1, 32 // group)
    if ql <= narrow or _ceil_div(c + ql, KV_TILE) < 32:
        return narrow
    return min(ql, max(1, 256 // group))


def _ceil_div(a, b):
    return -(-a // b)


def _slab(rows, d):
    """fp32 elements of a partial result (rule 6)."""
    return _ceil_div(rows * (d + 2), 4) * 4


def _narrow_split(narrow, slots, alone):
    """Split size of the narrow families that may be cut: one (tiles, rows, is prefill) per family.  alone: whether
    the batch has no others."""
    lengths = {x[0] for x in narrow}
    if len(lengths) == 1:
        nb, families = narrow[0][0], len(narrow)
        best_k = min(range(1, nb + 1), key=lambda k: (_ceil_div(families * k, slots) * (_ceil_div(nb, k) + 1), k))
        return _ceil_div(nb, best_k)
    share = _ceil_div(sum(x[0] for x in narrow), slots)
    if alone and share <= 16:
        for size in range(max(share, 2), max(share + 1, 5 * share // 4) + 1):
            if sum(_ceil_div(x[0], size) for x in narrow) <= slots:
                return size
    return min(max(share, 2), max(16, min(64, 2 * share // 5)))


def _wide_pieces(nb, prefill, size, floor):
    """Pieces of a wide family of nb tiles; size 0: PREFILL whole, others cut at 16 tiles."""
    if size == 0:
        return 1 if prefill else _ceil_div(nb, 16)
    if floor:
        size = max(size, nb if nb <= 4 else min(8, max(2, _ceil_div(nb, 4))))
    return _ceil_div(nb, size)


def _wide_estimate(wide, size, w, narrow_tiles):
    """Half tiles until the last worker is done: pieces (2 per tile + 5) longest first to the worker with the least
    load, 4 for a merge pass, and never less than all the work over all workers."""
    costs = []
    cut = False
    for nb, _rows, prefill in wide:
        k = _wide_pieces(nb, prefill, size, False)
        cut = cut or k > 1
        costs += [2 * (((p + 1) * nb) // k - (p * nb) // k) + 5 for p in range(k)]
    load = [0] * w
    for x in sorted(costs, reverse=True):
        heapq.heapreplace(load, load[0] + x)
    return max(max(load) + (4 if cut else 0), _ceil_div(sum(costs) + 2 * narrow_tiles, w))


def _wide_cut(wide, narrow_tiles, narrow_load, narrow_ws, w, d, cost_floor):
    """Rule 2, wide part: (size, floor) of the cut.  wide: one (tiles, rows, is prefill) per family."""
    if not wide:
        return 0, False
    total, longest = sum(x[0] for x in wide), max(x[0] for x in wide)

    def pieces(size, floor):
        return sum(_wide_pieces(nb, pre, size, floor) for nb, _r, pre in wide)

    def fits(size, floor):
        ws = sum(_wide_pieces(nb, pre, size, floor) * _slab(rows, d)
                 for nb, rows, pre in wide if _wide_pieces(nb, pre, size, floor) > 1)
        return ws <= STATIC_WORKSPACE_FLOATS - narrow_ws

    if 2 * len(wide) <= w:
        if not narrow_load * 2 < max(max(r, cost_floor) * nb for nb, r, _p in wide) * (w - len(wide)):
            return 0, False
        tile_load = max(max(r, cost_floor) for _nb, r, _p in wide)
        both = total * tile_load + narrow_load // 2
        size = _ceil_div(both, w * tile_load)
        room = _ceil_div(w + _ceil_div(w * total * tile_load, both), 2)
        while size < longest and pieces(size, True) > room:
            size += 1
        size = max([size] + [nb for nb, _r, pre in wide if _wide_pieces(nb, pre, size, True) == 1])
        while size < longest and not fits(size, True):
            size *= 2
        return size, True
    if 4 * (2 * longest + 5) <= _ceil_div(2 * total + 5 * len(wide) + 2 * narrow_tiles, w):
        return 0, False
    best, chosen = _wide_estimate(wide, 0, w, narrow_tiles) * 4 // 5 + 1, 0
    first = _ceil_div(len(wide), w)
    for rounds in range(first, first + 3):
        size = max(2, _ceil_div(total, rounds * w))
        while size < longest and pieces(size, False) > rounds * w:
            size += 1
        if size >= longest or not fits(size, False):
            continue
        t = _wide_estimate(wide, size, w, narrow_tiles)
        if t < best:
            best, chosen = t, size
    return chosen, False


def plan_oracle(cfg, seqs):
    """cfg: dict with the plan parameters; seqs: list of
    (query_len, context_len, kind, mask_kind, mask_word_offset).

    Returns (units, worker_offsets, merges, workspace_floats) where units and
    merges are numpy structured arrays laid out like the C structs.
    """
    hq, hkv = cfg["num_q_heads"], cfg["num_kv_heads"]
    d = cfg["head_dim"]
    w = cfg["num_workers"]
    group = hq // hkv
    fam_units = []
    merges = []
    ws_floats = 0
    split_narrow = split_wide = cfg["split_kv_blocks"]
    wide_size, wide_floor = 0, False
    if cfg["split_kv_blocks"] == SPLIT_AUTO:
        wide = []               # (tiles, rows, is prefill) of every family of more than 32 rows
        narrow_load = narrow_tiles = 0
        narrow = []             # (tiles, rows) of every family of at most 32 rows
        for ql, c, kind, mk, _off in seqs:
            t = cfg["prefill_tile_tokens"] if kind == PREFILL else _verify_tile(cfg, ql, c, group)
            hc = cfg["prefill_heads_per_unit"] if kind == PREFILL else group
            for q_begin in range(0, ql, t):
                q_count = min(t, ql - q_begin)
                last = c + ql if mk == MASK_TREE else c + q_begin + q_count
                nb, rows = _ceil_div(last, KV_TILE), q_count * hc
                if rows > NARROW_ROWS:
                    wide += [(nb, rows, kind == PREFILL)] * (hq // hc)
                    continue
                narrow_load += max(rows, cfg["cost_row_floor"]) * nb * (hq // hc)
                narrow_tiles += nb * (hq // hc)
                narrow += [(nb, rows, kind == PREFILL)] * (hq // hc)
        split_wide = 16

        def choose(whole):
            """(fits XY_STATIC_WORKSPACE_BYTES, narrow size, wide size, wide floor), PREFILL whole up to that many tiles."""
            may_cut = [x for x in narrow if not x[2] or x[0] > whole]
            size = _narrow_split(may_cut, 4 * w, not wide and len(may_cut) == len(narrow))
            ws = sum(_ceil_div(nb, size) * _slab(rows, d) for nb, rows, _pre in may_cut if nb > size)
            wide_cut = _wide_cut(wide, narrow_tiles, narrow_load, ws, w, d, cfg["cost_row_floor"])
            for nb, rows, pre in wide:
                k = _wide_pieces(nb, pre, *wide_cut)
                ws += k * _slab(rows, d) if k > 1 else 0
            return ws <= STATIC_WORKSPACE_FLOATS, size, *wide_cut

        prefill_whole = (2 * sum(x[0] for x in wide) + 5 * len(wide) + 2 * narrow_tiles) // (4 * w)
        if not choose(prefill_whole)[0] and choose(NEVER)[0]:
            prefill_whole = NEVER
        _, split_narrow, wide_size, wide_floor = choose(prefill_whole)
    for i, (ql, c, kind, mk, _off) in enumerate(seqs):
        if kind == PREFILL:
            tile, hc = cfg["prefill_tile_tokens"], cfg["prefill_heads_per_unit"]
        else:
            tile, hc = _verify_tile(cfg, ql, c, group), group
        for q_begin in range(0, ql, tile):
            q_count = min(tile, ql - q_begin)
            last_key_excl = c + ql if mk == MASK_TREE else c + q_begin + q_count
            nb = _ceil_div(last_key_excl, KV_TILE)
            for head_begin in range(0, hq, hc):
                rows = q_count * hc
                s = split_narrow if rows <= NARROW_ROWS else split_wide
                if rows > NARROW_ROWS and wide_size:
                    k = _wide_pieces(nb, kind == PREFILL, wide_size, wide_floor)
                else:
                    may_split = kind != PREFILL or (cfg["split_kv_blocks"] == SPLIT_AUTO and rows <= NARROW_ROWS
                                                    and nb > prefill_whole)
                    k = _ceil_div(nb, s) if (may_split and s > 0 and nb > s) else 1
                slab = _slab(rows, d)
                base = -1
                if k > 1:
                    base = ws_floats
                    ws_floats += k * slab
                    merges.append((i, head_begin, hc, q_begin, q_count, k, base))
                for p in range(k):
                    lo, hi = (p * nb) // k, ((p + 1) * nb) // k
                    cost = max(rows, cfg["cost_row_floor"]) * (hi - lo)
                    off = -1 if k == 1 else base + p * slab
                    fam_units.append((i, head_begin, hc, q_begin, q_count, lo, hi, p, k,
                                      kind | (mk << 2), cost, off))
    by_time = cfg.get("assign_policy", 0) == 2 and cfg["cost_row_floor"] >= 128

    def load_of(u):
        return 2 * (u[6] - u[5]) + 5 if by_time and u[2] * u[4] > NARROW_ROWS else u[10]
    order = sorted(range(len(fam_units)),
                   key=lambda x: (-load_of(fam_units[x]), fam_units[x][0], fam_units[x][1],
                                  fam_units[x][3], fam_units[x][7]))
    per_worker = [[] for _ in range(w)]
    shared = []                 # policy 2: the narrow units, for all workers
    if cfg.get("assign_policy", 0) == 0:
        for pos, x in enumerate(order):
            rnd, lane = divmod(pos, w)
            per_worker[lane if rnd % 2 == 0 else w - 1 - lane].append(fam_units[x])
    else:
        load = np.zeros(w, dtype=np.int64)
        narrow_costs = {u[10] for u in fam_units if u[2] * u[4] <= NARROW_ROWS}
        any_wide = any(u[2] * u[4] > NARROW_ROWS for u in fam_units)
        longest_narrow = max((u[6] - u[5] for u in fam_units if u[2] * u[4] <= NARROW_ROWS), default=0)
        share = cfg.get("assign_policy", 0) == 2 and (any_wide or (len(narrow_costs) > 1 and longest_narrow > 2))
        # chiplet-aware placement of the wide units (rule 5a)
        per_chip = w // CHIPLETS if w % CHIPLETS == 0 else 0
        chip_of_group = None
        if per_chip:
            group_cost = {}
            for u in fam_units:
                if u[2] * u[4] > NARROW_ROWS:
                    key = u[0] * hkv + u[1] // group
                    group_cost[key] = group_cost.get(key, 0) + load_of(u)
            chip_load = [0] * CHIPLETS
            chip_of_group = {}
            for key in sorted(group_cost, key=lambda g: (-group_cost[g], g)):
                x = chip_load.index(min(chip_load))
                chip_of_group[key] = x
                chip_load[x] += group_cost[key]
            if max(chip_load) * CHIPLETS * 100 > sum(chip_load) * 103:
                chip_of_group = None
        def assign(chips):
            lists, load, shared_list, wide_units = [[] for _ in range(w)], np.zeros(w, dtype=np.int64), [], 0
            for x in order:
                u = fam_units[x]
                narrow = u[2] * u[4] <= NARROW_ROWS
                if share and narrow:
                    shared_list.append(u)
                    continue
                wide_units += not narrow
                if not narrow and chips is not None:
                    lo = chips[u[0] * hkv + u[1] // group] * per_chip
                    k = lo + int(np.argmin(load[lo:lo + per_chip]))
                else:
                    k = int(np.argmin(load))          # first index of the minimum
                lists[k].append(u)
                load[k] += load_of(u)
            return lists, shared_list, int(load.max()), wide_units

        per_worker, shared, largest, wide_units = assign(chip_of_group)
        if chip_of_group is not None and 0 < wide_units <= 2 * w:
            plain = assign(None)
            if largest * 100 > plain[2] * 103:
                per_worker, shared = plain[:2]
    flat = [u for lst in per_worker for u in lst] + shared
    offsets = np.zeros(w + 1, dtype=np.int32)
    offsets[1:] = np.cumsum([len(lst) for lst in per_worker])
    units = np.array(flat, dtype=UNIT_DTYPE) if flat else np.zeros(0, dtype=UNIT_DTYPE)
    marr = np.array(merges, dtype=MERGE_DTYPE) if merges else np.zeros(0, dtype=MERGE_DTYPE)
    return units, offsets, marr, ws_floats
