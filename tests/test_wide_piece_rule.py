"""Pieces of a family of more than 32 rows that is cut to fill idle workers, over the tiles it visits (worked out by
hand), and the C++ planner against the oracle planner on the same batches."""
import math
import random

import pytest

from oracle import planner as PL
from paper_2412_18106_amd import binding as X
from test_planner_parity import compare


@pytest.mark.parametrize("tiles,pieces", [(1, 1), (4, 1), (5, 3), (6, 3), (8, 4), (9, 3), (12, 4), (13, 4), (31, 4), (32, 4),
                                          (33, 5), (64, 8), (200, 25)])
def test_pieces_of_a_lone_wide_family(tiles, pieces):
    # one 64-token prefill tile of one head group, 256 workers: smallest piece nb (<= 4 tiles), else
    # min(8, max(2, ceil(nb / 4))): 5, 6, 8 -> 2 tiles, 9, 12 -> 3, 13 -> 4, from 31 on 8
    cfg = X.xy_attn_default_config(4, 1, 256)
    seqs = [(64, 128 * tiles - 64, X.XY_PREFILL, 0, 0)]
    units = PL.plan_oracle(cfg.as_dict(), seqs)[0]
    assert len(units) == pieces and set(units["num_splits"].tolist()) == {pieces}
    compare(cfg, seqs)


def test_pieces_follow_the_lengths_of_few_families():
    # four verify families of 32 heads in 8: 40, 60, 80, 120 tiles for 24 workers, sum 300 -> T from 13 on: 13 gives
    # 4 + 5 + 7 + 10 = 26, 14: 3 + 5 + 6 + 9 = 23 <= 24
    cfg = X.xy_attn_default_config(4, 1, 256, num_workers=24)
    seqs = [(31, 128 * t - 31, X.XY_VERIFY, 0, 0) for t in (40, 60, 80, 120)]
    units = PL.plan_oracle(cfg.as_dict(), seqs)[0]
    assert [int((units["seq"] == i).sum()) for i in range(4)] == [3, 5, 6, 9]
    compare(cfg, seqs)


@pytest.mark.parametrize("count,pieces", [(6, 1), (8, 1), (9, 3), (10, 3), (16, 1), (32, 1)])
def test_many_equal_families_are_cut_where_a_round_is_nearly_empty(count, pieces):
    # eight workers, families of 40 tiles: 85 half tiles a round.
    # 6: one round; two pieces each (45) take two rounds, 94, four (25) three, 79: not 68 or less.
    # 9, 10: two rounds, 170, of which the second is nearly empty; two pieces each: 3 x 45 + 4 = 139, three (33, 31, 31):
    # 27 or 30 pieces are four rounds of at most 33 + 4: 136 or less.  8, 16, 32: full rounds.
    cfg = X.xy_attn_default_config(4, 1, 256, num_workers=8)
    units = compare(cfg, [(64, 128 * 40 - 64, X.XY_PREFILL, 0, 0)] * count)
    assert set(units["num_splits"].tolist()) == {pieces}


def test_partial_results_stay_within_the_library_workspace():
    # 64 prefill families of 24 tiles beside 680 narrow ones of 6 tiles in 3 pieces each (34 MB of partials): four pieces
    # each would take the sum beyond 64 MiB, which xy_attn_run_static refuses
    cfg = X.xy_attn_default_config(32, 8, 256)
    seqs = [(64, 24 * 128 - 64, X.XY_PREFILL, 0, 0)] * 8 + [(8, 6 * 128 - 8, X.XY_VERIFY, 0, 0)] * 85
    units, _, _, ws = PL.plan_oracle(cfg.as_dict(), seqs)
    assert 4 * ws <= X.XY_STATIC_WORKSPACE_BYTES
    compare(cfg, seqs)


@pytest.mark.parametrize("heavy,counts", [(1030, [2, 1] * 8), (1031, [1] * 3 + [2] * 8 + [1] * 5)])
def test_chiplet_groups_of_a_short_list_are_dropped_for_a_level_list(heavy, counts):
    # Sixteen workers, two per chiplet; eight groups of three equal units (three heads of one KV head), seven groups of
    # 1000 tiles a unit and one of `heavy`.  By chiplet a worker has two units: at most 2 heavy.  Without, the three
    # heavy units have a worker each and no worker more than 2000.  2060 * 100 = 2000 * 103: kept; 2062: dropped.  The
    # chiplets are within 3 % of their mean both times (1031: 3093 * 800 = 2474400 <= (3093 + 21000) * 103 = 2481579).
    cfg = X.xy_attn_default_config(3, 1, 1031, num_workers=16, prefill_heads_per_unit=1, prefill_tile_tokens=128,
                                   split_kv_blocks=0, cost_row_floor=1, assign_policy=1)
    seqs = [(128, 128 * (heavy - 1), X.XY_PREFILL, 0, 0)] + [(128, 128 * 999, X.XY_PREFILL, 0, 0)] * 7
    compare(cfg, seqs)
    offs = PL.plan_oracle(cfg.as_dict(), seqs)[1]
    assert [int(offs[w + 1] - offs[w]) for w in range(16)] == counts


@pytest.mark.parametrize("floor", [128, 2**31 - 1])
@pytest.mark.parametrize("families", [1, 11, 21, 40])
def test_loads_beyond_64_bits_times_the_workers(floor, families):
    # workers x load of the wide families passes 2^63 from 11 families of 100000 tiles on (2^12 x 2^31 x 10^5 each)
    cfg = X.xy_attn_default_config(4, 1, 100000, num_workers=4096, cost_row_floor=floor, assign_policy=1)
    units = compare(cfg, [(64, 128 * 100000 - 64, X.XY_PREFILL, 0, 0)] * families + [(1, 12800 * 64 - 1, X.XY_DECODE, 0, 0)])
    assert (units["seq"] < families).sum() > families


@pytest.mark.parametrize("seqs", [
    [(8, 256000 - 8, X.XY_PREFILL, 0, 0)] * 44,                                             # 352 families in 29 pieces: 162 MiB
    [(8, 256000 - 8, X.XY_PREFILL, 0, 0)] * 40 + [(8, 256000 - 8, X.XY_VERIFY, 0, 0)] * 3,
    # five tails beside verify families of 160 rows on 9 x 16 tiles, 57 MiB of partials of their own
    [(8, 300000 - 8, X.XY_PREFILL, 0, 0)] * 5 + [(40, 144 * 128 - 40, X.XY_VERIFY, 0, 0)] * 10 + [(1, 40 * 128, X.XY_DECODE, 0, 0)] * 5])
def test_cut_prompt_tails_stay_within_the_library_workspace(seqs):
    # the last 8 tokens of a prompt are families of 32 rows; whole, they need no workspace, and no batch that
    # xy_attn_run_static takes that way is pushed beyond what it holds by cutting them
    cfg = X.xy_attn_default_config(32, 8, 4096)
    units = compare(cfg, seqs)
    assert 4 * PL.plan_oracle(cfg.as_dict(), seqs)[3] <= X.XY_STATIC_WORKSPACE_BYTES
    assert set(units["num_splits"][units["kind_flags"] == X.XY_PREFILL].tolist()) == {1}
    # a few of them, where the partials fit, are cut as before
    units = compare(cfg, seqs[:1] + [(1, 300, X.XY_DECODE, 0, 0)])
    assert units["num_splits"].max() > 1


@pytest.mark.parametrize("seed", range(40))
def test_both_planners_agree_on_drawn_batches_with_wide_families(seed):
    rng = random.Random(seed)
    cfg = X.xy_attn_default_config(*rng.choice([(4, 1), (8, 2), (32, 8), (64, 8), (8, 8)]), 4096, num_workers=rng.choice([6, 8, 16, 40, 256]))
    seqs = []
    for _ in range(rng.randrange(1, 10)):
        q, c = int(math.exp(rng.uniform(2, 7))), int(math.exp(rng.uniform(3, 9.5)))
        if rng.random() < 0.6:
            seqs.append((q, c if rng.random() < 0.7 else 0, X.XY_PREFILL, 0, 0))
        else:
            seqs.append((min(q, 31), c, X.XY_VERIFY, 0, 0))
    seqs += [(1, int(math.exp(rng.uniform(3, 9))), X.XY_DECODE, 0, 0) for _ in range(rng.choice([0, 0, 1, 5, 30]))]
    compare(cfg, seqs)
