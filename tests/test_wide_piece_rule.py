"""Pieces of a family of more than 32 rows that is cut to fill idle workers, over the tiles it visits (worked out by
hand), and the C++ planner against the oracle planner on the same batches."""
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
