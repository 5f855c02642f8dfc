"""The records xy_attn_copy_block_rows makes of its list of copies (no GPU: the library call is replaced)."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2412_18106_amd import binding as X


@pytest.mark.parametrize("copies", [[(1, 2, 3)], [(7, 8, 9), (np.int32(4), np.int64(5), 6)], [(1, 2)], [(1, 2), (3, 4, 5)],
                                    [(2**31, 0, 1)], [[-1, 0, 0]]])
def test_records_are_those_of_the_structure(monkeypatch, copies):
    seen = []

    def call(arr, n, *rest):
        seen.append(bytes(arr)[:12 * n])
        return 0
    monkeypatch.setattr(X, "_lib", type("L", (), {"xy_attn_copy_block_rows": staticmethod(call)}))
    monkeypatch.setattr(X, "_stream", lambda s: 0)
    k = torch.zeros(2, 1, 16, 128, dtype=torch.bfloat16)
    X.xy_attn_copy_block_rows(copies, 1, k, k)
    want = (X.xy_kv_copy * len(copies))(*[X.xy_kv_copy(*map(int, c)) for c in copies])
    assert seen == [bytes(want)]


def test_records_that_can_be_read_only_once(monkeypatch):
    seen = []
    monkeypatch.setattr(X, "_lib", type("L", (), {"xy_attn_copy_block_rows": staticmethod(
        lambda arr, n, *rest: seen.append(bytes(arr)[:12 * n]) or 0)}))
    monkeypatch.setattr(X, "_stream", lambda s: 0)
    k = torch.zeros(2, 1, 16, 128, dtype=torch.bfloat16)
    for copies in ([(1, 2, 3), (4, 5)], [(1, 2)], [(2**31, 0, 1)], [(1, 2, 3)]):
        X.xy_attn_copy_block_rows([iter(c) for c in copies], 1, k, k)
        assert seen.pop() == bytes((X.xy_kv_copy * len(copies))(*[X.xy_kv_copy(*c) for c in copies]))


def test_a_copy_of_four_fields_is_refused():
    k = torch.zeros(2, 1, 16, 128, dtype=torch.bfloat16)
    for copies in ([(1, 2, 3, 4)], [(1, 2), (3, 4, 5, 6)]):
        with pytest.raises((TypeError, ValueError)):
            X.xy_attn_copy_block_rows(copies, 1, k, k)
