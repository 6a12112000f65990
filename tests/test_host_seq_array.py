"""SeqArray fills the C structures of four and more sequences column by column; every field has to be what a structure made
from the sequence's own values holds, for whatever numbers and page tables callers pass."""
import numpy as np
import pytest

from paper_2507_17769_amd import binding as B
from paper_2507_17769_amd import workloads as W


def _fields(q):
    return q.req_id, q.n_new, q.kv_len, [q.page_table[j] for j in range(q.n_pages)], q.n_pages


def _rows(first_id):
    frozen = np.arange(7, dtype=np.int32)
    frozen.flags.writeable = False
    pages = [np.arange(5, dtype=np.int32), np.arange(12, dtype=np.int64)[::2], [4, 3], frozen, np.zeros(0, np.int32), np.arange(9, dtype=np.int32)[::-1], (1, 2, 3)]
    return [(first_id + i, np.int64(1 + i), [3, 2 ** 31 - 1, 2 ** 32 + 5, -1, 0, 16, 17][i], p) for i, p in enumerate(pages)]


@pytest.mark.parametrize("first_id", [0, -(2 ** 63), 2 ** 63 - 3, 2 ** 64 + 9])
@pytest.mark.parametrize("n", [0, 1, 3, 4, 7])
def test_every_field_is_what_a_structure_of_its_own_holds(n, first_id):
    rows = _rows(first_id)[:n]
    sa = B.SeqArray(rows)
    assert sa.n == n and sa.n_tokens == sum(int(r[1]) for r in rows) and len(sa.array) == max(n, 1)
    for q, r in zip(sa.array, rows):
        t = np.ascontiguousarray(r[3], dtype=np.int32)
        assert _fields(q) == _fields(B.ps_seq(int(r[0]), int(r[1]), int(r[2]), t.ctypes.data_as(B._I32P), len(t)))


def test_objects_and_tables_that_lie_in_place():
    seqs = [W.SeqSpec(10 + i, 1, 20 + i, np.arange(2, dtype=np.int32)) for i in range(5)]
    sa = B.SeqArray(seqs)
    for q, s in zip(sa.array, seqs):
        assert _fields(q) == (s.req_id, 1, s.kv_len, [0, 1], 2)
        s.pages[1] = 77                       # the structure points at the caller's table
        assert q.page_table[1] == 77
    with pytest.raises((TypeError, ValueError)):
        B.SeqArray([(i, 1, None, [0]) for i in range(5)])
