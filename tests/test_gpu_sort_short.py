"""Sorts without a scan launch: one element, a chunk, the most chunks that go without one and one more, for digits of 8, 10
and 11 bits.  And the sums of rows that cross many spans, whose partial sums several waves share."""
import numpy as np
import pytest

from tests.test_gpu_push_edges import _step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,chunks", [(1 << 8, 64), (1 << 16, 64), ((1 << 16) + 1, 8), (1 << 20, 8), ((1 << 20) + 1, 3), (1 << 22, 3),
                                      ((1 << 22) + 1, 64)])
@pytest.mark.parametrize("offset", [None, -1, 0, 1, 1024])
def test_lists_around_the_most_chunks_without_a_scan(R, chunks, offset):
    n = 1 if offset is None else chunks * 1024 + offset
    rng = np.random.default_rng(n)
    _step((min(R - 1, 60000) ** rng.random(n)).astype(np.uint64) + 1, 4, R)


# 16 spans are a wave's share, 64 a block; spans have 8 occurrences here
@pytest.mark.parametrize("D", [100, 128, 256])
@pytest.mark.parametrize("spans", [16, 17, 63, 64, 65, 80, 129, 700])
def test_rows_over_many_spans_of_wide_rows(D, spans):
    rng = np.random.default_rng(spans)
    lengths = [8 * 61 + 3, 8 * spans, 5, 8 * spans + 9, 40]
    keys = np.repeat(np.arange(1, len(lengths) + 1), lengths)
    _step(rng.permutation(keys), D, 64)


# one below and at the sizes from 2 M on where the span length changes for narrow rows
@pytest.mark.parametrize("D,n", [(4, (2 << 20) - 1), (4, 2 << 20), (16, (4 << 20) - 1), (16, 4 << 20)])
def test_span_length_of_narrow_rows_in_long_lists(D, n):
    rng = np.random.default_rng(n)
    _step((200000 ** rng.random(n)).astype(np.uint64) + 1, D, 200002)


# the same in tables of many rows (or, of 8 columns at 3 Mi, of few), and of 32 columns at 10 Mi, whose gradients are walked in windows
@pytest.mark.parametrize("D,first,rows", [(4, 7 << 19, 1 << 22), (8, 5 << 19, 1 << 22), (8, 3 << 20, 1 << 18), (12, 11 << 19, 1 << 22),
                                          (32, 10 << 20, 1 << 20)])
@pytest.mark.parametrize("below", [1, 0])
def test_lines_of_the_span_length_in_long_lists(D, first, rows, below):
    from oracle import ctr_oracle as O
    from paper_2201_05500_amd.binding import CtrTable, ctr_debug_push_span
    from tests.parity_util import compare_tables, run_step, to_device
    from tests.test_gpu_push_edges import _batch
    n = first - below
    gt, ot = CtrTable(rows, D, init_seed=3), O.OracleTable(200002, D, init_seed=3)  # rows in use count, not the capacity
    assert ctr_debug_push_span(gt.cfg, first - 1) != ctr_debug_push_span(gt.cfg, first)
    keys = (200000 ** np.random.default_rng(n).random(n)).astype(np.uint64) + 1
    for step in range(2):
        b = _batch(keys, D, 1 + step)
        run_step(gt, ot, to_device(b), b)
    compare_tables(gt, ot)
