"""Where the state between blocks of the dense dL/dalpha is kept in float64 from 384 nodes on, read off the workspace
(host arithmetic only; one event range, so that nothing else differs)."""
import pytest

import paper_2604_01342_amd as H


def need(n, M, chunk_log2=0, **tuning):
    try:
        H.set_tuning(dense_ranges=1, **tuning)
        return H.workspace_bytes(n, M, chunk_log2=chunk_log2)
    finally:
        H.set_tuning()


@pytest.mark.parametrize("M,padded,block", [(384, 384, 7), (512, 512, 7), (513, 576, 8), (1000, 1024, 8)])
def test_sixteen_rows_keep_float64(M, padded, block):
    rows = (1 << 20 >> block) * padded + 1024   # and slack past the last row
    assert need(1 << 20, M, dense_rows=16) - need(1 << 20, M) == 2 * 4 * rows   # U and K: 8 bytes for 4
    assert need(1 << 20, M, dense_rows=32) == need(1 << 20, M)


@pytest.mark.parametrize("cols", [64, 128])
def test_narrow_columns_keep_float64(cols):
    assert need(1 << 20, 700, dense_cols=cols) == need(1 << 20, 700, dense_cols=cols, dense_rows=16)


def test_long_chunks_keep_float64():
    assert need(1 << 26, 700, chunk_log2=25) == need(1 << 26, 700, chunk_log2=25, dense_rows=16)
    assert need(1 << 26, 700, chunk_log2=24) < need(1 << 26, 700, chunk_log2=24, dense_rows=16)
