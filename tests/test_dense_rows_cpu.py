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


@pytest.mark.parametrize("M", [384, 513, 1000, 1500, 4096])
def test_sixteen_rows_keep_float64(M):
    assert need(1 << 20, M, dense_rows=16) > need(1 << 20, M)
    assert need(1 << 20, M, dense_rows=32) == need(1 << 20, M)


def test_bytes_of_the_rows():
    rows = (1 << 20 >> 7) * 384   # one column block either way: U and K, 8 bytes for 4
    assert need(1 << 20, 384, dense_rows=16) - need(1 << 20, 384) == 2 * 4 * (rows + 1024)


@pytest.mark.parametrize("cols", [64, 128])
def test_narrow_columns_keep_float64(cols):
    for M in (384, 700):
        assert need(1 << 20, M, dense_cols=cols) == need(1 << 20, M, dense_cols=cols, dense_rows=16)


def test_long_chunks_keep_float64():
    assert need(1 << 26, 700, chunk_log2=25) == need(1 << 26, 700, chunk_log2=25, dense_rows=16)
    assert need(1 << 26, 700, chunk_log2=24) != need(1 << 26, 700, chunk_log2=24, dense_rows=16)
