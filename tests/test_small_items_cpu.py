"""The length of the small-M engine's items for one sequence, read off the workspace it asks for (host arithmetic
only): enough items to keep the chip's lanes busy on a long sequence, never more than the workspace's bound."""
import pytest

import paper_2604_01342_amd as H


def items(n):
    """Items of a one-node log-likelihood: 48 bytes an item, and as much as one more item per 64 of them."""
    return H.workspace_bytes(n, 1, grad=False) / (48.0 * 65 / 64)


@pytest.mark.parametrize("n,least", [(4_000_000, 28_000), (10_000_000, 36_000), (30_000_000, 36_000),
                                     (100_000_000, 36_000), (300_000_000, 60_000), (3_000_000_000, 60_000)])
def test_long_sequences_have_many_items(n, least):
    assert least < items(n) < 68_000


@pytest.mark.parametrize("n", [1_000, 100_000, 1_000_000, 3_000_000])
def test_short_sequences_have_few(n):
    assert items(n) < 26_000
