"""Limits of the index-free kernels that the host decides, without a launch."""
import pytest

from paper_2206_10581_amd import binding
from paper_2206_10581_amd.binding import make_config


def _bytes(n, d, r, max_batch, flags=0):
    rc, nbytes = binding.tt_emb_workspace_bytes(make_config(n, d, r, max_batch, flags=flags))
    assert rc == 0
    return nbytes


# any-shape tables: flag 2 leaves out the index-free kernels and nothing else
@pytest.mark.parametrize("n,d,r", [((6, 1, 3), (8, 9, 1), (2, 100)), ((10, 10, 10), (2, 2, 2), (4, 4)),
                                   ((125, 140, 140), (4, 5, 5), (32, 32)), ((9, 2, 2), (4096, 1, 1), (64, 1)),
                                   ((40, 30, 20), (3, 5, 7), (9, 14))])
@pytest.mark.parametrize("max_batch", [1, 300, 9_000, 200_000])
def test_index_free_kernels_add_a_bounded_workspace(n, d, r, max_batch):
    """What those kernels keep per item is no more than 32 MiB (and a little alignment), and lies in the
    memory that batches with index structures use: a large handle needs not a byte more for them."""
    extra = _bytes(n, d, r, max_batch) - _bytes(n, d, r, max_batch, flags=2)
    assert 0 <= extra <= (32 << 20) + (1 << 16)
    if max_batch >= 200_000:
        assert extra == 0
