"""Blocks of sorted slots of the segment and grouping kernels: batches that fill their last block exactly, by one
slot less and one more; the largest batch of every block size and the one above it, for the number of blocks and for
the rounds of loads in which a grouping block adds up their counts; a table whose counts do not fit the small blocks.  Oracle and tolerances are those of test_gpu_parity."""
import pytest

from tests.test_block_sizes import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,B", [((40, 30, 50), 12_287), ((40, 30, 50), 12_288), ((40, 30, 50), 12_289),
                                 ((20, 130, 600), 111_616), ((20, 130, 600), 111_617), ((20, 130, 600), 223_232),
                                 ((20, 130, 600), 223_233), ((9, 600, 593), 425_985), ((3, 1100, 1200), 30_001),
                                 ((20, 130, 600), 122_880), ((20, 130, 600), 122_881), ((40, 30, 50), 262_144),
                                 ((40, 30, 50), 262_145), ((20, 130, 600), 491_520), ((20, 130, 600), 491_521)])
def test_slot_blocks(n, B):
    _check(n, (2, 2, 2), (4, 4), B, flags=8)


@pytest.mark.parametrize("n,B", [((100, 100, 50), 65_536), ((100, 100, 50), 65_537), ((9, 600, 593), 32_768),
                                 ((9, 600, 593), 32_769), ((60, 60, 60), 262_144), ((60, 60, 60), 262_145)])
def test_sorts_with_and_without_a_column_scan(n, B):
    """As many rows of counts as the scatter adds up itself, and one more: digits of 1024 and 2048 values in blocks
    of 1024 ids, of 512 values in blocks of 2048."""
    _check(n, (2, 2, 2), (4, 4), B, flags=8)
