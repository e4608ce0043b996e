"""Gradients per id at ranks 64 and 128, where several ids of a prefix are one step: prefixes with every number of ids
around the steps' sizes, in batches where a wavefront takes a prefix and a block the long ones, and where a block takes
every prefix.  Oracle and tolerances are those of test_gpu_parity."""
import numpy as np
import pytest

from oracle.tt_oracle import Shape
from tests.test_gpu_parity import check_against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [(4, 4, 8), (8, 4, 4)])
@pytest.mark.parametrize("rank,counts", [(64, [1, 2, 3, 4, 5, 7, 8, 9, 1, 1, 2, 6]), (64, [1, 2, 3, 15, 16, 17, 63, 64, 65, 80]),
                                         (128, [1, 2, 3, 4, 5, 9, 1, 1]), (128, [3, 16, 17, 33, 70])])
def test_ids_of_a_prefix(d, rank, counts):
    n = (4, 5, 80)
    s = Shape(n, d, (rank, rank))
    rng = np.random.default_rng(rank + len(counts))
    cores = tuple((rng.standard_normal(c) / np.sqrt(rank)).astype(np.float32) for c in s.core_shapes())
    prefixes = rng.permutation(n[0] * n[1])[: len(counts)]
    ids = np.concatenate([p * n[2] + rng.permutation(n[2])[:k] for p, k in zip(prefixes, counts)])
    ids = rng.permutation(np.concatenate([ids, ids[:3]])).astype(np.int64)  # three ids twice
    grad = (rng.standard_normal((ids.size, s.D)) / np.sqrt(ids.size)).astype(np.float32)
    check_against_oracle(n, d, (rank, rank), cores, ids, grad, 0.01, flags=8)


def _check(n, d, rank, counts):
    """A batch with so many ids of one prefix each, the prefixes in this order."""
    s = Shape(n, d, (rank, rank))
    rng = np.random.default_rng(rank + len(counts))
    cores = tuple((rng.standard_normal(c) / np.sqrt(rank)).astype(np.float32) for c in s.core_shapes())
    ids = rng.permutation(np.concatenate([p * n[2] + rng.permutation(n[2])[:k] for p, k in enumerate(counts)]))
    grad = (rng.standard_normal((ids.size, s.D)) / np.sqrt(ids.size)).astype(np.float32)
    check_against_oracle(n, d, (rank, rank), cores, ids.astype(np.int64), grad, 0.01, flags=8)


@pytest.mark.parametrize("d", [(4, 4, 8), (8, 4, 4)])
@pytest.mark.parametrize("rank", [64, 128])
def test_long_prefixes_beside_short_ones(rank, d):
    """Four prefixes are a block's turn: none, one, two and four of them with more than 128 ids, and one in a last turn of
    two; fewer than sixteen ids each on average, so that wavefronts take the others."""
    turns = [1, 128, 127, 2] + [1, 129, 1, 3] + [200, 1, 130, 1] + [255, 256, 129, 250]
    _check((20, 30, 256), d, rank, turns + [1] * 109 + [140])


@pytest.mark.parametrize("d", [(4, 4, 8), (8, 4, 4)])
@pytest.mark.parametrize("rank", [64, 128])
def test_blocks_take_more_than_one_prefix(rank, d):
    """256 prefixes (512 with two slabs) of sixteen ids, each a block's, and 136 (264) blocks: the LDS of a block holds the
    sums of one prefix and then of another."""
    _check((16, 16, 16), d, rank, [16] * 256)
