"""Gradients per id at ranks 64 and 128, where several ids of a prefix are one step: prefixes with every number of ids
around the steps' sizes, in batches where a wavefront takes a prefix (fewer than sixteen ids each on average) and
where a block does.  Oracle and tolerances are those of test_gpu_parity."""
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
