"""Sizes at which the index pipeline and the any-shape kernels change how they cut their work: the
largest batch of every sort block size and the one above it (with a hot id, out-of-range ids, and
tables of one, two and three sort passes); row products with and without 16-byte operands; prefixes
of more ids than the id table of the prefix-gradient kernel holds, and rows too long for its split of
the contraction index.  Oracle and tolerances are those of test_gpu_parity."""
import numpy as np
import pytest

from oracle.tt_oracle import Shape
from tests.test_gpu_parity import check_against_oracle

pytestmark = pytest.mark.gpu


def _check(n, d, r, B, hot=4, seed=0):
    s = Shape(n, d, r)
    rng = np.random.default_rng(seed + B)
    cores = tuple((rng.standard_normal(c) / np.sqrt(r[0])).astype(np.float32) for c in s.core_shapes())
    ids = rng.integers(0, s.N, B).astype(np.int64)
    ids[rng.permutation(B)[: B // hot]] = s.N - 1
    ids[B // 2: B // 2 + 3] = [-1, s.N, 1 << 40]
    grad = (rng.standard_normal((B, s.D)) / np.sqrt(B)).astype(np.float32)
    check_against_oracle(n, d, r, cores, ids, grad, 0.01)


@pytest.mark.parametrize("B", [65_536, 65_537, 262_143, 262_144, 262_145, 524_288, 524_289])
def test_sort_block_sizes(B):
    _check((40, 30, 50), (2, 2, 2), (4, 4), B)


@pytest.mark.parametrize("n", [(7, 5, 9), (300, 290, 310)])
def test_one_and_three_passes(n):
    _check(n, (2, 2, 2), (4, 4), 70_001)


# The row tolerance is relative to a row's largest element, so rows have at least sixteen: the error of
# an element is bounded by a few ulp of the sum of its terms' magnitudes, which a row of one element
# that cancels (4e-5 of itself at d = (1, 1, 1)) does not bound.
@pytest.mark.parametrize("d,r", [((4, 5, 5), (32, 32)), ((3, 5, 7), (6, 12)), ((3, 5, 7), (12, 6)),
                                 ((4, 6, 9), (24, 20)), ((6, 7, 11), (36, 44)), ((2, 3, 65), (4, 8)),
                                 ((2, 3, 64), (4, 8)), ((1, 2, 8), (1, 4)), ((4, 5, 5), (128, 128))])
def test_any_shape_rows_and_prefix_gradients(d, r):
    _check((9, 8, 150), d, r, 9_001)          # every prefix has more than 64 ids
    _check((40, 45, 20), d, r, 9_001, seed=1)  # and here a handful
