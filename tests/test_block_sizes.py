"""Sizes at which the index pipeline and the any-shape kernels change how they cut their work: the
largest batch of every sort block size and the one above it (with a hot id, out-of-range ids, and
tables of one, two and three sort passes, one of them with factors near the bucket limit); row
products with and without 16-byte operands; shapes at the limits of the any-shape kernels of both kinds
(what only those without matrix-core tiles take is in test_any_shape_kernels).  Oracle and tolerances are
those of test_gpu_parity."""
import numpy as np
import pytest

from oracle.tt_oracle import Shape
from tests.test_gpu_parity import check_against_oracle

pytestmark = pytest.mark.gpu


def _check(n, d, r, B, hot=4, seed=0, **kw):
    s = Shape(n, d, r)
    rng = np.random.default_rng(seed + B)
    cores = tuple((rng.standard_normal(c) / np.sqrt(r[0])).astype(np.float32) for c in s.core_shapes())
    ids = rng.integers(0, s.N, B).astype(np.int64)
    ids[rng.permutation(B)[: B // hot]] = s.N - 1
    ids[B // 2: B // 2 + 3] = [-1, s.N, 1 << 40]
    grad = (rng.standard_normal((B, s.D)) / np.sqrt(B)).astype(np.float32)
    check_against_oracle(n, d, r, cores, ids, grad, 0.01, **kw)


@pytest.mark.parametrize("B", [65_536, 65_537, 262_143, 262_144, 262_145, 524_288, 524_289])
def test_sort_block_sizes(B):
    _check((40, 30, 50), (2, 2, 2), (4, 4), B)


@pytest.mark.parametrize("B", [5, 255, 1023, 1024, 1025, 4096, 4097, 8192, 8193, 16_384, 16_385])
def test_small_batches_with_indices(B):
    """Flag 2 keeps small batches on the index structures: histograms beside the chunk records and in
    their memory."""
    _check((40, 30, 50), (2, 2, 2), (4, 4), B, flags=2)


@pytest.mark.parametrize("n", [(7, 5, 9), (300, 290, 310), (3, 1000, 900)])
def test_one_to_three_passes(n):
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


@pytest.mark.parametrize("n,d,r", [((9, 8, 150), (2, 2, 4), (4, 16)), ((9, 8, 150), (4, 4, 4), (4, 4)),
                                   ((9, 8, 150), (2, 4, 8), (4, 9)), ((70, 60, 5), (4, 4, 4), (4, 4)),
                                   ((70, 60, 5), (3, 3, 3), (6, 7))])
def test_small_prefix_gradients(n, d, r):
    """Products of up to 64 elements and one above, of prefixes with many ids and with few: the smallest
    tiles of the middle kernel."""
    _check(n, d, r, 9_001)


@pytest.mark.parametrize("d,r", [((4, 5, 5), (32, 32)), ((16, 2, 3), (5, 32)), ((17, 2, 3), (5, 33)),
                                 ((3, 5, 4), (70, 13)), ((2, 1, 9), (1, 1))])
def test_prefix_products_by_columns(d, r):
    """Chunks of up to 16 prefixes cut by columns: one run, several, a ragged last one; the largest d1 that
    the matrix-core tiles take and the next one, ranks they take and one they leave."""
    _check((70, 6, 5), d, r, 9_001)
