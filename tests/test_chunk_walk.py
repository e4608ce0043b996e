"""The order in which the middle backward kernel of ranks up to 32 takes the chunks of the G3 gradient: groups of ids with
one i3 of equal and of very different sizes, empty ones, one group in all, and fewer chunks than XCDs.  A chunk that is
left out or taken by nobody shows in the G3 step.  Oracle and tolerances are those of test_gpu_parity."""
import numpy as np
import pytest

from oracle.tt_oracle import Shape
from tests.test_gpu_parity import check_against_oracle

pytestmark = pytest.mark.gpu

N12 = 60 * 50  # prefixes, the most ids of a group


@pytest.mark.parametrize("sizes", [[300] * 40, [3000] + [40] * 39, [0] * 20 + [2900, 1, 0, 9, 1200, 130] + [64, 0] * 7,
                                   [0] * 39 + [3000], [3000], [1] * 40, [9, 0, 3, 8], [513] + [65, 64, 63] * 13,
                                   list(range(0, 2000, 50))])
@pytest.mark.parametrize("d,r", [((4, 4, 8), 32), ((8, 4, 4), 16), ((4, 4, 4), 8)])
def test_groups_of_unequal_sizes(sizes, d, r):
    n = (60, 50, len(sizes))
    s = Shape(n, d, (r, r))
    rng = np.random.default_rng(len(sizes) + r)
    ids = np.concatenate([rng.permutation(N12)[:k] * n[2] + i3 for i3, k in enumerate(sizes)])
    ids = rng.permutation(ids).astype(np.int64)
    cores = tuple((rng.standard_normal(c) / np.sqrt(r)).astype(np.float32) for c in s.core_shapes())
    grad = (rng.standard_normal((ids.size, s.D)) / np.sqrt(ids.size)).astype(np.float32)
    check_against_oracle(n, d, (r, r), cores, ids, grad, 0.01, flags=8)
