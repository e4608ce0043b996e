"""Sums of gradient rows over repeated ids: wavefronts of 64 sorted ids of which none, some, nearly all or all
occur more than once, with runs that cross from one wavefront into the next, at every row length the kernel
has a form for.  Oracle and tolerances are those of test_gpu_parity."""
import numpy as np
import pytest

from oracle.tt_oracle import Shape
from tests.test_gpu_parity import check_against_oracle

pytestmark = pytest.mark.gpu

REPEATED = (0, 2, 7, 8, 9, 15, 16, 17, 24, 25, 47, 48, 49, 50, 63, 64, 0, 64, 64, 3)
# around 32 of 64, where rows of other lengths than 128 change their walk, mixed with full and empty wavefronts
AROUND_32 = (31, 32, 33, 34, 64, 30, 32, 0, 33, 1, 32, 64, 33, 33, 31, 2, 48, 49, 40, 41)


def _sorted_ids(repeated=REPEATED):
    """Ascending ids, 64 of them per entry k of REPEATED: runs of two and three over the last k, then, for odd
    entries, the last run goes on into the next group."""
    ids, u = [], 0
    for k in repeated:
        group = []
        while len(group) < 64 - k:
            u += 1
            group.append(u)
        n = 2
        while len(group) < 64:
            u += 1
            group += [u] * min(n, 64 - len(group))
            n = 5 - n
        ids += group
        if k % 2:
            u -= 1  # the next group starts with this id
    return np.array(ids, np.int64)


@pytest.mark.parametrize("n,d,r", [((12, 11, 16), (4, 4, 4), (16, 16)), ((12, 11, 16), (4, 4, 8), (32, 32)),
                                   ((12, 11, 16), (3, 5, 4), (8, 8)), ((12, 11, 16), (4, 5, 5), (8, 8)),
                                   ((12, 11, 16), (4, 5, 8), (8, 8))])
def test_wavefronts_with_few_and_many_repeats(n, d, r):
    _check(n, d, r, _sorted_ids())


@pytest.mark.parametrize("d,r", [((4, 4, 4), (16, 16)), ((8, 4, 4), (16, 16)), ((4, 4, 8), (32, 32)), ((3, 5, 4), (8, 8)),
                                 ((4, 5, 5), (8, 8)), ((4, 5, 8), (8, 8)), ((4, 8, 8), (8, 8))])
def test_wavefronts_where_the_walk_changes(d, r):
    _check((12, 11, 16), d, r, _sorted_ids(AROUND_32))


def _check(n, d, r, ids):
    s = Shape(n, d, r)
    assert ids.max() < s.N and len(ids) == 64 * len(REPEATED)
    rng = np.random.default_rng(len(ids))
    cores = tuple((rng.standard_normal(c) / np.sqrt(r[0])).astype(np.float32) for c in s.core_shapes())
    grad = (rng.standard_normal((len(ids), s.D)) / np.sqrt(len(ids))).astype(np.float32)
    order = rng.permutation(len(ids))
    check_against_oracle(n, d, r, cores, ids[order], grad, 0.01, flags=2)
