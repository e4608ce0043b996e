"""The prefix kernels of ranks 64 and 128 where dG2 partials stand for several chunks (the group
grows with the number of chunks): groups that begin and end inside a slice's chunks, chunks of
every fill, slices without a prefix.  Oracle and tolerances are those of test_gpu_parity."""
import numpy as np
import pytest

from oracle.tt_oracle import Shape
from tests.test_gpu_parity import check_against_oracle

pytestmark = pytest.mark.gpu


# groups of 4 (66,000 prefixes at rank 64) and 2 (16,000 at rank 128); n2 leaves about 14 and 8 chunks
# per slice, the last ones part empty
@pytest.mark.parametrize("n,d,r,B", [((260, 300, 2), (4, 4, 4), (64, 64), 150_000),
                                     ((130, 140, 2), (4, 4, 8), (128, 128), 40_000),
                                     ((3, 9, 40), (4, 4, 8), (64, 64), 9_000)])
def test_groups_of_chunks(n, d, r, B):
    s = Shape(n, d, r)
    rng = np.random.default_rng(r[0])
    cores = tuple((rng.standard_normal(c) / np.sqrt(r[0])).astype(np.float32) for c in s.core_shapes())
    ids = rng.integers(0, s.N, B).astype(np.int64)
    ids[(ids // n[2]) % n[1] == 1] = 0                       # a slice of G2 that no id touches
    grad = rng.standard_normal((B, s.D)).astype(np.float32)
    check_against_oracle(n, d, r, cores, ids, grad, 0.01)
