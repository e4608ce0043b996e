"""The prefix kernels of ranks 64 and 128 where dG2 partials stand for several chunks (the group
grows with the number of chunks): groups that begin and end inside a slice's chunks, chunks of
every fill, slices without a prefix.  Oracle and tolerances are those of test_gpu_parity."""
import numpy as np
import pytest

from oracle import tt_oracle as ora
from oracle.tt_oracle import Shape
from tests.test_gpu_parity import check_against_oracle, run_gpu

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


def test_groups_of_chunks_add_in_two_levels():
    """Terms of one sign show how long the chains of a sum are: m roundings of rms 0.41 u each (u = 2^-24)
    on growing partial sums leave 0.41 u sqrt(m / 3).  Here a slice has 14 chunks of 64 terms in groups of
    four.  Chunk by chunk that is sqrt(64/3 / 14 + 4/3 / 3.5 + 14/3 / 4) * 0.41 u = 4e-8 with the update's
    own rounding; 256 terms in one chain would be 1.2e-7.  The bound lies between."""
    n, d, r, B = (260, 300, 2), (4, 4, 4), (64, 64), 150_000
    s = Shape(n, d, r)
    rng = np.random.default_rng(9)
    cores = tuple((np.abs(rng.standard_normal(c)) / 8).astype(np.float32) for c in s.core_shapes())
    ids = rng.integers(0, s.N, B).astype(np.int64)
    grad = (1e4 * np.abs(rng.standard_normal((B, s.D)))).astype(np.float32)
    _, new, _ = run_gpu(n, d, r, cores, ids, grad, 1.0)
    ref = ora.backward_update(s, *cores, ids, grad, 1.0)[1].astype(np.float64)
    step = np.linalg.norm(cores[1] - ref)
    assert np.linalg.norm(new[1] - ref) <= 7e-8 * step
