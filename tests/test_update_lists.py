"""Lists of partial gradients of the update kernel: as many entries as its rounds of eight and of four take at a time,
one fewer and one more.  Oracle and tolerances are those of test_gpu_parity."""
import numpy as np
import pytest

from oracle.tt_oracle import Shape
from tests.test_gpu_parity import check_against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 127, 128, 129, 511, 512, 513, 640, 1023, 1024, 1025, 1153, 1537, 1700])
def test_prefixes_of_an_i1(k):
    """Slices of eight floats of G1 leave 128 threads side by side on the list of the k prefixes with i1 = 1."""
    n, d, r = (3, 1700, 2), (2, 2, 2), (4, 4)
    s = Shape(n, d, r)
    rng = np.random.default_rng(k)
    cores = tuple((rng.standard_normal(c) / 2).astype(np.float32) for c in s.core_shapes())
    ids = rng.permutation((1700 + rng.permutation(1700)[:k]) * 2 + rng.integers(0, 2, k)).astype(np.int64)
    grad = (rng.standard_normal((k, s.D)) / np.sqrt(k)).astype(np.float32)
    check_against_oracle(n, d, r, cores, ids, grad, 0.01, flags=8)
