"""The middle of the backward pass at ranks up to 32, where prefixes with many ids are taken by a whole block:
chunks with no, one, some and only such prefixes, with lengths at the edges of its rounds, in blocks of eight
wavefronts and (few ids per prefix of the table) of four.  Oracle and tolerances are those of test_gpu_parity."""
import numpy as np
import pytest

from oracle.tt_oracle import Shape
from tests.test_gpu_parity import check_against_oracle

pytestmark = pytest.mark.gpu

# ids per prefix, in the chunks of 16 prefixes of one i2 each
CHUNKS = ([300, 129, 128, 127, 65, 64, 63, 33, 32, 17, 16, 15, 9, 8, 1, 1], [40] * 16, [300], [17] + [1] * 15,
          [16] * 16, [3, 250, 2, 1])


@pytest.mark.parametrize("r", [8, 16, 32])
@pytest.mark.parametrize("d", [(4, 4, 4), (4, 4, 8), (8, 4, 4)])
@pytest.mark.parametrize("n", [(16, 6, 300), (200, 60, 300)])
def test_long_and_short_prefixes(n, d, r):
    s = Shape(n, d, (r, r))
    rng = np.random.default_rng(r)
    ids = []
    for i2, counts in enumerate(CHUNKS):
        for i1, k in enumerate(counts):
            i3 = rng.permutation(n[2])[:k]
            ids.append((i1 * n[1] + i2) * n[2] + i3)
    ids = np.concatenate(ids + ids[:1]).astype(np.int64)
    cores = tuple((rng.standard_normal(c) / np.sqrt(r)).astype(np.float32) for c in s.core_shapes())
    grad = (rng.standard_normal((len(ids), s.D)) / np.sqrt(len(ids))).astype(np.float32)
    order = rng.permutation(len(ids))
    check_against_oracle(n, d, (r, r), cores, ids[order], grad, 0.01, flags=8)
