"""Rows of prepared batches above and at the size where their tiles change: bit-identical to those of a forward
that builds its own index structures."""
import numpy as np
import pytest
import torch

from paper_2206_10581_amd import TTEmbedding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r,d3", [(8, 4), (8, 8), (16, 4), (16, 8), (32, 4), (32, 8), (64, 8)])
def test_rows_of_prepared_batches(r, d3):
    n, d, most = (40, 30, 50), (4, 4, d3), 262_177
    rng = np.random.default_rng(r + d3)
    shapes = ((n[0], 4, r), (n[1], r, 4, r), (n[2], r, d3))
    cores = [(rng.standard_normal(s) / np.sqrt(r)).astype(np.float32) for s in shapes]
    emb = TTEmbedding(n, d, (r, r), most, cores)
    for B in (131_072, 131_073, 262_144, 262_145, most):
        ids = rng.integers(0, n[0] * n[1] * n[2], B)
        ids[: B // 4] = 59_999
        ids[B // 2: B // 2 + 3] = [-1, 60_000, 1 << 40]
        t = torch.from_numpy(rng.permutation(ids)).cuda()
        want = emb.forward(t).clone()
        emb.backward_update(torch.zeros_like(want), 0.0)
        emb.prepare(t)
        got = emb.forward(t)
        torch.cuda.synchronize()
        assert torch.equal(got.view(torch.int32), want.view(torch.int32))
        emb.backward_update(torch.zeros_like(want), 0.0)
    emb.close()


@pytest.mark.parametrize("r,d1", [(8, 4), (8, 8), (16, 4), (16, 12), (32, 4), (32, 8)])
def test_rows_of_64_floats_on_both_sides_of_their_line(r, d1):
    """Up to 131,072 rows of the kernels' table (d1/4 for each id) tiles are short, above they are long: rows against
    lookups, which form the same sums without products in memory."""
    n, d = (40, 30, 50), (d1, 4, 4)
    rng = np.random.default_rng(r + d1)
    shapes = ((n[0], d1, r), (n[1], r, 4, r), (n[2], r, 4))
    cores = [(rng.standard_normal(s) / np.sqrt(r)).astype(np.float32) for s in shapes]
    line = 131_072 // (d1 // 4)
    emb = TTEmbedding(n, d, (r, r), line + 33, cores)
    for B in (line, line + 1, line + 33):
        ids = rng.integers(0, n[0] * n[1] * n[2], B)
        ids[: B // 4] = 59_999
        ids[B // 2: B // 2 + 3] = [-1, 60_000, 1 << 40]
        t = torch.from_numpy(rng.permutation(ids)).cuda()
        want = emb.forward_eval(t).clone()
        got = emb.forward(t)
        emb.backward_update(torch.zeros_like(got), 0.0)
        torch.cuda.synchronize()
        assert torch.equal(got.view(torch.int32), want.view(torch.int32))
    emb.close()
