"""The any-shape kernels with products on the matrix cores where their tiles, fills and limits end: lines,
ranks and row widths on both sides of a tile of 16, ranks that are no multiple of four, rows and buffers that
do not allow 16-byte accesses, prefixes of one id, of more than 64 and of none in a chunk, the largest shapes
they take and the next ones (which take the kernels of tt_emb_compute).  Oracle and tolerances are those of
test_gpu_parity."""
import numpy as np
import pytest
import torch

from oracle import tt_oracle as ora
from oracle.tt_oracle import Shape
from paper_2206_10581_amd import TTEmbedding
from tests.test_gpu_parity import check_against_oracle, core_error, row_error, ROW_TOL

pytestmark = pytest.mark.gpu


def _inputs(n, d, r, B, seed):
    s = Shape(n, d, r)
    rng = np.random.default_rng(seed)
    cores = tuple((rng.standard_normal(c) / np.sqrt(r[0])).astype(np.float32) for c in s.core_shapes())
    ids = rng.integers(0, s.N, B).astype(np.int64)
    ids[rng.permutation(B)[: B // 5]] = s.N - 1
    ids[7:10] = [-1, s.N, 1 << 40]
    grad = (rng.standard_normal((B, s.D)) / np.sqrt(B)).astype(np.float32)
    return s, cores, ids, grad


@pytest.mark.parametrize("d,r", [
    ((4, 4, 16), (16, 16)), ((4, 4, 16), (17, 15)), ((1, 17, 15), (15, 17)),     # 16 and 17 lines
    ((8, 4, 8), (32, 33)), ((4, 8, 7), (33, 32)), ((3, 11, 3), (8, 8)),          # 32 and 33
    ((2, 5, 1), (64, 64)), ((2, 2, 3), (64, 63)), ((2, 2, 16), (65, 64)), ((2, 3, 17), (12, 65)),
    ((16, 2, 2), (5, 7)), ((17, 1, 4), (6, 6)), ((1, 1, 33), (3, 2)), ((2, 9, 32), (4, 20))])
def test_edges_of_tiles(d, r):
    for n, B in (((9, 8, 150), 9_001), ((70, 61, 5), 8_999)):   # prefixes of more than 64 ids; of two
        s, cores, ids, grad = _inputs(n, d, r, B, d[1] + r[0])
        check_against_oracle(n, d, r, cores, ids, grad, 0.01, flags=8)


@pytest.mark.parametrize("B", [1, 11, 12, 13, 47, 48, 49, 1_025])
def test_few_ids(B):
    s, cores, ids, grad = _inputs((11, 13, 17), (4, 5, 5), (12, 20), max(B, 16), B)
    check_against_oracle((11, 13, 17), (4, 5, 5), (12, 20), cores, ids[-B:], grad[-B:], 0.01, flags=8)


@pytest.mark.parametrize("shift", [1, 2, 4])
def test_buffers_at_any_float(shift):
    """Rows and gradients that begin 4 and 8 bytes off a 16-byte boundary, as this shape may have them."""
    n, d, r, B = (30, 31, 32), (4, 5, 5), (32, 32), 9_003
    s, cores, ids, grad = _inputs(n, d, r, B, 3)
    emb = TTEmbedding(n, d, r, B, cores)
    out = torch.zeros(B * s.D + 8, device="cuda")[shift:shift + B * s.D].view(B, s.D)
    g = torch.zeros(B * s.D + 8, device="cuda")[shift:shift + B * s.D].view(B, s.D)
    g.copy_(torch.from_numpy(grad))
    emb.forward(torch.from_numpy(ids).cuda(), out)
    emb.backward_update(g, 0.01)
    torch.cuda.synchronize()
    assert row_error(out.cpu().numpy(), ora.forward(s, *cores, ids)) <= ROW_TOL
    for new, ref in zip(emb.cores, ora.backward_update(s, *cores, ids, grad, 0.01)):
        assert core_error(new.cpu().numpy(), ref) <= 1e-4
    emb.close()


def test_an_infinity_stays_where_it_is():
    """Edges are masked in both operands: an infinite entry of a core reaches the rows of its ids only, an
    infinite gradient the slices of its id only."""
    n, d, r, B = (12, 11, 10), (4, 5, 5), (6, 7), 9_000
    s, cores, ids, grad = _inputs(n, d, r, B, 5)
    ids = np.where((ids < 0) | (ids >= s.N), 0, ids)
    cores[0][3, 1, 2] = np.inf
    i1, i2, i3 = ids // 110, ids // 10 % 11, ids % 10
    emb = TTEmbedding(n, d, r, B, cores)
    out = emb.forward(torch.from_numpy(ids).cuda())
    assert np.array_equal(np.isfinite(out.cpu().numpy()).all(1), i1 != 3)
    cores[0][3, 1, 2] = 1.0
    emb2 = TTEmbedding(n, d, r, B, cores)
    grad[100, 0] = np.inf
    emb2.forward(torch.from_numpy(ids).cuda())
    emb2.backward_update(torch.from_numpy(grad).cuda(), 0.01)
    for k, (c, i) in enumerate(zip(emb2.cores, (i1, i2, i3))):
        bad = ~torch.isfinite(c).flatten(1).all(1).cpu().numpy()
        assert bad[i[100]] and bad.sum() == 1, k
    emb.close()
    emb2.close()
