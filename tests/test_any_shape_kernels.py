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


def _slots(n, d, r, B, ids, grad, cores):
    """Launches of a profiled step: without prefix_bwd the middle of the backward pass was one launch."""
    emb = TTEmbedding(n, d, r, B, cores, flags=8)
    emb.profile(True)
    emb.forward(torch.from_numpy(ids).cuda())
    emb.backward_update(torch.from_numpy(grad).cuda(), 0.0)
    slots = {k: v["launches"] for k, v in emb.profile_read().items()}
    emb.close()
    return slots


# r1 and r2 that fill a run of 4, 8, 12 or 16 indices of each lane group in part, in whole words and not; with
# many ids per prefix, with one fewer than that, and with few; fused: the middle is one launch (many, few)
@pytest.mark.parametrize("d,r,fused", [
    ((4, 5, 5), (20, 28), (1, 1)), ((4, 5, 5), (24, 32), (1, 1)), ((3, 5, 4), (36, 44), (1, 1)),
    ((4, 4, 4), (44, 36), (1, 1)), ((2, 2, 4), (52, 60), (1, 1)), ((2, 2, 3), (60, 52), (1, 1)),
    ((4, 5, 5), (30, 31), (1, 1)), ((4, 4, 3), (18, 17), (1, 1)), ((2, 3, 12), (24, 24), (0, 1)),
    ((2, 3, 12), (33, 32), (0, 0)), ((2, 2, 2), (33, 63), (0, 1)), ((4, 5, 5), (33, 35), (0, 0)),
    ((3, 7, 2), (48, 56), (0, 0))])
def test_ranks_between_runs(d, r, fused):
    for n, B, many in (((33, 34, 9), 8_976, True), ((33, 34, 9), 8_975, False), ((70, 61, 5), 8_999, False)):
        s, cores, ids, grad = _inputs(n, d, r, B, r[0] + r[1])
        check_against_oracle(n, d, r, cores, ids, grad, 0.01, flags=8)
        slots = _slots(n, d, r, B, ids, grad, cores)
        assert slots["u_bwd"] == slots["dg3"] == 1 and slots["prefix_bwd"] == 1 - fused[0 if many else 1]


# What is left to the kernels of tt_emb_compute: more than 32 lines, ranks above 64, d3 above 16, d1 above 16.
# Prefix gradients with and without the id table (products of up to 64 elements and one line more; lines and ids
# per prefix on both sides of its rule), staged rows with and without whole words, products cut by columns.
@pytest.mark.parametrize("d,r", [((17, 2, 3), (4, 1)), ((33, 1, 2), (3, 2)), ((11, 3, 2), (6, 2)), ((5, 1, 33), (6, 4)),
                                 ((4, 1, 33), (6, 4)), ((5, 1, 33), (3, 13)), ((1, 1, 40), (1, 1)), ((6, 7, 2), (12, 8)),
                                 ((5, 7, 3), (9, 6)), ((3, 3, 5), (70, 72)), ((3, 3, 5), (66, 67)),
                                 ((17, 2, 17), (20, 66)), ((4, 9, 5), (65, 68))])
def test_larger_shapes(d, r):
    for n, B in (((9, 8, 150), 9_001), ((70, 61, 5), 8_999)):
        s, cores, ids, grad = _inputs(n, d, r, B, d[0] + r[1])
        check_against_oracle(n, d, r, cores, ids, grad, 0.01, flags=8)
        assert _slots(n, d, r, B, ids, grad, cores)["prefix_bwd"] == 1
