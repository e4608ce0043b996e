"""Lookups of the matrix-core shapes with ranks up to 32 (ids sorted by prefix, i2 in front, products
formed tile by tile): every tile length, slab count, rank and row width, tiles that end inside a prefix and
a G2 slice, out-of-range ids, renumbered ids.  Rows are compared bit by bit with the kernels that have index
structures (flag 8), which add the same terms in the same order and which test_gpu_parity compares with the
oracle; counters with NumPy."""
import numpy as np
import pytest
import torch

from paper_2206_10581_amd import TTEmbedding, binding

pytestmark = pytest.mark.gpu


def _ids(kind, N, B, rng):
    ids = rng.integers(0, N, B)
    if kind == "hot":
        ids[rng.permutation(B)[: B // 2]] = N - 1
    if B > 16:
        ids[3:7] = [-1, N, 1 << 40, 0]
    return ids.astype(np.int64)


def _lookup(n, d, r, cores, ids, flags, new_id=None):
    emb = TTEmbedding(n, d, (r, r), ids.size, cores, flags=flags)
    if new_id is not None:
        emb.set_reindex(new_id)
    out = emb.forward_eval(torch.from_numpy(ids).cuda()).clone()
    stats = [emb.stats(check=False) for _ in range(2)]
    assert stats[0] == stats[1]
    emb.close()
    return out, stats[0]


def _compare(n, d, r, B, kind, reindex=False):
    N = n[0] * n[1] * n[2]
    rng = np.random.default_rng(B + r)
    cores = [torch.from_numpy((rng.standard_normal(s) / np.sqrt(r)).astype(np.float32)).cuda()
             for s in ((n[0], d[0], r), (n[1], r, d[1], r), (n[2], r, d[2]))]
    ids = _ids(kind, N, B, rng)
    new_id = torch.from_numpy(rng.permutation(N).astype(np.int32)).cuda() if reindex else None
    out, stats = _lookup(n, d, r, cores, ids, 0, new_id)
    ref, ref_stats = _lookup(n, d, r, cores, ids, binding.TT_EMB_FLAG_INDEXED_KERNELS, new_id)
    assert torch.equal(out, ref)
    rows = ids[(ids >= 0) & (ids < N)]
    if reindex:
        rows = new_id.cpu().numpy()[rows]
    assert stats == ref_stats
    assert stats == {"U": np.unique(rows).size, "Q": np.unique(rows // n[2]).size, "out_of_range": B - rows.size}


# tiles of 16, 32 and 64 slots: the largest batch of each and the one above, odd sizes
@pytest.mark.parametrize("B", [8_193, 16_384, 16_385, 50_001, 262_144, 262_145])
@pytest.mark.parametrize("r", [8, 16, 32])
def test_tiles(r, B):
    _compare((30, 28, 33), (4, 4, 8), r, B, "uniform")
    _compare((210, 190, 50), (4, 4, 4), r, B, "hot")


# slabs of four lines of G1: one to eight, in one round and in two
@pytest.mark.parametrize("d1", [4, 8, 12, 16, 20, 32])
@pytest.mark.parametrize("r,d3", [(8, 8), (16, 4), (32, 8)])
def test_slabs(r, d3, d1):
    _compare((41, 37, 19), (d1, 4, d3), r, 9_001, "hot")
    _compare((41, 37, 19), (d1, 4, d3), r, 17_003, "uniform", reindex=True)


# with and without loads ahead: the most ids that have them and one more, slabs in one round and in two; large batches
@pytest.mark.parametrize("d1,r,d3,B", [(4, 32, 8, 131_072), (4, 16, 4, 131_073), (8, 8, 4, 98_304), (8, 32, 8, 98_305),
                                       (20, 16, 4, 40_001), (4, 32, 8, 16_384), (8, 32, 4, 16_384), (20, 32, 4, 16_384),
                                       (8, 32, 8, 16_385), (20, 32, 8, 16_385)])
def test_loads_ahead(d1, r, d3, B):
    _compare((41, 37, 19), (d1, 4, d3), r, B, "hot")


# one prefix in all, one i2, one i3, few ids of a large table
@pytest.mark.parametrize("n", [(1, 1, 50), (60, 1, 1), (1, 70, 1), (400, 900, 7), (3, 1000, 900)])
def test_table_forms(n):
    _compare(n, (4, 4, 4), 16, 9_999, "uniform")
    _compare(n, (8, 4, 8), 32, 9_999, "hot")


def test_largest_keys():
    _compare((2_095_000, 1, 1025), (4, 4, 4), 8, 20_001, "uniform")


def test_an_infinity_stays_one():
    """Rows of other ids in the tile, slab and batch of one that reads an infinite core entry stay finite."""
    n, d, r = (5, 6, 40), (8, 4, 4), 16
    rng = np.random.default_rng(0)
    cores = [torch.from_numpy((rng.standard_normal(s) / 4).astype(np.float32)).cuda()
             for s in ((n[0], d[0], r), (n[1], r, d[1], r), (n[2], r, d[2]))]
    cores[0][2, 1, 3] = float("inf")
    cores[2][7, 5, 2] = float("nan")
    ids = rng.integers(0, 1200, 9_000).astype(np.int64)
    out, _ = _lookup(n, d, r, cores, ids, 0)
    ref, _ = _lookup(n, d, r, cores, ids, binding.TT_EMB_FLAG_INDEXED_KERNELS)
    assert torch.equal(out.isnan(), ref.isnan()) and torch.equal(out.nan_to_num(), ref.nan_to_num())
    touched = (ids // 240 == 2) | (ids % 40 == 7)
    assert torch.equal(torch.isfinite(out).all(1).cpu(), torch.from_numpy(~touched))
