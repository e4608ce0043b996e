"""The kernels that need no index structures (small batches, runs of table rows) at the sizes where
their work is cut: teams of one and four wavefronts, batch sizes around a block of items and around
the largest batch they take, dimension factors and ranks that leave tiles part empty, runs of rows
that begin and end inside a prefix.  Oracle and tolerances are those of test_gpu_parity."""
import numpy as np
import pytest

from oracle import tt_oracle as ora
from oracle.tt_oracle import Shape
from tests.test_gpu_parity import ROW_TOL, check_against_oracle, row_error, run_gpu

pytestmark = pytest.mark.gpu

SHAPES = [((5, 6, 7), (2, 2, 2), (4, 4)), ((9, 11, 13), (4, 4, 8), (8, 8)), ((9, 11, 13), (4, 4, 4), (16, 16)),
          ((9, 11, 13), (4, 4, 8), (32, 32)), ((7, 5, 9), (8, 4, 4), (64, 64)), ((5, 4, 9), (4, 4, 8), (128, 128)),
          ((8, 7, 6), (4, 5, 5), (32, 32)), ((8, 7, 6), (4, 5, 5), (16, 16)), ((4, 3, 5), (3, 5, 7), (6, 10)),
          ((4, 3, 5), (5, 3, 2), (7, 3)), ((4, 3, 5), (9, 2, 3), (130, 5))]


def _inputs(n, d, r, B, seed):
    s = Shape(n, d, r)
    rng = np.random.default_rng(seed)
    cores = tuple((rng.standard_normal(c) / np.sqrt(r[0])).astype(np.float32) for c in s.core_shapes())
    ids = rng.integers(0, s.N, B).astype(np.int64)
    ids[: B // 4] = ids[0]                                   # a hot id
    if B > 8:
        ids[B // 2: B // 2 + 3] = [-1, s.N, 1 << 40]
    grad = rng.standard_normal((B, s.D)).astype(np.float32)
    return s, cores, ids, grad


@pytest.mark.parametrize("n,d,r", SHAPES)
@pytest.mark.parametrize("B", [1, 4, 63, 515])
def test_small_batches(n, d, r, B):
    _, cores, ids, grad = _inputs(n, d, r, B, 31 * B + r[0])
    check_against_oracle(n, d, r, cores, ids, grad, 0.01)


@pytest.mark.parametrize("n,d,r,B", [((9, 11, 13), (4, 4, 4), (16, 16), 8192), ((9, 11, 13), (4, 4, 4), (16, 16), 8193),
                                     ((9, 11, 13), (4, 4, 8), (32, 32), 4096), ((9, 11, 13), (4, 4, 8), (32, 32), 4097),
                                     ((5, 6, 7), (2, 2, 2), (4, 4), 2049), ((5, 6, 7), (2, 2, 2), (4, 4), 8191)])
def test_around_the_largest_batch(n, d, r, B):
    _, cores, ids, grad = _inputs(n, d, r, B, B)
    check_against_oracle(n, d, r, cores, ids, grad, 0.01)


@pytest.mark.parametrize("n,d,r", SHAPES + [((3, 5, 136), (4, 4, 8), (32, 32)), ((3, 4, 200), (4, 5, 5), (32, 32))])
def test_runs_of_table_rows(n, d, r):
    import torch
    from paper_2206_10581_amd import TTEmbedding
    s, cores, _, _ = _inputs(n, d, r, 16, 5)
    table = ora.forward(s, *cores, np.arange(s.N, dtype=np.int64))
    emb = TTEmbedding(n, d, r, 10, cores)
    for first, count in [(0, s.N), (1, 1), (n[2] - 1, 2), (n[2] + 1, n[2] - 2), (s.N - 3, 3), (2, s.N // 2)]:
        out = torch.full((count + 2, s.D), 7.0, device="cuda")      # rows around the run stay as they are
        emb.materialize(first, count, out[1:-1])
        got = out.cpu().numpy()
        assert row_error(got[1:-1], table[first:first + count]) <= ROW_TOL, (first, count)
        assert (got[0] == 7).all() and (got[-1] == 7).all()
    emb.close()


@pytest.mark.parametrize("flags", [0, 2])
@pytest.mark.parametrize("n,d,r", [((5, 6, 7), (2, 2, 2), (4, 4)), ((4, 3, 5), (3, 5, 7), (7, 10)),
                                   ((4, 3, 5), (1, 2, 4), (20, 3)), ((4, 3, 5), (5, 3, 2), (18, 3)),
                                   ((9, 11, 13), (4, 4, 8), (8, 8))])
def test_infinities_stay_where_they_belong(n, d, r, flags):
    """An infinity in the last row of a G2 slice reaches the rows of that slice as an infinity, and one
    in a gradient the slices of its id: operands padded to the size of a tile or a round of loads add
    nothing, where zero times the repeated value would make them NaN.  The oracle pads nothing."""
    s, cores, _, grad = _inputs(n, d, r, 40, 3)
    ids = np.random.default_rng(4).integers(0, s.N, 40).astype(np.int64)
    first = int(ids[0])
    i2 = (first // n[2]) % n[1]

    def same_specials(got, ref):
        got, ref = np.asarray(got, np.float64), np.asarray(ref, np.float64)
        np.testing.assert_array_equal(np.isnan(got), np.isnan(ref))
        np.testing.assert_array_equal(np.where(np.isinf(got), np.sign(got), 0), np.where(np.isinf(ref), np.sign(ref), 0))

    hot = [c.copy() for c in cores]
    hot[1][i2, r[0] - 1, 0, 0] = np.inf
    ref = ora.forward(s, *hot, ids)
    assert np.isinf(ref[0]).any() and not np.isnan(ref).any()
    out, _, _ = run_gpu(n, d, r, hot, ids, grad, 0.0, flags=flags)
    same_specials(out, ref)
    g = grad.copy()
    g[0, s.D - 1] = np.inf                                   # the last row of the (j1,j2) index
    ref = ora.backward_update(s, *cores, ids, g, 0.01)
    assert np.isinf(ref[1]).any() and not np.isnan(ref[1]).any()
    _, new, _ = run_gpu(n, d, r, cores, ids, g, 0.01, flags=flags)
    for k in range(3):
        same_specials(new[k], ref[k])


def _core_errors(n, d, r, B, flags=0):
    """Per core, 2-norm of the error of a step over 2-norm of the step, for a batch of one id with cores
    and gradients of one sign (nothing cancels) and a step that dwarfs the cores."""
    s = Shape(n, d, r)
    rng = np.random.default_rng(B + r[0])
    cores = tuple((np.abs(rng.standard_normal(c)) / np.sqrt(r[0])).astype(np.float32) for c in s.core_shapes())
    ids = np.full(B, s.N // 2, dtype=np.int64)
    grad = (1e4 * np.abs(rng.standard_normal((B, s.D)))).astype(np.float32)
    _, new, _ = run_gpu(n, d, r, cores, ids, grad, 1.0, flags=flags)
    ref = [c.astype(np.float64) for c in ora.backward_update(s, *cores, ids, grad, 1.0)]
    return [np.linalg.norm(new[k] - ref[k]) / np.linalg.norm(cores[k] - ref[k]) for k in range(3)]


@pytest.mark.parametrize("n,d,r,B", [((9, 11, 13), (4, 4, 4), (16, 16), 1024), ((9, 11, 13), (4, 4, 8), (32, 32), 1024),
                                     ((9, 11, 13), (4, 4, 8), (64, 64), 1024), ((4, 3, 5), (5, 3, 2), (7, 3), 2048),
                                     ((9, 11, 13), (2, 2, 2), (4, 4), 100), ((9, 11, 13), (2, 2, 2), (4, 4), 2048)])
def test_sums_of_a_hot_id_add_in_two_levels(n, d, r, B):
    """m roundings of rms 0.41 u each (u = 2^-24) on growing partial sums leave 0.41 u sqrt(m / 3).  Chains
    are at most 64 rounds long here, two side by side at least: 0.41 u sqrt(64/3/2 + 2) = 8.7e-8 at
    most with the last additions.  In one chain the 1024 terms of a wavefront's share would leave
    0.41 u sqrt(1024/3/4) = 2.3e-7."""
    assert max(_core_errors(n, d, r, B)) <= 1.2e-7


@pytest.mark.parametrize("n,d,r", [((16400, 1024, 1), (2, 2, 1), (3, 2)),        # 16.8 million prefixes, a block each
                                   ((2050, 2048, 1), (4, 4, 4), (128, 128))])   # 4.2 million, a wavefront each
def test_table_rows_over_several_launches(n, d, r):
    """One launch holds fewer than 2^32 threads: a run of that many prefixes is cut into launches of a
    million blocks.  Rows around every cut and a sample of the others, against the oracle."""
    import torch
    from paper_2206_10581_amd import TTEmbedding
    s = Shape(n, d, r)
    gen = torch.Generator(device="cuda").manual_seed(1)
    cores = [torch.randn(c, generator=gen, device="cuda") / r[0] ** 0.5 for c in s.core_shapes()]
    emb = TTEmbedding(n, d, r, 10, cores)
    first, count = 1, s.N - 2
    out = torch.full((count + 2, s.D), 7.0, device="cuda")
    emb.materialize(first, count, out[1:-1])
    cuts = np.arange(0, s.N, 1 << 20)[:, None] + np.arange(-3, 4)
    rows = np.unique(np.concatenate([cuts.ravel(), np.random.default_rng(2).integers(0, s.N, 20_000), [1, s.N - 2]]))
    rows = rows[(rows >= first) & (rows < first + count)]
    got = out[torch.from_numpy(rows).cuda()].cpu().numpy()   # out[0] stands before row 1
    err = np.abs(got - ora.forward(s, *(c.cpu().numpy() for c in cores), rows)).max(1)
    # rows of four or 64 elements: relative to a typical row, not to one that may cancel
    assert err.max() <= ROW_TOL * np.abs(got).max(1).mean()
    assert (out[0] == 7).all() and (out[-1] == 7).all()
    emb.close()


def test_table_rows_by_lookup():
    """Products and G3 slices beyond a block's LDS: the run is looked up, max_batch rows at a time."""
    from paper_2206_10581_amd import TTEmbedding
    n, d, r = (3, 4, 5), (4, 4, 256), (4, 8)
    s, cores, _, _ = _inputs(n, d, r, 16, 5)
    emb = TTEmbedding(n, d, r, 10, cores)
    emb.profile(True)
    got = emb.materialize(7, 37).cpu().numpy()
    assert emb.profile_read()["table"]["launches"] == 0
    assert row_error(got, ora.forward(s, *cores, np.arange(7, 44, dtype=np.int64))) <= ROW_TOL
    emb.close()


@pytest.mark.parametrize("B", [1, 63, 149, 150, 151, 299, 301])
@pytest.mark.parametrize("d,r", [((4, 4, 8), (16, 16)), ((5, 3, 2), (7, 3)), ((2, 2, 2), (4, 4))])
def test_fewer_items_than_slices(d, r, B):
    """Cores with more slices than the batch has items, with as many, and with fewer: ids that share one
    coordinate and no other, the first position out of range, the last one's slices its own."""
    n = (300, 150, 151)
    s, cores, _, grad = _inputs(n, d, r, B, B)
    rng = np.random.default_rng(B)
    i1, i2, i3 = (rng.integers(0, k - 1, B) for k in n)
    i1[B // 5: B // 3], i2[B // 4: B // 2], i3[B // 3:] = i1[0], i2[-1], i3[B // 2]
    ids = (i1 * n[1] + i2) * n[2] + i3
    if B > 1:
        ids[0] = -1
    ids[-1] = s.N - 1
    check_against_oracle(n, d, r, cores, ids.astype(np.int64), grad, 0.01)


def test_two_ids_of_a_table_with_two_to_the_31_entries():
    """A middle core of 2^31 floats: the kernels launch for the two slices that the batch touches."""
    import torch
    from paper_2206_10581_amd import TTEmbedding
    n, d, r = (2, 2048, 2), (1, 1, 1), (1024, 1024)
    gen = torch.Generator(device="cuda").manual_seed(3)
    cores = [torch.randn((2, 1, 1024), generator=gen, device="cuda"), torch.zeros((2048, 1024, 1, 1024), device="cuda"),
             torch.randn((2, 1024, 1), generator=gen, device="cuda")]
    i2 = [5, 2047]
    cores[1][i2] = torch.randn((2, 1024, 1, 1024), generator=gen, device="cuda") / 32
    small = [c.cpu().numpy() for c in (cores[0], cores[1][i2], cores[2])]
    ids = torch.tensor([(0 * 2048 + i2[0]) * 2 + 1, (1 * 2048 + i2[1]) * 2], device="cuda")
    grad = torch.ones((2, 1), device="cuda")
    emb = TTEmbedding(n, d, r, 2, cores)
    emb.profile(True)
    out = emb.forward(ids)
    emb.backward_update(grad, 0.01)
    torch.cuda.synchronize()
    assert emb.profile_read()["direct_apply"]["launches"] == 1
    s = Shape((2, 2, 2), d, r)
    small_ids = np.array([(0 * 2 + 0) * 2 + 1, (1 * 2 + 1) * 2], dtype=np.int64)
    # rows are about 32: sums of 1024 products of unit scale
    np.testing.assert_allclose(out.cpu().numpy(), ora.forward(s, *small, small_ids), rtol=0, atol=32 * ROW_TOL)
    ref = ora.backward_update(s, *small, small_ids, np.ones((2, 1), np.float32), 0.01)
    for got, want in zip((cores[0], cores[1][i2], cores[2]), ref):
        np.testing.assert_allclose(got.cpu().numpy(), want, rtol=0, atol=1e-4 * np.abs(want).max())
    cores[1][i2] = 0
    assert torch.count_nonzero(cores[1].view(-1)[: 1 << 30]).item() == 0
    assert torch.count_nonzero(cores[1].view(-1)[1 << 30:]).item() == 0
    emb.close()


def test_lookup_consumes_the_batch_prepared_for_it():
    """Between the limits of the two directions (some 500 and 8192 ids here) a batch is prepared, but a
    lookup of it takes the index-free kernels.  The lookup uses up what was prepared all the same: when
    the caller then fills the same buffer with other ids, the next forward sees those."""
    import torch
    from paper_2206_10581_amd import TTEmbedding
    n, d, r, B = (9, 11, 13), (8, 9, 1), (2, 100), 1000
    s, cores, ids, _ = _inputs(n, d, r, B, 6)
    buf = torch.from_numpy(ids).cuda()
    emb = TTEmbedding(n, d, r, B, cores)
    emb.prepare(buf)
    assert row_error(emb.forward_eval(buf).cpu().numpy(), ora.forward(s, *cores, ids)) <= ROW_TOL
    ids = np.ascontiguousarray(ids[::-1])
    buf.copy_(torch.from_numpy(ids))
    emb.profile(True)
    assert row_error(emb.forward(buf).cpu().numpy(), ora.forward(s, *cores, ids)) <= ROW_TOL
    assert emb.profile_read()["sort_hist"]["launches"] > 0     # its structures were built for it
    emb.close()


def test_small_steps_leave_prepared_batches_alone():
    """With a batch waiting in every index set, a step on the index-free kernels and the counts of its
    batch (the host counts them) use up none: all four are served afterwards without a sort.  The
    profile names the step's own launches only."""
    import torch
    from paper_2206_10581_amd import TTEmbedding
    n, d, r, B, small = (9, 11, 13), (4, 4, 4), (16, 16), 9000, 300
    s, cores, ids, grad = _inputs(n, d, r, B, 7)
    emb = TTEmbedding(n, d, r, B, cores, flags=4)             # the ids are in memory at every prepare
    valid = ids[(ids >= 0) & (ids < s.N)]
    bufs = [torch.from_numpy(np.roll(ids, k)).cuda() for k in range(4)]
    t_grad = torch.from_numpy(grad).cuda()
    torch.cuda.synchronize()
    for b in bufs:
        emb.prepare(b)
    torch.cuda.synchronize()
    emb.profile(True)
    few = bufs[1][:small].clone()
    for _ in range(5):                                        # more steps than there are events for them
        out = emb.forward(few)
        emb.backward_update(t_grad[:small], 0.0)
        emb.wait_backward(1)
    st = emb.stats(check=False)
    f = few.cpu().numpy()
    inside = f[(f >= 0) & (f < s.N)]
    assert st == {"U": np.unique(inside).size, "Q": np.unique(inside // n[2]).size, "out_of_range": small - inside.size}
    assert row_error(out.cpu().numpy(), ora.forward(s, *cores, f)) <= ROW_TOL
    for b in bufs:
        out = emb.forward(b)
        emb.backward_update(t_grad, 0.0)
        assert row_error(out.cpu().numpy(), ora.forward(s, *cores, b.cpu().numpy())) <= ROW_TOL
        st = emb.stats(check=False)
        assert st["out_of_range"] == B - valid.size and st["U"] == np.unique(valid).size
    launches = {k: v["launches"] for k, v in emb.profile_read().items() if v["launches"]}
    assert launches["direct_fwd"] == 5 and launches["prefix_fwd"] == 4 and "sort_hist" not in launches
    emb.close()


def test_prepare_of_a_small_batch_orders_its_forward():
    """Small batches need no index work, but prepare still takes over the order of its stream: ids that
    are on their way on one stream when prepare is called there are awaited by the forward on another.
    The copies wait behind a kernel that spins for some tens of milliseconds."""
    import torch
    from paper_2206_10581_amd import TTEmbedding
    n, d, r, B = (9, 11, 13), (4, 4, 8), (16, 16), 300
    s, cores, ids, _ = _inputs(n, d, r, B, 8)
    emb = TTEmbedding(n, d, r, B, cores)
    batches = [torch.from_numpy(np.roll(ids, k)).cuda() for k in range(3)]
    bufs = [torch.zeros_like(b) for b in batches]
    out = torch.empty((B, s.D), device="cuda")
    emb.prepare(bufs[0])                                      # streams and events exist from here on
    emb.forward(bufs[0], out)
    loader = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(loader):
        torch.cuda._sleep(50_000_000)
        for b, src in zip(bufs, batches):
            b.copy_(src)
            emb.prepare(b)
    got = [emb.forward(bufs[0], out).clone()]
    emb.backward_update(torch.zeros((B, s.D), device="cuda"), 0.0)
    got += [emb.forward_eval(b).clone() for b in bufs[1:]]
    torch.cuda.synchronize()
    for x, b in zip(got, batches):
        assert row_error(x.cpu().numpy(), ora.forward(s, *cores, b.cpu().numpy())) <= ROW_TOL
    emb.close()


@pytest.mark.parametrize("n,d,r", [((9, 11, 13), (4, 4, 8), (16, 16)), ((9, 11, 13), (4, 4, 4), (64, 64)),
                                   ((40, 30, 20), (8, 4, 4), (16, 16)), ((9, 11, 300), (5, 3, 2), (7, 300)), ((9, 8, 7), (20, 1, 9), (70, 2))])
@pytest.mark.parametrize("hot", [64, 65, 256, 257, 511, 512, 513, 1024, 1025, 1300])
def test_slices_of_many_items_in_parts(n, d, r, hot):
    """Slices that as many items share as a part holds (64 to 512) and slices that more share, one of every core, beside slices with few
    items and slices with a part and a bit: parts that are full and one item long.  The parts are
    listed in the order in which the device counts, the sums do not depend on it."""
    rng, B = np.random.default_rng(hot), 2000 if r[0] < 64 else 1024   # more than two parts of every shape
    hot = min(hot, B)
    i = [rng.integers(0, k, B) for k in n]
    i[0][:hot], i[1][:hot], i[2][:hot] = 1, 2, 3              # one id
    i[1][hot:hot + 600] = 4                                   # a shared slice of G2 only
    ids = ((i[0] * n[1] + i[1]) * n[2] + i[2]).astype(np.int64)
    rng.shuffle(ids)
    s, cores, _, grad = _inputs(n, d, r, B, hot)
    _, new, _ = check_against_oracle(n, d, r, cores, ids, grad, 0.01)
    for _ in range(3):
        _, again, _ = run_gpu(n, d, r, cores, ids, grad, 0.01)
        for a, b in zip(new, again):
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("n,d,max_batch,streamed", [((128, 132, 2), (4, 4, 8), 32_768, False),
                                                    ((128, 132, 2), (8, 4, 4), 32_768, False),
                                                    ((128, 132, 2), (4, 4, 8), 32_767, True),
                                                    ((128, 132, 1), (4, 5, 5), 16_384, False),
                                                    ((32, 32, 17), (4, 4, 8), 17_408, True)])
def test_large_products_with_few_rows_are_looked_up(n, d, max_batch, streamed):
    """Rank 128: rows are streamed unless few of them share a product and many products are asked for at
    once, where the lookup's sharing of the G2 slices pays."""
    from paper_2206_10581_amd import TTEmbedding
    r = (128, 128)
    s, cores, _, _ = _inputs(n, d, r, 16, 9)
    emb = TTEmbedding(n, d, r, max_batch, cores)
    emb.profile(True)
    got = emb.materialize(1, s.N - 2).cpu().numpy()
    assert (emb.profile_read()["table"]["launches"] > 0) == streamed
    assert row_error(got, ora.forward(s, *cores, np.arange(1, s.N - 1, dtype=np.int64))) <= ROW_TOL
    emb.close()
