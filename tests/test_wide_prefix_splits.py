"""Ranks 64 and 128: the products of the prefix kernels are formed from bf16 parts of their operands, which do
not hold for infinities, for numbers that round up to one and for very small ones; tiles that meet such
numbers are formed again.  The reference is float64."""
import numpy as np
import pytest
import torch

from paper_2206_10581_amd import TTEmbedding

pytestmark = pytest.mark.gpu

N3, D3_, B = (11, 9, 10), (4, 4, 4), 900
FLAG_INDEXED = 8


def _case(r, seed=0):
    rng = np.random.default_rng(seed)
    shapes = ((N3[0], D3_[0], r), (N3[1], r, D3_[1], r), (N3[2], r, D3_[2]))
    cores = [rng.standard_normal(s).astype(np.float32) / np.float32(np.sqrt(r)) for s in shapes]
    ids = rng.integers(0, N3[0] * N3[1] * N3[2], B)
    grad = rng.standard_normal((B, 64)).astype(np.float32)
    return cores, ids, grad


def _gpu(cores, ids, grad, r, lr=1.0):
    emb = TTEmbedding(N3, D3_, (r, r), B, [c.copy() for c in cores], flags=FLAG_INDEXED)
    out = emb.forward(torch.from_numpy(ids).cuda()).cpu().numpy()
    emb.backward_update(torch.from_numpy(grad).cuda(), lr)
    torch.cuda.synchronize()
    new = [c.cpu().numpy() for c in emb.cores]
    emb.close()
    return out, new


def _ref(cores, ids, grad, r):
    c1, c2, c3 = (torch.from_numpy(c.astype(np.float64)).requires_grad_() for c in cores)
    i1, i2, i3 = (torch.from_numpy(x) for x in (ids // 90, ids // 10 % 9, ids % 10))
    p = torch.bmm(c1[i1], c2[i2].reshape(B, r, 4 * r)).reshape(B, 16, r)
    out = torch.bmm(p, c3[i3]).reshape(B, 64)
    (out * torch.from_numpy(grad.astype(np.float64))).sum().backward()
    return out.detach().numpy(), [c.grad.numpy() for c in (c1, c2, c3)]


def _check_steps(old, new, ref, lr):
    """The steps the cores took, recovered from them.  2e-6: sums of at most 900 * 64 terms of random signs, whose
    roundings add up to a few 2^-24, and the rounding of the core that the step is added to."""
    for o, g, x in zip(old, ref, new):
        step = lr * g
        assert np.linalg.norm((o.astype(np.float64) - x) - step) <= 2e-6 * max(np.linalg.norm(step), np.linalg.norm(o))
        assert np.linalg.norm(step) >= 0.2 * np.linalg.norm(o)      # (the bound is one on the step)


@pytest.mark.parametrize("r", [64, 128])
@pytest.mark.parametrize("scale", [1.0, 2.0 ** -100, 2.0 ** -110, 2.0 ** -118, 2.0 ** 60])
def test_scaled_gradients(r, scale):
    """Gradients of G1 and G2 keep their accuracy down to the end of the normal range, where the lower parts of
    their operands are no bf16 numbers any more.  (The leading part alone is off by 2^-10 of a step.)"""
    cores, ids, grad = _case(r)
    grad *= np.float32(scale)
    old = [c.copy() for c in cores]
    _, new = _gpu(cores, ids, grad, r, 1.0 / scale)
    _, ref = _ref(cores, ids, grad, r)
    _check_steps(old, new, ref, 1.0 / scale)


@pytest.mark.parametrize("r", [64, 128])
@pytest.mark.parametrize("small,large", [(-106, 40), (-112, 60), (-118, 80), (-124, 100)])
def test_small_numbers_with_large_factors(r, small, large):
    """Small operands whose products are ordinary numbers: nothing in the results tells of the parts they lost."""
    cores, ids, grad = _case(r, 3)
    # prefix products: G1 small, G2 large, and the other way round
    for k in (0, 1):
        c = [x.copy() for x in cores]
        c[k] *= np.float32(2.0 ** small)
        c[1 - k] *= np.float32(2.0 ** large)
        out, _ = _gpu(c, ids, grad, r, 0.0)
        want = _ref(c, ids, grad, r)[0]
        assert np.linalg.norm(out - want) <= 1e-6 * np.linalg.norm(want)
    # gradients of one core: small dPsum times a large core, step by step in units of its own
    for k in (0, 1):
        c, g = [x.copy() for x in cores], grad * np.float32(2.0 ** small)
        c[1 - k] *= np.float32(2.0 ** large)
        lr = 2.0 ** -(small + large)
        _, new = _gpu(c, ids, g, r, lr)
        _, ref = _ref(c, ids, g, r)
        _check_steps([c[k]], [new[k]], [ref[k]], lr)


@pytest.mark.parametrize("r", [64, 128])
@pytest.mark.parametrize("big", [np.inf, 3.4e38])
def test_infinite_and_largest_entries(r, big):
    """One entry of G1 that has no finite bf16 neighbour: rows of its slice read it, others do not."""
    cores, ids, grad = _case(r, 1)
    cores[0][4, 2, 7] = big
    cores[1] = np.abs(cores[1])                      # no cancellation of infinities of both signs
    cores[2] = np.abs(cores[2]) * np.float32(1e-3)
    out, _ = _gpu(cores, ids, grad * 0, r)
    rows = out.reshape(B, 4, 16)
    hit = ids // 90 == 4
    assert np.isfinite(rows[~hit]).all() and np.isfinite(rows[hit][:, [0, 1, 3]]).all()
    with np.errstate(invalid="ignore", over="ignore"):
        want = _ref(cores, ids, grad * 0, r)[0].reshape(B, 4, 16)[hit][:, 2].astype(np.float32)
    got = rows[hit][:, 2]
    assert np.array_equal(np.isnan(got), np.isnan(want))
    if big == np.inf:
        assert np.array_equal(got, want)
    else:
        assert np.abs(got / want - 1).max() <= 1e-5


@pytest.mark.parametrize("r", [64, 128])
def test_tiny_cores(r):
    """Cores of G1 near the smallest normal number: products keep their relative accuracy."""
    cores, ids, grad = _case(r, 2)
    cores[0] *= np.float32(2.0 ** -112)
    out, _ = _gpu(cores, ids, grad, r, 0.0)
    want = _ref(cores, ids, grad, r)[0]
    assert np.linalg.norm(out - want) <= 1e-6 * np.linalg.norm(want)
