"""Any-shape batches whose launches, one block or wavefront per chunk of prefixes, would hold 2^32 threads or
more, which a launch cannot: they take the kernels that walk their work with a bounded grid.  The reference is
float64 on the GPU (tables of one column per first-core line, where it is one matrix)."""
import pytest
import torch

from paper_2206_10581_amd import TTEmbedding

pytestmark = pytest.mark.gpu


def _step(n, d2, r2, B):
    gen = torch.Generator(device="cuda").manual_seed(3)
    cores = [torch.randn(s, generator=gen, device="cuda") for s in ((n[0], 1, 1), (n[1], 1, d2, r2), (1, r2, 1))]
    old = [c.double().clone() for c in cores]
    ids = torch.arange(B, device="cuda")
    grad = torch.randn((B, d2), generator=gen, device="cuda") * 1e-3
    emb = TTEmbedding((n[0], n[1], 1), (1, d2, 1), (1, r2), B, cores)
    out = emb.forward(ids)
    emb.backward_update(grad, 0.1)
    assert emb.stats() == {"U": B, "Q": B, "out_of_range": 0}
    emb.close()
    # row i1 of the reference at a time block: ids i1*n2 + i2 of the batch
    g1, g2, g3 = old[0].view(-1), old[1].view(n[1], d2, r2), old[2].view(r2)
    p = g2 @ g3                                                  # n2 x d2
    full = torch.zeros((n[0] * n[1], d2), device="cuda")
    full[:B] = grad
    d1 = torch.zeros_like(g1)
    dp = torch.zeros((n[1], d2), dtype=torch.float64, device="cuda")
    worst = 0.0
    for a in range(0, n[0], 1000):
        b = min(a + 1000, n[0])
        g = full[a * n[1]: b * n[1]].view(b - a, n[1], d2).double()
        d1[a:b] = (g * p).sum((1, 2))
        dp += (g * g1[a:b, None, None]).sum(0)
        have = out[a * n[1]: min(b * n[1], B)].double()
        want = (g1[a:b, None, None] * p).reshape(-1, d2)[: have.shape[0]]
        worst = max(worst, float((have - want).norm() / want.norm()))
    assert worst <= 1e-6
    # G3's gradient is one sum of up to 134 million terms of both signs, added up 16 at a time: a walk of 8.4
    # million partial sums has an error of about 1e-5 of its result (1e-4 of that is allowed of every step)
    steps = (d1, dp[:, :, None] * g3, (dp[:, :, None] * g2).sum((0, 1)))
    for got, was, step in zip(emb.cores, old, steps):
        miss = (got.double() - was).view(-1) + 0.1 * step.reshape(-1)
        assert float(miss.norm()) <= 0.1 * 1e-4 * float(step.norm()) + 2.0 ** -24 * float(was.norm())


def test_blocks_of_the_middle_kernel():
    _step((65_600, 2048), 1, 1, 134_300_000)


def test_strips_of_the_prefix_products():
    _step((14_000, 2000), 20, 32, 27_000_000)
