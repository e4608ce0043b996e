"""Sizes that the host decides, without a launch: what a workspace holds, and the largest batch of the lookup
without one."""
import pytest

from paper_2206_10581_amd import binding
from paper_2206_10581_amd.binding import TT_EMB_ENOSPC, make_config

TABLES = [((136, 136, 136), (4, 4, 8), 32, 372_304), ((480, 480, 482), (4, 4, 8), 16, 58_944),
          ((480, 500, 500), (8, 4, 4), 128, 4_026), ((125, 140, 140), (4, 5, 5), 32, 282_432),
          ((10, 10, 10), (2, 2, 2), 4, 876_544)]


@pytest.mark.parametrize("n,d,r,most", TABLES)
def test_largest_batch_of_the_lookup_without_a_workspace(n, d, r, most):
    def lookup(B):  # a device that is not the current one: nothing is launched, and no address is used
        return binding.tt_emb_lookup_static(make_config(n, d, (r, r), B, 63), 256, 512, 768, 1024, B, 2048, 0)
    assert lookup(most) not in (0, TT_EMB_ENOSPC)
    assert lookup(most + 1) == TT_EMB_ENOSPC


@pytest.mark.parametrize("n,d,r,most", TABLES)
@pytest.mark.parametrize("B", [40_000, 500_000])
def test_every_byte_of_a_workspace_is_used(n, d, r, most, B):
    """Four index sets and the arrays of the arithmetic, each rounded up to 256 bytes."""
    slabs = d[0] // 4 if d == (8, 4, 4) else 1
    n1, d1, b = n[0] * slabs, d[0] // slabs, B * slabs
    q, pn, D = min(b, n1 * n[1]), d1 * d[1] * r, d1 * d[1] * d[2]
    c3, c2 = -(-b // 8) + n[2], -(-q // 16) + n[1]
    up = lambda x, k: -(-x // k)
    sets = (16 * b + 4 * b + 16 * b + 16 * b + 12 * q          # sort, slots, unique ids, prefixes
            + up(b, 1024) * 24 + 2048 * 4 + 8 * n1             # blocks of slots, digit totals, prefixes of an i1
            + up(b, 4096) * (8192 + 4 * n[2]) + up(q, 4096) * 4 * n[1]
            + 32 * n[2] + c3 * (16 + 16 * 8) + c2 * (16 + 16 * 16) + 4 * (n[2] + n[1]))
    arithmetic = 4 * (2 * q * pn + b * D + up(b, 32) * 2 * D + q * d1 * r + c3 * r * d[2] + c2 * r * d[1] * r)
    rc, nbytes = binding.tt_emb_workspace_bytes(make_config(n, d, (r, r), B, flags=binding.TT_EMB_FLAG_INDEXED_KERNELS))
    assert rc == 0
    assert 0 <= nbytes - (4 * sets + arithmetic) <= 256 * 120
