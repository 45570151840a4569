"""Both activation quantisers at the edges of their split (one thread per 32
codes: partial waves, the longest row of one pass, the first of two passes) and
on values of every size: codes, layout bytes and scales bit-exact against the
CPU oracle."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import _announce, dev, half_bits, host, mq, tc  # noqa: F401

pytestmark = pytest.mark.gpu


def _rows(M, K):
    """Normal rows, rows over many binades, rows of multiples of half their
    scale (ties), subnormal rows, a zero row and rows of one large value."""
    rng = np.random.default_rng(M * 7 + K)
    x = rng.standard_normal((M, K))
    x[0::6] *= 2.0 ** rng.integers(-12, 12, (len(x[0::6]), K))
    for r in range(1, M, 6):
        q = 127 if r % 12 == 1 else 7
        x[r] = rng.integers(-2 * q, 2 * q + 1, K) * 2.0 ** rng.integers(-14, 6) / 2
        x[r, 0] = np.abs(x[r]).max()
    x[2::6] *= 2.0 ** -24 * 20
    x[3::6] = 0
    if M > 4:
        x[4] = np.sign(x[4]) * 2.0 ** -24
        x[4, K // 2] = 65504
    return x.astype(np.float16)


@pytest.mark.parametrize("M,K", [(1, 128), (13, 2176), (31, 4096), (7, 32768), (7, 32896), (300, 1024), (64, 8192)])
def test_quantisers_bit_exact(tc, mq, orc, M, K):
    x = _rows(M, K)
    d = dev(tc, x)
    Xq, s4 = mq.quantize_act(d)
    Xq8, s8 = mq.quantize_act8(d)
    codes8 = mq.unpack_act8(Xq8)
    again = mq.repack_act8(codes8)
    tc.cuda.synchronize()
    q4, r4 = orc.quantize_act(x)
    q8, r8 = orc.quantize_act8(x)
    assert np.array_equal(half_bits(s4), r4) and np.array_equal(half_bits(s8), r8)
    assert np.array_equal(orc.packed_from_act6(host(Xq), K), q4)
    assert np.array_equal(host(codes8), q8)
    assert np.array_equal(host(again), host(Xq8))       # every layout byte, zeros of either sign as +0
