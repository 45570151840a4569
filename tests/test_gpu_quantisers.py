"""Both activation quantisers at the edges of their split (one thread per 32
codes: partial waves, the longest row of one pass, the first of two passes) and
on values of every size: codes, layout bytes and scales bit-exact against the
CPU oracle."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import _announce, dev, gpu_pw, half_bits, host, mq, random_operands, tc  # noqa: F401

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
    _check_quantisers(tc, mq, orc, M, K)


# both sides of every line between the splits: half a quarter or a quarter a
# thread (by rows and length), one, two or more pieces a thread
@pytest.mark.parametrize("M,K", [(9000, 128), (1300, 1024), (70, 1152), (256, 2048), (257, 2048), (1024, 2176), (1025, 2176),
                                 (9, 8192), (9, 8320), (3, 16384), (7, 65536), (7, 65664)])
def test_quantisers_at_the_split_edges(tc, mq, orc, M, K):
    _check_quantisers(tc, mq, orc, M, K)


def _check_quantisers(tc, mq, orc, M, K):
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


@pytest.mark.parametrize("K,N", [(128, 128), (1024, 256), (8192, 128), (16384, 128), (32896, 128), (65664, 128)])
def test_rows_with_infinities_and_nans(tc, mq, orc, K, N):
    """A row with an infinity has an infinite scale and INT4 codes 0, so its
    outputs are NaN; its INT8 codes are -127 where x is infinite and 0
    elsewhere.  A row with a NaN has a NaN scale and outputs, INT4 codes 0 and
    INT8 codes -127.  The rows beside them are as without it."""
    x = _rows(8, K)
    x[1, 5], x[2, K - 1], x[5, 7] = np.inf, -np.inf, np.nan
    x[6] = -np.inf
    x[7, 3], x[7, K // 2] = np.inf, -np.nan
    d = dev(tc, x)
    Xq, s4 = mq.quantize_act(d)
    Xq8, s8 = mq.quantize_act8(d)
    q4, q8 = host(mq.unpack_act(Xq)), host(mq.unpack_act8(Xq8))
    for s in (host(s4), host(s8)):
        assert np.array_equal(np.isinf(s), [0, 1, 1, 0, 0, 0, 1, 0]) and np.array_equal(np.isnan(s), [0, 0, 0, 0, 0, 1, 0, 1])
    bad = [1, 2, 5, 6, 7]
    assert not q4[bad].any()
    nan_row = np.isnan(x).any(1)
    want8 = np.where(nan_row[:, None] | ~np.isfinite(x), -127, 0)
    assert np.array_equal(q8[bad], want8[bad])
    good = [0, 3, 4]
    assert np.array_equal(q8[good], orc.quantize_act8(x[good])[0])
    ops = random_operands(1, N, K, 1, seed=K)
    pw = gpu_pw(tc, mq, N, K, *ops[2:6], *ops[7:])
    for rows in ([1], [0, 1, 2, 3], [4, 5, 6, 7], list(range(8))):      # one kernel at few codes, two otherwise
        Y = host(mq.linear(d[rows].contiguous(), pw))
        assert np.array_equal(np.isnan(Y).all(1), [r in bad for r in rows])
        assert np.array_equal(np.isnan(Y).any(1), [r in bad for r in rows])
