"""Weight preparation kernels at the edges of their splits: the block selection
over few, many and equal scores, against a stable sort; the diagonal Hessian at
token and channel counts that leave partial steps and on unaligned rows, bit
for bit against the sequential fp64 sum."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import B, _announce, dev, host, mq, tc  # noqa: F401

pytestmark = pytest.mark.gpu


def _scores(kind, NB, KB, rng):
    n = NB * KB
    if kind == "normal":
        s = rng.standard_normal(n) * 10.0 ** rng.integers(-8, 9, n)     # both signs, many exponents
    elif kind == "ties":
        s = rng.integers(-2, 3, n).astype(np.float64)
        s[s == 0] *= rng.choice([1.0, -1.0], int((s == 0).sum()))       # zeros of both signs are equal
    elif kind == "equal":
        s = np.full(n, 3.25)
    else:                                                               # keys that differ in the last bit only
        s = np.where(rng.random(n) < 0.5, 1.0, np.nextafter(1.0, 2.0))
    return s.reshape(NB, KB)


# n = 1, one item a thread with a remainder, the register limit and one past
# it, several tiles
@pytest.mark.parametrize("kind", ["normal", "ties", "equal", "lastbit"])
@pytest.mark.parametrize("NB,KB", [(1, 1), (3, 7), (33, 32), (128, 128), (129, 127), (1, 16385), (300, 200)])
def test_select_blocks_matches_a_stable_sort(tc, mq, kind, NB, KB):
    _check_selection(tc, mq, kind, NB, KB)


# the largest and the next block count of each instantiation of the kernel
@pytest.mark.parametrize("kind", ["normal", "ties", "equal", "lastbit"])
@pytest.mark.parametrize("NB,KB", [(7, 9), (8, 8), (5, 13), (32, 32), (25, 41), (64, 64), (17, 241)])
def test_select_blocks_at_the_split_edges(tc, mq, kind, NB, KB):
    _check_selection(tc, mq, kind, NB, KB)


def _check_selection(tc, mq, kind, NB, KB):
    rng = np.random.default_rng(NB * 1000 + KB)
    score = _scores(kind, NB, KB, rng)
    n = NB * KB
    order = np.argsort(-score.ravel(), kind="stable")
    d = dev(tc, score)
    for nnzb in sorted({0, 1, n // 10, n // 2, n - 1, n}):
        rowptr, kb = mq.select_blocks(d, nnzb)
        tc.cuda.synchronize()
        mask = np.zeros(n, bool)
        mask[order[:nnzb]] = True
        mask = mask.reshape(NB, KB)
        assert np.array_equal(host(rowptr), np.concatenate([[0], np.cumsum(mask.sum(1))])), nnzb
        assert np.array_equal(host(kb), np.nonzero(mask)[1]), nnzb


@pytest.mark.parametrize("T,K,ldx,offset", [(1, 8, 8, 0), (255, 64, 64, 0), (256, 72, 80, 0), (257, 136, 136, 0),
                                            (513, 200, 203, 0), (600, 100, 100, 0), (300, 128, 136, 1)])
def test_hessian_diag_is_the_sequential_sum(tc, mq, T, K, ldx, offset):
    """fp16 values over many binades (some partial sums round, so the order of
    the additions shows)."""
    _check_hessian(tc, mq, T, K, ldx, offset)


# tokens that fill whole sixteens of the last step, and one more or less
@pytest.mark.parametrize("T", [8, 15, 16, 17, 31, 271, 272, 273])
def test_hessian_diag_last_step(tc, mq, T):
    _check_hessian(tc, mq, T, 72, 72, 0)


def _check_hessian(tc, mq, T, K, ldx, offset):
    rng = np.random.default_rng(T + K)
    buf = (rng.standard_normal(T * ldx + 8) * 2.0 ** rng.integers(-9, 10, T * ldx + 8)).astype(np.float16)
    x = np.lib.stride_tricks.as_strided(buf[offset:], (T, K), (2 * ldx, 2)).astype(np.float64)
    acc = np.zeros(K)
    for t in range(T):
        acc = acc + x[t] * x[t]
    want = 2.0 / T * acc
    d = dev(tc, buf)
    h = tc.empty((K,), dtype=tc.float64, device="cuda")
    st = mq.load().mq_hessian_diag(d.data_ptr() + 2 * offset, T, K, ldx, h.data_ptr(), None)
    tc.cuda.synchronize()
    assert st == 0
    assert np.array_equal(host(h), want)
