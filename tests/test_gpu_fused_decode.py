"""The one-kernel layer call (quantisation fused into the decode GEMM) against
mq_quantize_act followed by mq_fused_gemm, bit for bit: every row count it
takes, rows whose pieces share waves, threads of half a quarter and of quarters
(up to 4096 codes, and beyond), one tile and several tiles a workgroup, zero
rows and ties."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import _announce, dev, gpu_pw, mq, random_operands, tc  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K,nnzb", [(256, 128, 1), (384, 640, 3), (1024, 4096, 30), (16384, 1024, 100), (512, 2176, 0)])
def test_fused_decode_equals_two_calls(tc, mq, N, K, nnzb):
    _check_fused_decode(tc, mq, N, K, nnzb)


# more two-strip tiles (640, 768) than two workgroups a CU hold, and at least
# eight groups: workgroups take several tiles, at every M
@pytest.mark.parametrize("N,K,nnzb", [(20480, 1024, 100), (24576, 2048, 300)])
def test_fused_decode_several_tiles_a_workgroup(tc, mq, N, K, nnzb):
    assert N // 32 > 2 * 256 and K // 128 >= 8
    _check_fused_decode(tc, mq, N, K, nnzb)


# 4096 codes at M = 8; 3840 and 4480 at M = 6 and 7; one code piece a row more than a wave
@pytest.mark.parametrize("N,K,nnzb", [(384, 512, 4), (256, 640, 2), (5120, 1152, 20), (6144, 4096, 150)])
def test_fused_decode_at_the_split_of_codes(tc, mq, N, K, nnzb):
    _check_fused_decode(tc, mq, N, K, nnzb)


def _check_fused_decode(tc, mq, N, K, nnzb):
    _, _, Wq, s_w, rowptr, kb, _, Rq, s_r = random_operands(1, N, K, nnzb, seed=N + K)
    pw = gpu_pw(tc, mq, N, K, Wq, s_w, rowptr, kb, Rq, s_r)
    rng = np.random.default_rng(K)
    for M in range(1, 9):
        x = (rng.standard_normal((M, K)) * 2.0 ** rng.integers(-10, 10, (M, 1))).astype(np.float16)
        if M > 2:
            x[1] = 0
            x[2] = rng.integers(-14, 15, K) / 2
            x[2, 0] = 7
        X = dev(tc, x)
        assert (mq.linear_workspace_bytes(M, N, K) == 0) == (M * K <= (32768 if M <= 4 else 24576 if N <= 4096 else 16384))
        Y = mq.linear(X, pw)
        Xq, s_x = mq.quantize_act(X)
        want = mq.fused_gemm(Xq, s_x, pw)
        tc.cuda.synchronize()
        assert tc.equal(Y, want), M
