"""The W4A8 layer on the tiled kernel (128 x 256 tiles): shapes at which the
launch takes it, with ragged last tiles, one and several groups, no and many
residual blocks, and rows of Y off the 16-byte alignment its wide stores need,
against the CPU oracle: int32 sums bit-exact, fp16 outputs within the bar."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import TIGHT, _announce, dev, gpu_pw, host, maxabsrel, mq, orc_pw, random_operands, tc  # noqa: F401

pytestmark = pytest.mark.gpu

# rows in the last tile: 5, 1, 60, 128; K of one group, two, three (the ring), five
CASES = [(1157, 2048, 384, 9, 0), (2049, 1024, 128, 3, 0), (700, 3328, 256, 0, 0), (1152, 2048, 640, 80, 0),
         (1157, 2048, 384, 9, 1)]


@pytest.mark.parametrize("M,N,K,nnzb,off", CASES)
def test_a8_tiled_parity(tc, mq, orc, M, N, K, nnzb, off):
    assert mq.a8_tile(M, N, K) == (128, 256)
    _, s_x, Wq, s_w, rowptr, kb, sel, Rq, s_r = random_operands(M, N, K, nnzb, seed=M + N + K)
    codes = np.random.default_rng(M * 3 + N).integers(-127, 128, (M, K)).astype(np.int8)
    Tb_ref, Tr_ref, Y64 = orc.linear_a8(codes, s_x, orc_pw(orc, N, K, Wq, s_w, rowptr, kb, sel, Rq, s_r))
    pw = gpu_pw(tc, mq, N, K, Wq, s_w, rowptr, kb, Rq, s_r)
    Xq8 = mq.repack_act8(dev(tc, codes))
    Tb, Tr = mq.fused_gemm_a8_acc_i32(Xq8, pw)
    assert np.array_equal(host(Tb), Tb_ref) and np.array_equal(host(Tr), Tr_ref)
    sx = dev(tc, s_x).view(tc.float16)
    # the rows past M and the bytes around Y stay as they were
    buf = tc.full((off + M * N + 4096,), 7.0, dtype=tc.float16, device="cuda")
    p = lambda t: t.data_ptr() if t.numel() else None
    st = mq.load().mq_fused_gemm_a8(M, N, K, p(Xq8), p(sx), p(pw.Wq), p(pw.s_w), p(pw.rowptr) if nnzb else None,
                                    p(pw.kb) if nnzb else None, nnzb, p(pw.Rq) if nnzb else None,
                                    p(pw.s_r) if nnzb else None, buf.data_ptr() + 2 * off, N, None)
    tc.cuda.synchronize()
    assert st == 0
    assert maxabsrel(buf[off:off + M * N].view(M, N), Y64) <= TIGHT
    assert bool((buf[:off] == 7).all()) and bool((buf[off + M * N:] == 7).all())
