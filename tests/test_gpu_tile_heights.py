"""The large tiled GEMM on tiles of 256, 192 and 128 rows with last tile rows of
every height, in one round and in several (where the short tiles come last):
int32 sums bit-exact, fp16 outputs within the bar, rows past M untouched."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import TIGHT, _announce, dev, dev_x, gpu_pw, host, maxabsrel, mq, orc_pw, random_operands, tc  # noqa: F401

pytestmark = pytest.mark.gpu

# last tile rows of 133, 36, 100 and 230 rows behind 224 full tiles; 192-row
# tiles with 156 and 124 rows left; 128-row tiles; one row past a tile
CASES = [(1157, 14336, 256, 40), (1060, 14336, 128, 9), (1124, 14336, 128, 0), (1254, 14336, 128, 5),
         (1500, 8192, 384, 20), (700, 14336, 256, 30), (2049, 512, 512, 6), (257, 1024, 384, 4), (1, 256, 256, 1)]


@pytest.mark.parametrize("M,N,K,nnzb", CASES)
def test_tile_heights(tc, mq, orc, M, N, K, nnzb):
    Xq, s_x, Wq, s_w, rowptr, kb, sel, Rq, s_r = random_operands(M, N, K, nnzb, seed=M + 3 * N + K)
    Tb_ref, Tr_ref, Y64 = orc.linear(Xq, s_x, orc_pw(orc, N, K, Wq, s_w, rowptr, kb, sel, Rq, s_r))
    pw = gpu_pw(tc, mq, N, K, Wq, s_w, rowptr, kb, Rq, s_r)
    Xq_d, sx_d = dev_x(tc, Xq), dev(tc, s_x).view(tc.float16)
    Tb, Tr = mq.fused_gemm_acc_i32(Xq_d, pw, variant="tiled_large")
    assert np.array_equal(host(Tb), Tb_ref) and np.array_equal(host(Tr), Tr_ref)
    buf = tc.full((M + 300, N), 7.0, dtype=tc.float16, device="cuda")
    mq.fused_gemm(Xq_d, sx_d, pw, variant="tiled_large", out=buf[:M])
    tc.cuda.synchronize()
    assert maxabsrel(buf[:M], Y64) <= TIGHT
    assert bool((buf[M:] == 7).all())
