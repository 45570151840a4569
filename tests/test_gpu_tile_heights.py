"""The large tiled GEMM on tiles of 256, 192 and 128 rows with last tile rows of
every height, in one round and in several (where the short tiles come last):
int32 sums bit-exact, fp16 outputs within the bar, rows past M untouched."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import TIGHT, _announce, dev, dev_x, gpu_pw, host, maxabsrel, mq, orc_pw, random_operands, tc  # noqa: F401

pytestmark = pytest.mark.gpu

# 256-row tiles with 133, 36 and 100 rows left behind 224 full tiles; 192-row
# tiles with 102, 156 and 124 rows left; 128-row tiles, one row past a tile
CASES = [(1157, 14336, 256, 40), (1060, 14336, 128, 9), (1124, 14336, 128, 0), (1254, 14336, 128, 5),
         (1500, 8192, 384, 20), (700, 14336, 256, 30), (2049, 512, 512, 6), (257, 1024, 384, 4), (1, 256, 256, 1)]


@pytest.mark.parametrize("M,N,K,nnzb", CASES)
def test_tile_heights(tc, mq, orc, M, N, K, nnzb):
    _check_tiles(tc, mq, orc, M, N, K, nnzb)


# every height of a last tile row (sub-tile rows of 16 a wave, 1 .. 8; odd ones
# run the next even height's code) behind 256- and 192-row tiles
LAST_ROWS = [(449, 24576, 128, 12, 256, 7), (480, 28672, 256, 40, 256, 7), (481, 24576, 128, 3, 256, 8),
             (510, 24576, 256, 20, 256, 8), (385, 24576, 128, 9, 256, 5), (440, 24576, 128, 0, 256, 6),
             (850, 14336, 128, 11, 256, 3), (800, 24576, 128, 9, 192, 1), (620, 14336, 128, 5, 192, 2),
             (270, 24576, 256, 25, 192, 3), (320, 24576, 128, 6, 192, 4), (530, 14336, 128, 4, 192, 5),
             (570, 14336, 256, 14, 192, 6)]


@pytest.mark.parametrize("M,N,K,nnzb,height,last", LAST_ROWS)
def test_last_tile_rows(tc, mq, orc, M, N, K, nnzb, height, last):
    assert mq.tile(M, N, K, variant="tiled_large") == (height, 256)
    assert M > height and -(-(M % height) // 32) == last
    _check_tiles(tc, mq, orc, M, N, K, nnzb)


def _check_tiles(tc, mq, orc, M, N, K, nnzb):
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
