"""Split-K launches of the tiled kernel with CSR rows whose entries sit at the
edges of the splits, in one split only, in none and everywhere: int32 sums
bit-exact, fp16 outputs within the bar."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_util import TIGHT, _announce, dev, dev_x, gpu_pw, host, maxabsrel, mq, orc_pw, random_operands, tc  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K", [(100, 2048), (129, 4096), (64, 5248)])
def test_split_csr_rows(tc, mq, orc, M, K):
    N, G = 6 * 128, K // 128
    splits = mq.load().mq_fused_gemm_workspace_size(M, N, K) // (4 * M * N)
    assert splits > 1
    per = -(-G // splits)
    firsts = [g for g in range(0, G, per)]
    rows = [list(range(G)), firsts, sorted(set([g - 1 for g in firsts[1:]] + [G - 1])), [], list(range(per, min(2 * per, G))), [G - 1]]
    nnzb = sum(map(len, rows))
    Xq, s_x, Wq, s_w, _, _, _, Rq, s_r = random_operands(M, N, K, nnzb, seed=M + K)
    sel = np.zeros((6, G), bool)
    for r, cols in enumerate(rows):
        sel[r, cols] = True
    rowptr = np.concatenate([[0], np.cumsum(sel.sum(1))]).astype(np.int32)
    kb = np.nonzero(sel)[1].astype(np.int32)
    Tb_ref, Tr_ref, Y64 = orc.linear(Xq, s_x, orc_pw(orc, N, K, Wq, s_w, rowptr, kb, sel, Rq, s_r))
    pw = gpu_pw(tc, mq, N, K, Wq, s_w, rowptr, kb, Rq, s_r)
    Xd = dev_x(tc, Xq)
    Tb, Tr = mq.fused_gemm_acc_i32(Xd, pw, variant="tiled")
    assert np.array_equal(host(Tb), Tb_ref) and np.array_equal(host(Tr), Tr_ref)
    Y = mq.fused_gemm(Xd, dev(tc, s_x).view(tc.float16), pw, variant="tiled")
    assert maxabsrel(Y, Y64) <= TIGHT
