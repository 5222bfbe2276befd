"""GPU parity of the GEMM for windows of more than 48 rows: every block shape that small matrices get, one row tile and
several, row tiles that end in few rows, windows of fewer rows than expected (mid-block: the tiles shrink) and of more
(carried tokens: the workgroups walk on), feature tiles that do not divide into groups, K shared by two to four workgroups.
(The shapes of the 4B and 8B matrices: the full configurations.)"""
import pytest

import s2d2_inputs as I
from tests import harness as H
from tests.test_gpu_parity import run_steps

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,d_ffn,N,B,steps", [
    (512, 1536, 7, 7, 4),      # 49 / 98 rows: blocks of 2 x 2 and 4 x 2
    (512, 4096, 13, 5, 3),     # 65 / 130 rows: 2 x 2 with K shared by three, gate / up 4 x 4
    (512, 6144, 3, 32, 2),     # 96 / 192 rows: 4 x 2 with K shared by four
    (640, 6144, 8, 24, 2),     # 192 / 384 rows, 40 feature tiles: 4 x 3 with K shared by two
    (640, 12288, 8, 24, 1),    # 4 x 6 with K shared by four, gate / up 8 x 6
    (512, 12288, 16, 24, 1),   # 384 / 768 rows: 4 x 4 with K shared by two
    (512, 2080, 8, 24, 2),     # gate / up 6 x 4; 65 K tiles of the down projection (the tiled kernel)
    (512, 2048, 8, 32, 2),     # gate / up 8 x 4
    (512, 1536, 16, 24, 2),    # gate / up 6 x 6, QKV 8 x 4
    (2048, 1536, 16, 24, 1),   # output and down 8 x 4
    (640, 19456, 16, 24, 1),   # 8 x 6 with K shared by four
])
def test_blocks(d, d_ffn, N, B, steps):
    cfg = I.ModelCfg("block-rows", 2, d, 8, 4, 128, d_ffn, 2048)
    case = H.make_case(cfg, N, B, [20 + 13 * (i % 5) for i in range(N)], seed=43, synthetic_kv=True, page_size=16, room=4 * B + 16, norm_jitter=0.1)
    run, rep = run_steps(case, steps, seqs=sorted({0, N // 2, N - 1}))
    print("block rows:", d, d_ffn, N, B, rep)
    assert rep.max_logit_err_draft <= H.LOGIT_RTOL and rep.max_logit_err_verify <= H.LOGIT_RTOL
