"""GPU parity of the GEMMs for windows of 17 to 256 rows (the mid-size kernel up to 48 of a layer's rows and 64 logit rows, then blocks and
tiles) at the edges of row counts: row blocks of 16 that are full and that hold one row, one and two passes over the rows (windows that
carry more rows than a fresh block gives), K shared by several workgroups, feature tiles that do not divide into groups, and a K the
batches do not divide (the tiled kernel takes that one matrix)."""
import pytest

import s2d2_inputs as I
from tests import harness as H
from tests.test_gpu_parity import run_steps

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,B,d_ffn,vocab,steps", [
    (1, 17, 1536, 32000, 2),    # 17 draft rows, 34 verifier rows
    (2, 24, 4096, 32007, 2),    # 48 / 96 rows, long K of the down projection, vocabulary that ends inside a tile
    (13, 5, 1568, 32000, 4),    # 65 / 130 rows, 98 feature tiles, 49 K tiles
    (4, 32, 1536, 32000, 2),    # 128 / 256 rows
])
def test_windows_between_the_streaming_and_the_tiled_kernel(N, B, d_ffn, vocab, steps):
    cfg = I.ModelCfg("mid-rows", 2, 1024, 8, 4, 128, d_ffn, vocab)
    case = H.make_case(cfg, N, B, [20 + 13 * (i % 5) for i in range(N)], seed=41, synthetic_kv=True, page_size=16, room=4 * B + 16, norm_jitter=0.1)
    run, rep = run_steps(case, steps)
    print("mid rows:", N, B, rep)
    assert rep.max_logit_err_draft <= H.LOGIT_RTOL and rep.max_logit_err_verify <= H.LOGIT_RTOL
