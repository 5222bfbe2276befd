"""GPU parity of gate / up of many rows through LDS: row tiles of 128, 192 and 256 rows, one row more and one less than they hold, feature tiles that do not
fill the last group, windows of fewer rows than expected (mid-block: the tiles shrink) and of more (carried tokens: the workgroups walk on)."""
import pytest

import s2d2_inputs as I
from paper_2603_25702_amd.binding import s2d2_gemm_choice
from tests import harness as H
from tests.test_gpu_parity import run_steps

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,d_ffn,N,B,steps", [
    (2048, 6144, 16, 20, 2), (2048, 6176, 11, 35, 1), (2048, 6144, 12, 32, 1), (2560, 6176, 8, 24, 2), (2048, 6144, 19, 27, 1), (4096, 12288, 4, 41, 2), (4096, 12320, 16, 32, 1),
])
def test_gate_up_of_many_rows(d, d_ffn, N, B, steps):
    cfg = I.ModelCfg("gateup-rows", 1, d, 8, 4, 128, d_ffn, 2048)
    assert "tile" in [s2d2_gemm_choice(cfg, f, N, B, "gateup")[0] for f in ("draft", "verify")]   # (through LDS)
    case = H.make_case(cfg, N, B, [20 + 13 * (i % 5) for i in range(N)], seed=59, synthetic_kv=True, page_size=16, room=4 * B + 16, norm_jitter=0.1)
    run, rep = run_steps(case, steps, seqs=sorted({0, N // 2, N - 1}))
    print("gate / up rows:", d, d_ffn, N, B, rep)
    assert rep.max_logit_err_draft <= H.LOGIT_RTOL and rep.max_logit_err_verify <= H.LOGIT_RTOL
