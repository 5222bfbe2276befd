"""GPU parity of gate / up of many rows through LDS: row tiles of 128, 192 and 256 rows, one row more than one or three of them hold (129, 385 rows: a last tile of
one row) and one less than four (767, 1023), feature tiles that do not fill the last group, the kernel that each forward runs, windows of fewer rows than expected (mid-block: the tiles shrink) and of more (carried tokens: the workgroups walk on)."""
import pytest

import s2d2_inputs as I
from paper_2603_25702_amd.binding import s2d2_gemm_choice
from tests import harness as H
from tests.test_gpu_parity import run_steps

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,d_ffn,N,B,steps,draft,verify", [
    (2048, 6144, 16, 20, 2, "lds", "tile"), (2048, 6176, 11, 35, 1, "tile", "lds"), (2048, 6144, 12, 32, 1, "lds", "lds"), (2560, 6176, 8, 24, 2, "block", "lds"),
    (2560, 9728, 3, 43, 2, "lds", "tile"), (2048, 6144, 7, 55, 1, "lds", "lds"), (2048, 6144, 13, 59, 1, "lds", "lds"), (2048, 6144, 31, 33, 1, "lds", "lds"),
    (4096, 12288, 4, 41, 2, "lds", "lds"), (4096, 12320, 16, 32, 1, "tile", "lds"),
    (768, 6144, 7, 55, 1, "tile", "lds"), (768, 6144, 13, 59, 2, "lds", "lds"), (1024, 4096, 41, 25, 1, "lds", "tile"), (1536, 4608, 31, 33, 1, "lds", "lds"),   # (the fewest steps, the smallest matrices)
])
def test_gate_up_of_many_rows(d, d_ffn, N, B, steps, draft, verify):
    cfg = I.ModelCfg("gateup-rows", 1, d, 8, 4, 128, d_ffn, 2048)
    assert [s2d2_gemm_choice(cfg, f, N, B, "gateup")[0] for f in ("draft", "verify")] == [draft, verify]
    case = H.make_case(cfg, N, B, [20 + 13 * (i % 5) for i in range(N)], seed=59, synthetic_kv=True, page_size=16, room=4 * B + 16, norm_jitter=0.1)
    run, rep = run_steps(case, steps, seqs=sorted({0, N // 2, N - 1}))
    print("gate / up rows:", d, d_ffn, N, B, rep)
    assert rep.max_logit_err_draft <= H.LOGIT_RTOL and rep.max_logit_err_verify <= H.LOGIT_RTOL


@pytest.mark.parametrize("cfg,N,B", [(I.ModelCfg("gateup-alone", 1, 4096, 32, 8, 128, 12288, 2048), 13, 32), (I.ModelCfg("gateup-alone", 1, 4096, 32, 8, 128, 12288, 2048), 16, 32)])
def test_gate_up_through_lds_between_tiled_matrices(cfg, N, B):
    kernels = [s2d2_gemm_choice(cfg, "verify", N, B, m)[0] for m in ("qkv", "o", "gateup", "down")]
    assert kernels == ["tile", "tile", "lds", "tile"]
    case = H.make_case(cfg, N, B, [20 + 13 * (i % 5) for i in range(N)], seed=61, synthetic_kv=True, page_size=16, room=4 * B + 16, norm_jitter=0.1)
    run, rep = run_steps(case, 1, seqs=sorted({0, N // 2, N - 1}))
    print("gate / up alone:", N, B, rep)
    assert rep.max_logit_err_draft <= H.LOGIT_RTOL and rep.max_logit_err_verify <= H.LOGIT_RTOL
