"""GPU parity of the GEMM for windows of more than 48 rows: every kernel of it that the full models' matrices or small ones get, one row
tile and several, row tiles that end in few rows, windows of fewer rows than expected (mid-block: the tiles shrink) and of more
(carried tokens: the workgroups walk on), feature tiles that do not divide into groups, K shared by two to four workgroups."""
import pytest

import s2d2_inputs as I
from paper_2603_25702_amd.binding import s2d2_gemm_choice
from tests import harness as H
from tests.test_gpu_parity import run_steps

pytestmark = pytest.mark.gpu


def blocks(cfg, forward, N, B):
    """The kernels of a layer (QKV, output, gate / up, down) by the library's choice: blocks as row blocks x feature tiles, / workgroups
    that share K, s for streaming weight loads."""
    out = []
    for matrix in ("qkv", "o", "gateup", "down"):
        kernel, rb, ta, shares, stream = s2d2_gemm_choice(cfg, forward, N, B, matrix)
        out.append(f"{rb}x{ta}" + (f"/{shares}" if shares > 1 else "") + "s" * stream if kernel == "block" else kernel)
    return " ".join(out)


@pytest.mark.parametrize("d,d_ffn,heads,N,B,steps,draft,verify", [
    (512, 1536, (8, 4), 7, 7, 4, "2x2s 2x2s 2x2s 2x2s", "2x2 2x2 4x2 2x2"),
    (512, 4096, (8, 4), 13, 5, 3, "2x2 2x2 4x4 2x2/4", "4x2 2x2 6x4 2x2/3"),
    (512, 6144, (8, 4), 3, 32, 2, "2x2 2x2 4x6 2x2/4", "4x2 2x2 6x6 4x2/4"),
    (640, 6144, (8, 4), 8, 24, 2, "4x2 2x2 6x6 4x2/3", "4x4 4x2 tile 4x3/2"),
    (640, 12288, (8, 4), 8, 24, 1, "4x2 2x2 tile 4x3/4", "4x4 4x2 8x4 4x6/4"),
    (512, 12288, (8, 4), 16, 24, 1, "4x4 2x2 8x4 4x4/4", "8x4 4x2 tile 4x4/2"),
    (512, 2080, (8, 4), 8, 24, 2, "4x2 2x2 4x4 tile", "4x4 2x2 8x4 tile"),
    (512, 2048, (8, 4), 8, 32, 2, "4x2 2x2 4x4 2x2", "4x4 2x2 8x4 2x2"),
    (512, 1536, (8, 4), 16, 24, 2, "4x4 2x2 4x6 2x2", "8x4 4x2 6x6 4x2"),
    (2048, 1536, (8, 4), 16, 24, 1, "4x4 4x4 4x6 4x4", "8x4 8x4 6x6 8x4"),
    (640, 19456, (8, 4), 16, 24, 1, "4x4 4x2 tile 4x6/4", "8x4 4x3 tile 8x6/4"),
    (512, 6144, (32, 8), 2, 25, 2, "4x2s 2x2/4s 4x4s 2x2/4s", "4x3 2x2/4 4x6 2x2/4"),
    (1024, 2048, (16, 8), 9, 29, 1, "4x6 4x2 4x6 4x2", "8x6 4x3 8x6 4x3"),
    (512, 12288, (8, 4), 2, 25, 1, "2x2s 2x2s 4x6s 2x2/4s", "2x2 2x2 8x6s 2x2/4"),
    (512, 9728, (8, 4), 2, 17, 2, "tile mid tile mid", "2x2 2x2 6x6s 2x2/4"),
    (640, 1536, (8, 4), 17, 31, 1, "4x6 4x2 8x4 4x2", "4x4 4x6 tile 4x6"),
    (1536, 6144, (8, 4), 1, 25, 2, "mid mid mid mid", "2x2s 2x2s 4x4s 4x2/4s"),
    (2048, 1536, (8, 4), 17, 31, 1, "4x6 4x6 8x4 4x6", "8x6 8x6 4x6 8x6"),
    (4096, 6144, (8, 4), 1, 25, 1, "mid mid mid mid", "2x2s 2x2s 4x6s 4x4/4s"),
])
def test_blocks(d, d_ffn, heads, N, B, steps, draft, verify):
    cfg = I.ModelCfg("block-rows", 2, d, heads[0], heads[1], 128, d_ffn, 2048)
    assert blocks(cfg, "draft", N, B) == draft and blocks(cfg, "verify", N, B) == verify
    case = H.make_case(cfg, N, B, [20 + 13 * (i % 5) for i in range(N)], seed=43, synthetic_kv=True, page_size=16, room=4 * B + 16, norm_jitter=0.1)
    run, rep = run_steps(case, steps, seqs=sorted({0, N // 2, N - 1}))
    print("block rows:", d, d_ffn, N, B, rep)
    assert rep.max_logit_err_draft <= H.LOGIT_RTOL and rep.max_logit_err_verify <= H.LOGIT_RTOL
