"""GPU parity of the blocks of six row blocks of 16 (6 x 4 and 6 x 8 units), by the library's choice: full tiles, a last tile of few rows,
fewer rows than expected in later steps (the tiles shrink), down projections of few K tiles that keep the other shapes."""
import pytest

import s2d2_inputs as I
from tests import harness as H
from tests.test_gpu_block_rows import blocks
from tests.test_gpu_parity import run_steps

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,d_ffn,N,B,steps,draft,verify", [
    (2048, 1536, 16, 24, 1, "8x4 4x4 4x6 4x4", "6x8 6x4 6x6 8x4"),
    (2048, 1536, 15, 25, 2, "8x4 4x4 4x6 4x4", "6x8 6x4 6x6 8x4"),
    (4096, 2048, 11, 31, 2, "8x4 6x4 6x4 6x4", "6x8 6x8 6x4 6x8"),
])
def test_six_row_blocks(d, d_ffn, N, B, steps, draft, verify):
    cfg = I.ModelCfg("block-six-rows", 2, d, 16, 8, 128, d_ffn, 2048)
    assert blocks(cfg, "draft", N, B) == draft and blocks(cfg, "verify", N, B) == verify
    case = H.make_case(cfg, N, B, [20 + 13 * (i % 5) for i in range(N)], seed=47, synthetic_kv=True, page_size=16, room=4 * B + 16, norm_jitter=0.1)
    run, rep = run_steps(case, steps, seqs=sorted({0, N // 2, N - 1}))
    print("six row blocks:", d, d_ffn, N, B, rep)
    assert rep.max_logit_err_draft <= H.LOGIT_RTOL and rep.max_logit_err_verify <= H.LOGIT_RTOL


@pytest.mark.parametrize("N,B,draft,verify", [(12, 31, "4x4 4x3 4x6 4x3", "8x4 6x4 8x6 6x4"), (24, 32, "8x4 6x4 8x6 6x4", "8x4 6x8 tile 6x8")])
def test_six_row_blocks_of_the_fewest_columns(N, B, draft, verify):
    cfg = I.ModelCfg("block-six-rows", 2, 1792, 14, 2, 128, 1792, 2048)   # 56 K tiles
    assert blocks(cfg, "draft", N, B) == draft and blocks(cfg, "verify", N, B) == verify
    case = H.make_case(cfg, N, B, [20 + 13 * (i % 5) for i in range(N)], seed=47, synthetic_kv=True, page_size=16, room=4 * B + 16, norm_jitter=0.1)
    run, rep = run_steps(case, 2, seqs=sorted({0, N // 2, N - 1}))
    print("six row blocks, 56 K tiles:", N, B, rep)
    assert rep.max_logit_err_draft <= H.LOGIT_RTOL and rep.max_logit_err_verify <= H.LOGIT_RTOL
