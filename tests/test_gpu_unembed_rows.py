"""GPU parity of the unembedding of more than 16 rows: the edges of its row tiles (64, 128, 192, 256 rows, one more and one less, several tiles), fewer
feature tiles than workgroups, ranges of one group of 16 and of several with a part of one, a vocabulary that is no multiple of 16,
rows and fragment order; vocabularies too small for it, and a width whose K is no multiple of 64 (the other kernels')."""
import pytest

import s2d2_inputs as I
from paper_2603_25702_amd import Params
from paper_2603_25702_amd.binding import s2d2_gemm_choice
from tests import harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,vocab,N,B,kernel", [
    (512, 28673, 1, 17, "lds"), (512, 70007, 1, 64, "lds"), (512, 2041, 5, 13, "lds"), (512, 4096, 8, 16, "lds"), (512, 2048, 3, 43, "lds"), (256, 70007, 3, 64, "lds"),
    (256, 2048, 3, 64, "lds"), (512, 40007, 4, 64, "lds"), (512, 70007, 9, 29, "lds"), (256, 20483, 11, 47, "lds"), (576, 28680, 2, 9, "lds"), (1024, 24583, 2, 24, "lds"),
    (512, 2048, 1, 17, "stream"), (1024, 8199, 2, 24, "mid"), (1024, 2041, 1, 64, "mid"), (256, 2048, 1, 64, "tile"), (512, 2041, 4, 64, "tile"), (288, 2048, 3, 43, "tile"),   # (small vocabularies, columns)
])
def test_rows_of_the_unembedding(d, vocab, N, B, kernel):
    cfg = I.ModelCfg("unembed-rows", 1, d, 8, 4, 128, 512, vocab)
    for forward in ("draft", "verify"):
        assert s2d2_gemm_choice(cfg, forward, N, B, "unembed")[0] == kernel
    case = H.make_case(cfg, N, B, [20 + 13 * (n % 5) for n in range(N)], seed=53, synthetic_kv=True, page_size=16, room=4 * B + 16)
    run, rep, prm = H.DeviceRun(case), H.Report(), Params(seed=77)
    run.step(prm, advance=False)
    H.check_step(case, run, run.fetch(), prm, rep=rep, seqs=sorted({0, N // 2, N - 1}))
    print("unembedding rows:", d, vocab, N, B, rep)
    assert rep.max_logit_err_draft <= H.LOGIT_RTOL and rep.max_logit_err_verify <= H.LOGIT_RTOL
