"""GPU parity of the expert GEMMs at the edges of their row tiles: all experts chosen by every row, so that each has all of them (draft N B, verifier
twice that): tiles of 64, 128, 192 and 256 rows, one row more and one less, several tiles an expert; features that do not fill a
group of 128; an expert width whose K is no multiple of 64 (the tiled kernel's); more experts than one XCD has lists for, most without a row."""
import pytest

import s2d2_inputs as I
from paper_2603_25702_amd import Params
from tests import harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("experts,top_k,d_expert,N,B", [
    (2, 2, 64, 1, 1), (2, 2, 64, 1, 31), (2, 2, 192, 4, 16), (2, 2, 64, 5, 13), (2, 2, 128, 3, 43), (2, 2, 64, 12, 16), (2, 2, 320, 1, 64),
    (2, 2, 64, 4, 64), (2, 2, 64, 9, 29), (2, 2, 96, 3, 43), (256, 2, 64, 2, 9), (3, 1, 64, 7, 37),
])
def test_rows_of_an_expert(experts, top_k, d_expert, N, B):
    cfg = I.ModelCfg("expert-rows", 2, 256, 4, 2, 128, 0, 2048, n_experts=experts, top_k=top_k, d_expert=d_expert)
    case = H.make_case(cfg, N, B, [20 + 13 * (n % 5) for n in range(N)], seed=47, synthetic_kv=True, page_size=16, room=4 * B + 16)
    run, rep, prm = H.DeviceRun(case), H.Report(), Params(seed=99)
    run.step(prm, advance=False)
    H.check_step(case, run, run.fetch(), prm, rep=rep, seqs=sorted({0, N // 2, N - 1}), free_router=True)
    print("expert rows:", experts, d_expert, N, B, rep)
    assert rep.max_logit_err_draft <= H.LOGIT_RTOL and rep.max_logit_err_verify <= H.LOGIT_RTOL
