"""GPU: key splits of the wide attention kernel.  Its merge takes the partial sums of a query tile in rounds of twelve
splits; a lone long sequence of a small model is cut into more."""
import pytest

import s2d2_inputs as I
from paper_2603_25702_amd import Params
from tests import harness as H
from tests.test_gpu_parity import run_steps

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens", [
    [1536, 1537, 40],     # 12, 13 and one split (runs of four tiles of 32 keys)
    [3100],               # 25: three rounds, the last of one split
])
def test_more_splits_than_a_round_of_the_merge(lens):
    cfg = I.ModelCfg("splits", 2, 512, 8, 4, 128, 1536, 4096)
    case = H.make_case(cfg, len(lens), 16, lens, seed=27, synthetic_kv=True, page_size=16, room=96)
    # The values of the keys behind the first twelve splits lie around 2 instead of 0, those behind 24 around 60, so that the
    # few of them carry weight (the oracle without the keys from 1536 / 3072 on: logits off by 6e-2 or more / 5e-2 of the largest).
    for n, S in enumerate(lens):
        for first, offset in ((1536, 2.0), (3072, 60.0)):
            for page in case.page_table[n, first // 16:]:
                for l in range(cfg.n_layers):
                    case.v_pages[l][int(page)] += offset
    run, rep = run_steps(case, 2)
    print("splits:", lens, rep)
    assert rep.max_logit_err_draft <= H.LOGIT_RTOL and rep.max_logit_err_verify <= H.LOGIT_RTOL
    # the launch timer books the attention launch and the merge behind it, of either forward and each layer
    run.eng.s2d2_profile_start(4096)
    run.step(Params(step=2, seed=1234), advance=False)
    prof = run.eng.s2d2_profile_stop()
    assert prof["attention"]["launches"] == 2 * cfg.n_layers * 2
