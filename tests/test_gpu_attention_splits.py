"""GPU: key splits of the wide attention kernel.  Its merge takes the partial sums of a query tile in rounds of 2, 4, 8 or
twelve splits; a lone long sequence of a small model is cut into more.  Small caches of many sequences are not cut."""
import pytest

import s2d2_inputs as I
from paper_2603_25702_amd import Params
from tests import harness as H
from tests.test_gpu_parity import run_steps

pytestmark = pytest.mark.gpu


CFG = I.ModelCfg("splits", 2, 512, 8, 4, 128, 1536, 4096)


def attention_launches(run, step):
    """Attention launches of one more step, by the launch timer."""
    run.eng.s2d2_profile_start(4096)
    run.step(Params(step=step, seed=1234), advance=False)
    return run.eng.s2d2_profile_stop()["attention"]["launches"]


@pytest.mark.parametrize("lens", [
    [130, 385, 520, 1000, 1030],   # 2, 4, 5, 8 and 9 splits (runs of four tiles of 32 keys)
    [1536, 1537, 40],              # 12, 13 and one split
    [3100],                        # 25: three rounds, the last of one split
])
def test_every_round_of_the_merge(lens):
    case = H.make_case(CFG, len(lens), 16, lens, seed=27, synthetic_kv=True, page_size=16, room=96)
    # The values of the later keys lie around 2 instead of 0, those behind 24 splits around 60, so that the splits that hold
    # them carry weight (the oracle without the keys from 1536 / 3072 on: logits off by 6e-2 or more / 5e-2 of the largest).
    for n, S in enumerate(lens):
        for first, offset in ((min(1536, S // 2), 2.0), (3072, 60.0)):
            for page in case.page_table[n, first // 16:]:
                for l in range(CFG.n_layers):
                    case.v_pages[l][int(page)] += offset
    run, rep = run_steps(case, 2)
    print("splits:", lens, rep)
    assert rep.max_logit_err_draft <= H.LOGIT_RTOL and rep.max_logit_err_verify <= H.LOGIT_RTOL
    assert attention_launches(run, 2) == 2 * CFG.n_layers * 2   # the attention launch and the merge behind it, either forward


@pytest.mark.parametrize("N,tokens,merges", [(64, 576, 0), (64, 592, 1), (32, 224, 0), (32, 240, 1)])   # 18, 19, 7 and 8 tiles
def test_small_caches_of_many_sequences_are_not_cut(N, tokens, merges):
    lens = [tokens - 64 - 5 * (n % 7) for n in range(N)]
    case = H.make_case(CFG, N, 16, lens, seed=28, synthetic_kv=True, page_size=16, room=tokens - max(lens))
    run, rep = run_steps(case, 1, seqs=[0, N // 2 - 1, N - 1])
    assert rep.max_logit_err_draft <= H.LOGIT_RTOL and rep.max_logit_err_verify <= H.LOGIT_RTOL
    assert attention_launches(run, 1) == 2 * CFG.n_layers * (1 + merges)
