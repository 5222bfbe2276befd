"""GPU: expert choices over one tile of experts, part of one, more than 64 experts (several a lane), the most there are; rows that
fill a block of sixteen and that do not; every operand mode; short K."""
import pytest

import s2d2_inputs as I
from paper_2603_25702_amd import Params
from tests import harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("experts,top_k,d,act_planes,N,B", [
    (16, 4, 512, 0, 1, 4), (8, 2, 256, 2, 3, 8), (60, 5, 512, 0, 2, 16), (80, 3, 512, 2, 1, 9), (256, 8, 256, 0, 1, 4),
])
def test_choices_of_the_router(experts, top_k, d, act_planes, N, B):
    cfg = I.ModelCfg("router", 2, d, d // 64, 2, 128, 0, 4096, n_experts=experts, top_k=top_k, d_expert=128)
    case = H.make_case(cfg, N, B, [40 + 13 * n for n in range(N)], seed=41, synthetic_kv=True, page_size=16, room=96)
    run, rep, prm = H.DeviceRun(case, act_planes=act_planes), H.Report(), Params(seed=1234)
    run.step(prm, advance=False)
    H.check_step(case, run, run.fetch(), prm, rep=rep, free_router=True)
    print("router:", rep)
    assert rep.max_logit_err_draft <= H.LOGIT_RTOL and rep.max_logit_err_verify <= H.LOGIT_RTOL
    assert rep.router_agree >= 0.9 * rep.router_rows > 0   # (a row whose last expert is tied to rounding takes another one now and then)
