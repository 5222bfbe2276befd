"""GPU: query tiles of a window over workgroups by the rows that are expected: 5 to 8 tiles with rows in room for 8 to 12, windows with fewer rows than expected
in later steps, against the oracle."""
import pytest

import s2d2_inputs as I
from tests import harness as H
from tests.test_gpu_parity import run_steps

pytestmark = pytest.mark.gpu

CFG = I.ModelCfg("attention-groups", 2, 512, 16, 4, 128, 1536, 2048)


@pytest.mark.parametrize("B,lens", [(20, [300, 33, 257]), (24, [260, 500]), (27, [31, 640, 96]), (32, [200, 513])])   # 40, 48, 54, 64 rows of four heads each
def test_groups(B, lens):
    case = H.make_case(CFG, len(lens), B, lens, seed=73, synthetic_kv=True, page_size=16, room=4 * B + 16)
    run, rep = run_steps(case, 3)
    print("groups:", B, lens, rep)
    assert rep.max_logit_err_draft <= H.LOGIT_RTOL and rep.max_logit_err_verify <= H.LOGIT_RTOL
