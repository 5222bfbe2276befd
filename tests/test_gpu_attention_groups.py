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


@pytest.mark.parametrize("B,lens", [
    (24, [300 + 41 * (n % 5) for n in range(17)]),                # verification: 6 tiles in room for 9 make 3 groups of 3, 2 of them with rows: 136 workgroups of four wavefronts
    (32, [33 + 190 * (n % 4) for n in range(16)] + [1100]),       # 8 in room for 12, 3 groups of 4
    (28, [640] * 30 + [31, 97, 5]),                               # 7 in room for 11, 3 groups of 4, more sequences than a wavefront's half
])
def test_groups_of_four_wavefronts(B, lens):
    """More than 128 workgroups ahead of the key splits and several groups of query tiles: workgroups of four wavefronts, the last group with
    rows in part or without any."""
    case = H.make_case(CFG, len(lens), B, lens, seed=79, synthetic_kv=True, page_size=16, room=4 * B + 16)
    run, rep = run_steps(case, 3, seqs=sorted({0, len(lens) // 2, len(lens) - 1}))
    print("groups of four wavefronts:", B, lens[:5], rep)
    assert rep.max_logit_err_draft <= H.LOGIT_RTOL and rep.max_logit_err_verify <= H.LOGIT_RTOL
