"""GPU: runs of the wide attention kernel that are lengthened so that a ragged batch's splits are all resident (16 KV heads: 32 of them), one that
cannot be (a cache without the room for longer runs in the page tables that a workgroup keeps), one that needs none, and several wavefronts of sequences."""
import pytest

import s2d2_inputs as I
from tests import harness as H
from tests.test_gpu_parity import run_steps

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,B", [
    ([811, 1055, 1250, 334, 444, 1122], 16),   # 35 splits in runs of 5 tiles, 29 in runs of 6
    ([849, 385, 327, 1165, 1053, 1137, 838], 16), ([629, 752, 1088, 423, 603, 424, 753, 1276], 16),
    ([683, 703, 1203, 503, 802], 16),          # 33 and 28
    ([1290, 1290, 1290, 1283, 1283], 16),      # 30
    ([900 + 7 * (n % 5) for n in range(31)] + [1100], 16), ([150 + 97 * (n % 7) for n in range(70)], 8),
])
def test_ragged_batches(lens, B):
    cfg = I.ModelCfg("runs", 1, 512, 32, 16, 128, 512, 2048)
    case = H.make_case(cfg, len(lens), B, lens, seed=61, synthetic_kv=True, page_size=16, room=4 * B + 16)
    run, rep = run_steps(case, 1, seqs=sorted({0, len(lens) // 2, len(lens) - 1}))
    print("runs:", lens[:8], rep)
    assert rep.max_logit_err_draft <= H.LOGIT_RTOL and rep.max_logit_err_verify <= H.LOGIT_RTOL
