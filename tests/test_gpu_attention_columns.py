"""GPU: caches of up to 1024 keys with one query tile go by output columns (no merge through memory), longer ones of the same
batch by key splits: ends of a tile, of a wavefront's tiles and of the line between the two, against the oracle."""
import pytest

import s2d2_inputs as I
from tests import harness as H
from tests.test_gpu_parity import run_steps

pytestmark = pytest.mark.gpu

CFG = I.ModelCfg("columns", 2, 512, 8, 4, 128, 1536, 4096)


@pytest.mark.parametrize("lens,act_planes,page_size", [
    ([1, 31, 32, 33, 255, 256, 257], 0, 16),   # no tile for most wavefronts; a second tile for one
    ([511, 513, 769, 1000], 1, 16),            # three and four tiles; single bf16 planes
    ([1016, 1024, 1025, 1200], 0, 8),          # both sides of the line, crossed while decoding
    ([40], 2, 24),                             # pages that are no power of two
])
def test_short_caches_by_columns(lens, act_planes, page_size):
    case = H.make_case(CFG, len(lens), 4, lens, seed=31, synthetic_kv=True, page_size=page_size, room=96)
    # Values of the last keys lie around 2, so that a result without them is far off.
    for n, S in enumerate(lens):
        for page in case.page_table[n, (S // 2) // page_size:]:
            for l in range(CFG.n_layers):
                case.v_pages[l][int(page)] += 2.0
    run, rep = run_steps(case, 3, act_planes=act_planes, check_logits=act_planes != 1)
    print("columns:", lens, rep)
    if act_planes != 1:   # (single bf16 planes are outside the tolerance by design)
        assert rep.max_logit_err_draft <= H.LOGIT_RTOL and rep.max_logit_err_verify <= H.LOGIT_RTOL
