"""GPU: the fp32 attention behind pages of one key, of sizes that are no power of two and of those that are, against the oracle: caches that end inside a
page, at its end and behind it, and more keys than one round of the sums takes."""
import pytest

import s2d2_inputs as I
from tests import harness as H
from tests.test_gpu_parity import run_steps

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("page_size", [1, 12, 16, 64])
def test_page_sizes(page_size):
    lens = [1, 47, 48, 49, 191, 200, 420]
    case = H.make_case(I.CONFIGS[1].cfg, len(lens), 4, lens, seed=71, synthetic_kv=True, page_size=page_size, room=40)
    run, rep = run_steps(case, 2)
    print("pages:", page_size, rep)
    assert rep.max_logit_err_draft <= 2e-5 and rep.max_logit_err_verify <= 2e-5   # fp32 sums over up to 768 terms through two layers
