"""GPU: the narrow attention kernel behind short caches: ends of a tile, of a wavefront's tiles and of a split, against the oracle, and
sums that do not depend on the room a cache has."""
import pytest
import torch

import s2d2_inputs as I
from paper_2603_25702_amd import Params
from tests import harness as H
from tests.test_gpu_parity import run_steps

pytestmark = pytest.mark.gpu

CFG = I.ModelCfg("short-caches", 2, 512, 8, 4, 128, 1536, 4096)


@pytest.mark.parametrize("lens,act_planes,page_size", [
    ([1, 31, 32, 33, 255, 256, 257], 0, 16),   # no tile for most wavefronts; a second tile for one
    ([511, 513, 769, 1000], 1, 16),            # three and four tiles; single bf16 planes
    ([1016, 1024, 1025, 1200], 0, 8),          # four and five tiles, the line crossed while decoding
    ([40], 2, 24),                             # pages that are no power of two
])
def test_short_caches(lens, act_planes, page_size):
    case = H.make_case(CFG, len(lens), 4, lens, seed=31, synthetic_kv=True, page_size=page_size, room=96)
    # Values of the last keys lie around 2, so that a result without them is far off.
    for n, S in enumerate(lens):
        for page in case.page_table[n, (S // 2) // page_size:]:
            for l in range(CFG.n_layers):
                case.v_pages[l][int(page)] += 2.0
    run, rep = run_steps(case, 3, act_planes=act_planes, check_logits=act_planes != 1)
    print("short caches:", lens, rep)
    if act_planes != 1:   # (single bf16 planes are outside the tolerance by design)
        assert rep.max_logit_err_draft <= H.LOGIT_RTOL and rep.max_logit_err_verify <= H.LOGIT_RTOL


@pytest.mark.parametrize("lens,act_planes", [
    ([1, 33, 40, 129, 255, 256, 257], 0),   # two to four splits, most of them of the window alone or of nothing
    ([320, 511, 513, 600], 2),              # four splits, two and three cached tiles of a wavefront
    ([767, 769, 960, 992], 1),              # four tiles; a single plane
])
def test_room_of_the_cache_changes_no_bit(lens, act_planes):
    """The same pages under a page table for twice as many keys: equal logits of both forwards, equal keys and values of the window.
    (2048 and 4096 keys; either has as many splits as these lengths use.)"""
    case = H.make_case(CFG, len(lens), 4, lens, seed=32, synthetic_kv=True, page_size=16, room=96)
    got = []
    for pages in (128, 256):   # 2048 and 4096 keys
        run = H.DeviceRun(case, act_planes=act_planes)
        table = run.kv.page_table
        run.kv.page_table = torch.cat([table, table.new_zeros((len(lens), pages - table.shape[1]))], 1).contiguous()
        run.step(Params(seed=9), advance=False, append=False)
        torch.cuda.synchronize()
        rows = int(run.d.logit_row_of.max()) + 1
        got.append({"draft": run.d.logits[:rows].clone(), "verify": run.v.logits_ver[:rows].clone(),
                    "k": run.v.k_stage[:, :2 * rows].clone(), "v": run.v.v_stage[:, :2 * rows].clone()})
    for name, t in got[0].items():
        assert torch.equal(t, got[1][name]), name
