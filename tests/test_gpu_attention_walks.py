"""GPU: the walks of the wide attention kernel over pages of 8, 32 and 64 tokens (four pages to a tile, one, and half a one; other tests
have pages of 16).  Eight wavefronts: four that fetch for four in short splits, two key groups in splits of more than 24 tiles of 32 keys,
one group where more than half of the wavefronts have query rows.  Four wavefronts: plain loads in splits of up to 8 tiles of launches of
more than 256 workgroups, else streaming loads."""
import pytest
import torch

import s2d2_inputs as I
from paper_2603_25702_amd import Params
from tests import harness as H
from tests.test_gpu_parity import run_steps

pytestmark = pytest.mark.gpu

# Rounding leaves 5.4e-4 of the largest logit here or less (half operands; two bf16 planes 3.3e-4).  In the oracle, one tile of the longest
# case left out moves the logits by 2.3e-3 or more, its values with the halves of the head dimension exchanged by 2.9e-3, all of them
# exchanged by 3.8e-2.
RTOL = 1.5e-3
CFG = I.ModelCfg("walks", 2, 512, 32, 16, 128, 1536, 2048)   # 16 KV heads: 16 splits fill the chip, so two sequences of 200 tiles have splits of 25 and 26


@pytest.mark.parametrize("B,lens", [
    (32, [130, 333]),      # 64 verifier rows x 2 heads: four query tiles of six; two and three splits of two to four tiles
    (32, [6490, 6420]),    # 203 and 201 tiles: splits of 26 and 25, of 25 and 26, the last one with the window's two tiles
    (33, [333, 95]),       # five query tiles of seven
    (33, [3251, 41]),      # 102 tiles in splits of 6 or 7, and one split
    (16, [130, 333]),      # three query tiles, four wavefronts; four splits of 16 heads: streaming loads
    (16, [1303, 1010]),    # 41 and 32 tiles in splits of four: 304 workgroups, plain loads
    (16, [6490, 6420]),    # 32 splits of 12 and 13 tiles
])
@pytest.mark.parametrize("page_size,act_planes", [(8, 0), (32, 2), (64, 0)])
def test_walks(B, lens, page_size, act_planes):
    case = H.make_case(CFG, len(lens), B, lens, seed=37, synthetic_kv=True, page_size=page_size, room=96 + 2 * B)
    # Values of the last tiles, of the last page and of every other page between lie around other numbers than the rest.
    for n, S in enumerate(lens):
        used = case.page_table[n, :(S + page_size - 1) // page_size]
        for l in range(CFG.n_layers):
            for at, offset in ((used[::2], 0.5), (used[-max(1, 64 // page_size):], 1.0), (used[-1:], 2.0)):
                for page in at:
                    case.v_pages[l][int(page)] += offset
    run, rep = run_steps(case, 1, act_planes=act_planes)
    print("walks:", B, lens, page_size, act_planes, rep)
    assert rep.max_logit_err_draft <= RTOL and rep.max_logit_err_verify <= RTOL


@pytest.mark.parametrize("pages,B", [
    (25000, 32),   # 100 KB of page table: no LDS for the tiles of two key groups; a split of 31 tiles per sequence
    (40000, 32),   # 160 KB: twice as many splits
])
def test_long_page_tables(pages, B):
    """Caches with room for 200 000 tokens and more in pages of 8: still the wide kernel and its merge, two launches per layer and
    forward (the narrow kernel is one)."""
    lens = [900 + n for n in range(16)]
    case = H.make_case(CFG, len(lens), B, lens, seed=38, synthetic_kv=True, page_size=8, room=96 + 2 * B)
    run = H.DeviceRun(case)
    table = run.kv.page_table
    run.kv.page_table = torch.cat([table, table.new_zeros((len(lens), pages - table.shape[1]))], 1).contiguous()
    run.eng.s2d2_profile_start(4096)
    run.step(Params(seed=1234), advance=False)
    assert run.eng.s2d2_profile_stop()["attention"]["launches"] == 2 * CFG.n_layers * 2
    rep = H.check_step(case, run, run.fetch(), Params(seed=1234), seqs=[0, 7, 15])
    assert rep.max_logit_err_draft <= RTOL and rep.max_logit_err_verify <= RTOL
