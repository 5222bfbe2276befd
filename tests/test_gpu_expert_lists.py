"""GPU: the experts that have a row are shared out evenly among the XCDs, however few rows each has and however many experts have none."""
import pytest
import torch

import s2d2_inputs as I
from paper_2603_25702_amd import Params
from tests import harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("experts,top_k,N,B", [(64, 8, 1, 1), (64, 8, 3, 3), (64, 8, 2, 8), (64, 4, 1, 15), (256, 3, 1, 2), (256, 8, 5, 4), (60, 5, 2, 7)])
def test_experts_with_rows_are_spread(experts, top_k, N, B):
    cfg = I.ModelCfg("expert-lists", 3, 256, 4, 2, 128, 0, 2048, n_experts=experts, top_k=top_k, d_expert=64)
    case = H.make_case(cfg, N, B, [40 + 31 * n for n in range(N)], seed=83, synthetic_kv=True, page_size=16, room=4 * B + 16)
    run, prm = H.DeviceRun(case), Params(seed=5)
    for forward, rows in (("draft", N * B), ("verify", 2 * N * B)):   # (fresh blocks)
        if forward == "draft":
            run.eng.s2d2_draft(run.kv, run.st, N, B, prm, run.d)
        else:
            run.eng.s2d2_verify(run.kv, run.st, N, B, prm, run.d, run.v)
        with_rows = torch.bincount(run.eng.s2d2_moe_choices(rows)[-1].flatten().long(), minlength=experts).gt(0).sum().item()
        at = run.eng.s2d2_debug_buffer("moe_tiles") - run.eng.workspace.data_ptr()
        tiles = run.eng.workspace[at:at + 32].view(torch.int32).tolist()
        assert sum(tiles) == with_rows and max(tiles) - min(tiles) <= 1, (forward, with_rows, tiles)   # (an expert has at most 40 rows: one tile)
