"""GPU parity of the expert GEMMs at the edges of their row tiles: all experts chosen by every row, so that each has all of them (draft N B, verifier
twice that): tiles of 64, 128, 192 and 256 rows, one row more and one less, several tiles an expert; features that do not fill a
group of 128 and groups that do not divide into the slices of few experts; an expert width whose K is no multiple of 64 (the tiled kernel's); more experts than one XCD has lists for, most without a row."""
import pytest
import torch

import s2d2_inputs as I
from paper_2603_25702_amd import Params
from tests import harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("experts,top_k,d,d_expert,N,B", [
    (2, 2, 256, 64, 1, 1), (2, 2, 256, 64, 1, 31), (2, 2, 256, 8256, 4, 16), (2, 2, 256, 8192, 5, 13), (2, 2, 256, 8192, 3, 43), (2, 2, 256, 8192, 12, 16), (2, 2, 256, 8512, 1, 64),
    (2, 2, 256, 8192, 4, 64), (2, 2, 256, 8192, 9, 29), (2, 2, 256, 8224, 3, 43), (256, 2, 256, 64, 2, 9), (3, 1, 256, 5504, 7, 37), (2, 2, 256, 64, 3, 43),
    (2, 1, 1024, 8256, 1, 3), (2, 2, 1024, 8256, 9, 29), (8, 2, 1024, 2112, 1, 1), (8, 2, 1088, 2112, 11, 29), (15, 3, 512, 1152, 5, 13),   # (slices of the features: four and two, groups that do not divide into them)
])
def test_rows_of_an_expert(experts, top_k, d, d_expert, N, B):
    cfg = I.ModelCfg("expert-rows", 2, d, 4, 2, 128, 0, 2048, n_experts=experts, top_k=top_k, d_expert=d_expert)
    case = H.make_case(cfg, N, B, [20 + 13 * (n % 5) for n in range(N)], seed=47, synthetic_kv=True, page_size=16, room=4 * B + 16)
    run, rep, prm = H.DeviceRun(case), H.Report(), Params(seed=99)
    run.step(prm, advance=False)
    case.W = H.LazyF64Weights(case.W)
    H.check_step(case, run, run.fetch(), prm, rep=rep, seqs=sorted({0, N // 2, N - 1}), free_router=experts > 3)
    print("expert rows:", experts, d_expert, N, B, rep)
    assert rep.max_logit_err_draft <= H.LOGIT_RTOL and rep.max_logit_err_verify <= H.LOGIT_RTOL
    # the kernel that ran, by its tiles: of up to 256 rows an expert through LDS, of 128 in the tiled one (K that is no multiple of 64; few experts of small matrices)
    rows = torch.bincount(run.choices_verify[-1][:2 * N * B].flatten().long(), minlength=experts)
    tiles = [int(((rows + most - 1) // most).sum()) for most in (128, 256)]
    at = run.eng.s2d2_debug_buffer("moe_tiles") - run.eng.workspace.data_ptr()
    got = run.eng.workspace[at:at + 32].view(torch.int32).tolist()
    few = experts * ((d_expert + 127) // 128) < 128 and 2 * N * B * top_k >= 64 * experts
    if d_expert % 64 or few:
        assert got[0] == tiles[0]
    else:
        assert sum(got) == tiles[1]


def test_few_experts_are_sliced_over_all_xcds():
    """Two lists of up to four experts each, a quarter of the features of a list to each of four XCDs: one row's two experts keep all eight busy."""
    cfg = I.ModelCfg("expert-slices", 1, 1024, 4, 2, 128, 0, 2048, n_experts=8, top_k=2, d_expert=2048)
    case = H.make_case(cfg, 1, 1, [40], seed=47, synthetic_kv=True, page_size=16, room=20)
    run = H.DeviceRun(case)
    run.eng.s2d2_draft(run.kv, run.st, 1, 1, Params(seed=1), run.d)
    at = run.eng.s2d2_debug_buffer("moe_tiles") - run.eng.workspace.data_ptr()
    assert run.eng.workspace[at:at + 32].view(torch.int32).tolist() == [1, 1, 0, 0, 0, 0, 0, 0]
