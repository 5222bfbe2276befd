"""GPU: the cache append stores key-minor V in pieces of 16 bytes: rows that begin and end inside a piece, fill it, cross pages;
pages that cut a piece; sequences without rows and without room.  Every byte outside the rows stays what it was."""
import pytest
import torch

import s2d2_inputs as I
from paper_2603_25702_amd.runner import Session

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,page_size", [("bf16", 16), ("bf16", 24), ("bf16", 12), ("f32", 16), ("f32", 4), ("f32", 6)])
def test_rows_land_in_their_places(dtype, page_size):
    cfg = I.ModelCfg("append", 2, 512, 8, 4, 128, 1536, 4096) if dtype == "bf16" else I.CONFIGS[1].cfg
    N, B, cap = 6, 16, 96
    ses = Session(cfg, I.gen_weights(cfg, 0), N, B, cap, page_size, "cuda:0", page_table=I.gen_page_table(N, (cap + page_size - 1) // page_size, 5), max_block=B)
    kv, v = ses.kv, ses.v
    gen = torch.Generator(device="cuda:0").manual_seed(7)
    for t in (kv.k, kv.v, v.k_stage, v.v_stage):
        t.normal_(generator=gen)
    room = kv.page_table.shape[1] * page_size
    seq_len = [0, 5, 7, 31, 8, room - 3]
    lead, acc = [0, 3, 1, 16, 0, 2], [16, 5, 0, 16, 0, 7]       # 16, 8, 1, 32 and 0 rows; the last has no room for its nine
    row0 = [0, 40, 3, 60, 11, 20]
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device="cuda:0")
    kv.seq_len.copy_(i32(seq_len))
    ses.d.span_len.copy_(i32([B] * N))
    v.stage_row0.copy_(i32(row0))
    v.stage_lead.copy_(i32(lead))
    want_k, want_v, table = kv.k.clone(), kv.v.clone(), kv.page_table.cpu()
    for n in range(N - 1):
        for t in range(lead[n] + acc[n]):
            s = seq_len[n] + t
            page, slot = int(table[n, s // page_size]), s % page_size
            want_k[:, page, :, slot] = v.k_stage[:, row0[n] + t]
            want_v[:, page, :, :, slot] = v.v_stage[:, row0[n] + t]
    ses.eng.s2d2_kv_append(kv, N, B, ses.d, v, i32(acc))
    assert torch.equal(kv.k, want_k) and torch.equal(kv.v, want_v)
    assert kv.seq_len.cpu().tolist() == [s + a + b for s, a, b in zip(seq_len[:-1], lead, acc)] + seq_len[-1:]
    assert kv.status.cpu().tolist() == [0] * (N - 1) + [-2]
