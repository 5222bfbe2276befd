"""GPU parity of the prompt prefill: prompts of one token, of exactly the 192 a chunk takes, and of more (equal chunks, the
last of them ragged), against the oracle's causal forward; experts, two operand planes and a page size that the MFMA
attention does not take; a prompt the cache has no room for, and the calls that are refused."""
import numpy as np
import pytest
import torch

import s2d2_inputs as I
from oracle import s2d2_oracle as O
from paper_2603_25702_amd.binding import S2D2Error
from paper_2603_25702_amd.runner import Session
from tests import harness as H

pytestmark = pytest.mark.gpu

BF16 = I.ModelCfg("small-bf16", 2, 512, 8, 4, 128, 1536, 32000)
MODELS = {"tiny": I.CONFIGS[1].cfg, "bf16": BF16, "planes": BF16, "pages of 12": BF16,
          "shifted": I.ModelCfg("small-bf16", 2, 512, 8, 4, 128, 1536, 32000, right_shifted=True),
          "moe": I.ModelCfg("small-moe", 2, 512, 8, 4, 128, 0, 32000, n_experts=8, top_k=2, d_expert=256)}
ENOSPC, EINVAL = -2, -1


@pytest.mark.parametrize("model,lens", [("tiny", [192, 1, 150]), ("bf16", [193, 5, 385]), ("shifted", [64, 200]),
                                        ("planes", [100, 193]), ("pages of 12", [193, 30]), ("moe", [40, 193])])
def test_prefilled_cache_matches_a_causal_forward(model, lens):
    cfg = MODELS[model]
    W, N, ps = I.gen_weights(cfg, 3), len(lens), 12 if model == "pages of 12" else 16
    ids = [I.gen_prefix_ids(cfg, n, 3, i) for i, n in enumerate(lens)]
    pages = (max(lens) + 64 + ps - 1) // ps
    table = I.gen_page_table(N, pages, 3)
    ses = Session(cfg, W, N, 4, pages * ps, ps, "cuda:0", page_table=table, act_planes=2 if model == "planes" else 0)
    ses.prefill(ids)
    assert ses.kv.seq_len.cpu().tolist() == [n - int(model == "shifted") for n in lens]
    assert not ses.kv.status.cpu().any()
    k, v = ses.kv.k.float().cpu().numpy(), ses.kv.v.float().cpu().numpy()
    tol = 1e-4 if cfg.dtype == "f32" else H.LOGIT_RTOL
    for n, L in enumerate(lens):
        ck, cv = O.prefill(cfg, W, ids[n])
        at = np.arange(L)
        page, slot = table[n, at // ps], at % ps
        for l in range(cfg.n_layers):
            gk, gv = k[l, page, :, slot], v[l, page, :, :, slot]   # [L, Hkv, D]
            off = np.maximum(np.abs(gk - ck[l]).max(axis=(1, 2)) / np.abs(ck[l]).max(), np.abs(gv - cv[l]).max(axis=(1, 2)) / np.abs(cv[l]).max())
            if cfg.is_moe and l > 0:   # a token whose last expert is tied to rounding takes another one in layer 0: its rows of layer 1 differ, few of them
                assert (off > tol).mean() <= 0.05, (n, l, off.max())
            else:
                assert off.max() <= tol, (n, l, off.max())


def small_session(N=2, pages=4):
    cfg = MODELS["tiny"]
    return Session(cfg, I.gen_weights(cfg, 3), N, 4, pages * 16, 16, "cuda:0", max_block=4), cfg


def test_a_prompt_without_room_leaves_its_sequence_as_it_was():
    ses, cfg = small_session()
    ses.kv.seq_len.copy_(torch.tensor([60, 40], dtype=torch.int32))
    before = ses.kv.k.clone(), ses.kv.v.clone()
    tok = torch.arange(24, dtype=torch.int32, device="cuda:0").view(2, 12)
    ses.eng.s2d2_prefill(ses.kv, 2, 12, tok, 0, torch.tensor([5, 12], dtype=torch.int32, device="cuda:0"), ses.v.k_stage, ses.v.v_stage)
    assert ses.kv.status.cpu().tolist() == [ENOSPC, 0]         # 65 of 64 places, 52 of 64
    assert ses.kv.seq_len.cpu().tolist() == [60, 52]
    for t, b in zip((ses.kv.k, ses.kv.v), before):
        assert torch.equal(t[:, :4], b[:, :4]) and not torch.equal(t[:, 4:], b[:, 4:])
    # token counts outside [0, T] are cut: nothing for the first sequence, all of the chunk for the second
    ses.kv.status.zero_()
    ses.eng.s2d2_prefill(ses.kv, 2, 12, tok, 0, torch.tensor([-3, 99], dtype=torch.int32, device="cuda:0"), ses.v.k_stage, ses.v.v_stage)
    assert ses.kv.status.cpu().tolist() == [0, 0] and ses.kv.seq_len.cpu().tolist() == [60, 64]


def test_refused_calls():
    ses, cfg = small_session()
    kv, e = ses.kv, ses.eng
    tok = torch.zeros((2, 16), dtype=torch.int32, device="cuda:0")
    cnt = torch.ones(2, dtype=torch.int32, device="cuda:0")
    ks, vs = ses.v.k_stage, ses.v.v_stage

    def call(N=2, T=12, ld=16, tokens=tok.data_ptr(), n=cnt.data_ptr(), k=ks.data_ptr(), v=vs.data_ptr()):
        return e.lib.s2d2_prefill(e.ctx, kv.c(), N, T, tokens, ld, n, k, v)

    assert call() == 0
    for bad in (dict(N=0), dict(N=3), dict(T=0), dict(T=13), dict(ld=11), dict(tokens=None), dict(n=None), dict(k=None), dict(v=None),
                dict(k=ks.data_ptr() + 4), dict(v=vs.data_ptr() + 8)):
        assert call(**bad) == EINVAL, bad
    with pytest.raises(S2D2Error):
        e.s2d2_prefill(kv, 2, 13, tok, 0, cnt, ks, vs)
    assert ses.kv.seq_len.cpu().tolist() == [1, 1]
