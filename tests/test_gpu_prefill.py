"""GPU parity of the prompt prefill: prompts of one token, of exactly the 192 a chunk takes, and of more (equal chunks, the
last of them ragged), against the oracle's causal forward."""
import numpy as np
import pytest
import torch

import s2d2_inputs as I
from oracle import s2d2_oracle as O
from paper_2603_25702_amd.runner import Session
from tests import harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model,lens", [("tiny", [192, 1, 150]), ("bf16", [193, 5, 385]), ("shifted", [64, 200])])
def test_prefilled_cache_matches_a_causal_forward(model, lens):
    cfg = I.CONFIGS[1].cfg if model == "tiny" else I.ModelCfg("small-bf16", 2, 512, 8, 4, 128, 1536, 32000, right_shifted=model == "shifted")
    W, N, ps = I.gen_weights(cfg, 3), len(lens), 16
    ids = [I.gen_prefix_ids(cfg, n, 3, i) for i, n in enumerate(lens)]
    pages = (max(lens) + 64 + ps - 1) // ps
    table = I.gen_page_table(N, pages, 3)
    ses = Session(cfg, W, N, 4, pages * ps, ps, "cuda:0", page_table=table)
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
            assert np.abs(gk - ck[l]).max() <= tol * np.abs(ck[l]).max()
            assert np.abs(gv - cv[l]).max() <= tol * np.abs(cv[l]).max()
