"""GPU: expert choices on ties.  Router logits that are all zero, of either sign, are one big tie: the lowest indices win."""
import pytest
import torch

import s2d2_inputs as I
from paper_2603_25702_amd import Params
from paper_2603_25702_amd.runner import Session

pytestmark = pytest.mark.gpu


def test_zeros_of_either_sign_are_a_tie():
    """Embeddings of about 1e25 overflow the fp32 sum of squares: 1/rms is 0, and every logit behind a norm is a product
    of either sign times 0.  (The norms' gains bring the GEMM inputs back to half range, so the products are finite.)"""
    cfg = I.ModelCfg("moe-ties", 2, 512, 8, 4, 128, 0, 4096, n_experts=8, top_k=3, d_expert=256)
    W = I.gen_weights(cfg, 4)
    W["embed"] = (W["embed"].float() * 1e25 / I.WEIGHT_STD).to(cfg.torch_dtype)
    for k in W:
        if "norm" in k:
            W[k] = torch.full_like(W[k], 1e-25)
    N, B = 3, 8
    ses = Session(cfg, W, N, B, 64, 16, "cuda:0", max_block=B)
    ses.reset_blocks([5, 9, 16])
    tok = torch.arange(N * B, dtype=torch.int32).view(N, B) * 97 % cfg.mask_id     # different rows: signs of all kinds
    tok[:, -1] = cfg.mask_id
    ses.st.block_tokens.copy_(tok)
    ses.eng.s2d2_draft(ses.kv, ses.st, N, B, Params(), ses.d)
    got = ses.eng.s2d2_moe_choices(N * B).cpu().view(cfg.n_layers, N * B, cfg.top_k)
    assert torch.equal(got, torch.arange(cfg.top_k, dtype=got.dtype).expand_as(got))
