"""GPU: vocabulary statistics over infinities, NaN and ties wherever two logits can meet (a lane, a wavefront, a workgroup, chunks),
and draws of a row shared by eight, four, two workgroups or one, against 64 bits."""
import math

import numpy as np
import pytest
import torch

import s2d2_inputs as I
from oracle import s2d2_oracle as O
from paper_2603_25702_amd import Engine
from paper_2603_25702_amd.binding import S2D2_SAMPLE, Params
from paper_2603_25702_amd.runner import Session

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [4096 + 1000, 4096 + 1003])   # rows of 16 bytes and ragged ones
def test_statistics_of_special_rows(V):
    cfg = I.shrink(I.CONFIGS[2].cfg, n_layers=1, d_model=64, n_q_heads=1, n_kv_heads=1, head_dim=64, d_ffn=64, vocab=V)
    eng = Engine(cfg, I.gen_weights(cfg, 0), 1, 16)
    x = torch.randn((16, V), device="cuda:0", generator=torch.Generator(device="cuda:0").manual_seed(V)) * 3.0
    low = torch.finfo(torch.float32).min
    for r, at in enumerate([(5, 6), (5, 1029), (8, 200), (8, 300), (8, 900), (8, 4200), (4095, 4096)]):   # ties: one lane, wavefront, workgroup, two chunks
        x[r, list(at)] = 20.0
    x[7] = 1.5                                   # all the same
    x[8] = -math.inf                             # one comparable logit, at the end
    x[8, V - 1] = -3.0
    x[9] = low                                   # the lowest finite value, one above it
    x[9, 77] = 0.0
    x[10, :4096] = -math.inf                     # an empty chunk in front
    x[11] = low                                  # nothing but the lowest finite value
    x[12, 30] = math.inf
    x[13, 31] = math.nan
    x[14] = -math.inf
    got = {k: t.cpu() for k, t in eng.s2d2_vocab_draft_stats(x).items()}
    d = x[:12].double().cpu()
    lp = torch.log_softmax(d, dim=1)
    top = torch.topk(lp, 2, dim=1).values.exp()
    assert torch.equal(got["xhat"][:12].long(), (d == d.max(dim=1, keepdim=True).values).double().argmax(dim=1))
    want = {"p": top[:, 0], "margin": top[:, 0] - top[:, 1], "entropy_n": -torch.special.xlogy(lp.exp(), lp.exp()).sum(dim=1) / math.log(V)}
    for k, w in want.items():   # 16 terms per lane and a tree, 6e-8 each; exponentials within 2e-7, arguments within 1e-6
        assert (got[k][:12].double() - w).abs().max() <= 4e-6, k
    lse = torch.logsumexp(d, dim=1)
    assert ((got["lse"][:12].double() - lse).abs() <= 4e-6 * 21 + 1e-7 * lse.abs()).all()
    # no distribution: the largest comparable logit (the first index without one), and NaN where the sums are
    assert got["xhat"][12] == 30 and got["xhat"][14] == 0
    assert got["xhat"][13] == int(x[13].nan_to_num(-math.inf).argmax())
    for r in (12, 13):
        assert got["p"][r].isnan() and got["lse"][r].isnan() and got["margin"][r].isnan() and got["entropy_n"][r] == 0


@pytest.mark.parametrize("N,B", [(1, 3), (8, 8), (8, 16), (19, 7)])   # 8, 4, 2 workgroups and one a row
def test_draws_of_shared_rows(N, B):
    cfg = I.shrink(I.CONFIGS[1].cfg, vocab=6 * 4096 + 5)
    ses = Session(cfg, I.gen_weights(cfg, 1), N, B, 64, 16, "cuda:0", max_block=B)
    ses.reset_blocks([5] * N, torch.arange(N, dtype=torch.int32).numpy())
    T = 0.8
    for step in (3, 4):   # (the second finds the counters as the first left them)
        ses.eng.s2d2_draft(ses.kv, ses.st, N, B, Params(seed=11, step=step, mode=S2D2_SAMPLE, temperature=T), ses.d)
        rows, tok, p = ses.d.logit_row_of.cpu(), ses.d.xhat.cpu(), ses.d.p.cpu()
        prob = torch.softmax(ses.d.logits.double().cpu() / T, dim=1)
        drawn = 0
        for n in range(N):
            for i in range(B):
                if int(rows[n, i]) < 0:
                    continue
                q, t = prob[int(rows[n, i])], int(tok[n, i])
                u, hi = O.uniform(11, step, n, i, O.STREAM_DRAFT), float(q[: t + 1].sum())
                # two levels of fp32 sums of 24581 terms: at most 4 + 6 + 8 + 25 roundings of 6e-8 in a row, 2e-7 an exponential
                assert hi - float(q[t]) - 5e-6 <= u <= hi + 5e-6, (n, i, t)
                assert abs(float(p[n, i]) - float(q[t])) <= 4e-6
                drawn += 1
        assert drawn >= N * (B - 1)
