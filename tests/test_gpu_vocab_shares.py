"""GPU: vocabulary statistics of rows that one to all workgroups of their chunks share, against 64 bits: a chunk per workgroup, runs of two and of three chunks (the
most) with a shorter last one, a whole row in one workgroup, more chunks than lanes; called again and again (the arrival counters are back at zero)."""
import math

import pytest
import torch

import s2d2_inputs as I
from paper_2603_25702_amd import Engine

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,counts", [(266245, [17, 1]), (45003, [1100, 300, 3]), (45004, [1152]), (77003, [1152]), (77004, [1152, 900]), (12292, [1152]), (4096, [5]), (5, [2])])
def test_rows_shared_by_workgroups(V, counts):
    cfg = I.shrink(I.CONFIGS[2].cfg, n_layers=1, d_model=64, n_q_heads=1, n_kv_heads=1, head_dim=64, d_ffn=64, vocab=V)
    eng = Engine(cfg, I.gen_weights(cfg, 0), 18, 64)
    gen = torch.Generator(device="cuda:0").manual_seed(V)
    for rows in counts:
        for again in range(3):
            x = torch.randn((rows, V), device="cuda:0", generator=gen) * 3.0
            g = {k: t.clone() for k, t in eng.s2d2_vocab_draft_stats(x).items()}
            tok = torch.randint(0, V, (rows,), device="cuda:0", dtype=torch.int32, generator=gen)
            q, lse = eng.s2d2_vocab_score(x, tok)
            lp = torch.log_softmax(x.double(), dim=1)
            top = torch.topk(lp, 2, dim=1).values.exp()
            want = {"p": top[:, 0], "margin": top[:, 0] - top[:, 1], "entropy_n": -torch.special.xlogy(lp.exp(), lp.exp()).sum(dim=1) / math.log(V)}
            assert torch.equal(g["xhat"].long(), x.argmax(dim=1))
            for k, w in want.items():   # 6e-8 a term over a thread's 16 and the trees of lanes, wavefronts and chunks, exponentials within 2e-7, arguments within 1e-6
                assert (g[k].double() - w).abs().max() <= 4e-6, (k, rows, again)
            for l in (g["lse"], lse):
                assert (l.double() - torch.logsumexp(x.double(), dim=1)).abs().max() <= 4e-6 * 21
            assert (q.double() - lp.gather(1, tok.long().unsqueeze(1)).squeeze(1).exp()).abs().max() <= 4e-6
