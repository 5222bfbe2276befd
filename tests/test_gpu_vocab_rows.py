"""GPU: vocabulary statistics of thousands of rows (16383 and 16386 workgroups of 4096 logits), against the same statistics in 64 bits: arg-max and runner-up at the ends of the chunks, ties across them, -inf."""
import math

import pytest
import torch

import s2d2_inputs as I
from paper_2603_25702_amd import Engine

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [8195, 8196, 12288])   # rows that start unaligned; a last chunk of 4 logits; chunks that fill 1.5 of the larger ones
def test_statistics_on_either_side_of_the_line(V):
    cfg = I.shrink(I.CONFIGS[2].cfg, n_layers=1, d_model=64, n_q_heads=1, n_kv_heads=1, head_dim=64, d_ffn=64, vocab=V)
    eng = Engine(cfg, I.gen_weights(cfg, 0), 86, 64)
    below, above = 16383 // 3, 16383 // 3 + 1           # three chunks of 4096 in a row
    gen = torch.Generator(device="cuda:0").manual_seed(V)
    x = torch.randn((above, V), device="cuda:0", generator=gen) * 3.0
    edge = [0, 4095, 4096, 8191, 8192, V - 1]
    for r in range(len(edge)):                          # the two largest at the ends of chunks
        x[r, edge[r]], x[r, edge[(r + 3) % len(edge)]] = 20.0, 18.0
    x[6, 4095] = x[6, 4096] = x[6, 8192] = 20.0         # ties: the lowest index, no margin
    x[7, 1:] = -math.inf                                # one comparable logit
    x[8, : V - 2] = -math.inf                           # whole chunks of -inf
    got = [{k: t.clone() for k, t in eng.s2d2_vocab_draft_stats(x[:n]).items()} for n in (below, above)]
    scored = [eng.s2d2_vocab_score(x[:n], (g["xhat"] + 1) % V) for n, g in zip((below, above), got)]
    for r0 in range(0, above, 1024):
        d = x[r0:r0 + 1024].double()
        lp = torch.log_softmax(d, dim=1)
        top = torch.topk(lp, 2, dim=1).values.exp()
        want = {"p": top[:, 0], "margin": top[:, 0] - top[:, 1], "lse": torch.logsumexp(d, dim=1),
                "entropy_n": -torch.special.xlogy(lp.exp(), lp.exp()).sum(dim=1) / math.log(V)}
        want["xhat"] = (d == d.max(dim=1, keepdim=True).values).double().argmax(dim=1)   # lowest index of a tie
        for n, g, (q, lse) in zip((below, above), got, scored):
            m = min(n - r0, d.shape[0])
            assert torch.equal(g["xhat"][r0:r0 + m].long(), want["xhat"][:m])
            # a row's sums: up to 32 terms per thread and a tree behind them, 6e-8 each; exponentials within 2e-7 of a term
            # and arguments within 1e-6: 4e-6 in all
            for k in ("p", "margin", "entropy_n"):
                assert (g[k][r0:r0 + m].double() - want[k][:m]).abs().max() <= 4e-6, k
            for got_lse in (g["lse"], lse):                 # (two kernels finish the row: the same bound, not the same bits)
                assert (got_lse[r0:r0 + m].double() - want["lse"][:m]).abs().max() <= 4e-6 * 21
            nxt = ((want["xhat"][:m] + 1) % V).unsqueeze(1)
            assert (q[r0:r0 + m].double() - lp[:m].gather(1, nxt).squeeze(1).exp()).abs().max() <= 4e-6
