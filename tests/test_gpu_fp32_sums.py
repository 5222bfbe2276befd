"""GPU: the sums of the fp32 model.  Every sum has one association, so what a sequence gets depends neither on the batch it
runs in nor on the capacity of its cache; and the edges of the attention and GEMM kernels' passes against the oracle."""
import numpy as np
import pytest
import torch

import s2d2_inputs as I
from paper_2603_25702_amd import Params
from paper_2603_25702_amd.runner import Session
from tests import harness as H
from tests.test_gpu_parity import run_steps

pytestmark = pytest.mark.gpu

TINY = I.CONFIGS[1].cfg


def first_sequence(N, pages):
    """One step over N sequences with `pages` pages of page table each; what sequence 0 gets (its inputs are always the same)."""
    B, ps, used, S = 4, 16, 14, 190
    W = I.gen_weights(TINY, 5)
    table = np.zeros((N, pages), dtype=np.int32)
    table[:, :used] = np.arange(N * used, dtype=np.int32).reshape(N, used)   # (pages past the used ones: never reached)
    ses = Session(TINY, W, N, B, pages * ps, ps, "cuda:0", page_table=table, max_block=B)
    gen = torch.Generator().manual_seed(9)
    for t in (ses.kv.k, ses.kv.v):
        t[:, :used].copy_(torch.randn((t.shape[0], used) + tuple(t.shape[2:]), generator=gen) * I.kv_sigma(TINY))
        t[:, used:].copy_(t[:, :1])
    ses.reset_blocks([S] * N)
    ses.step(Params(seed=3), advance=False)
    torch.cuda.synchronize()
    rd, rv = ses.d.logit_row_of[0].long(), ses.v.logit_row_of[0].long()
    got = {"logits": ses.d.logits[rd], "logits_ver": ses.v.logits_ver[rv], "xhat": ses.d.xhat[0], "p": ses.d.p[0], "margin": ses.d.margin[0],
           "entropy_n": ses.d.entropy_n[0], "q": ses.v.q[0], "k": ses.v.k_stage[:, :2 * B], "v": ses.v.v_stage[:, :2 * B],
           "n_accept": ses.a.n_accept[0], "block": ses.st.block_tokens[0]}
    return {k: t.cpu().clone() for k, t in got.items()}


@pytest.mark.parametrize("N,pages", [
    (40, 20),      # 320 rows: more than one workgroup per compute unit in the down projection, which then keeps fewer loads in flight
    (1, 2500),     # a cache of 40000 keys, whose scores take all but a few KB of LDS
])
def test_a_sequence_gets_the_same_bits_in_any_batch_and_cache(N, pages):
    one, other = first_sequence(1, 20), first_sequence(N, pages)
    for k in one:
        assert torch.equal(one[k], other[k]), f"{k}: {(one[k].double() - other[k].double()).abs().max()}"


# Attention hands a chain of keys through four quarters of 12 keys each: 48 keys x (256 / head_dim) per pass.  The GEMM
# takes K in passes of 256 (fp32) whose last one may be ragged or leave wavefronts without a share.
@pytest.mark.parametrize("head_dim,d_ffn,lens", [
    (32, 1040, [383, 380, 1]),     # keys of the four draft rows: 387, 384 (one pass of 384 and a bit) and 5
    (64, 272, [188, 189, 600]),    # exactly one pass of 192, one key more, several; K of one pass and a single fragment
    (128, 528, [92, 93, 0]),       # 96 keys, 97, none cached
    (256, 2064, [44, 45, 300]),    # one chain per element, 48 keys, 49; K of eight passes and a bit
])
def test_edges_of_the_passes_over_keys_and_inputs(head_dim, d_ffn, lens):
    cfg = I.ModelCfg("edges-f32", 2, 256, 4, 2, head_dim, d_ffn, 4096, dtype="f32")
    case = H.make_case(cfg, len(lens), 4, lens, seed=15, synthetic_kv=True, page_size=16, room=64, norm_jitter=0.1)
    run, rep = run_steps(case, 2)
    print("edges:", head_dim, d_ffn, rep)
    # chains of up to 600 products and K of up to 2064, each rounding 6e-8 of a partial sum: the walk of the roundings
    # stays below sqrt(2064) * 6e-8 = 3e-6 of the largest logit; a missed or doubled key or input shows at 1e-3 and more
    assert rep.max_logit_err_draft <= 1e-5 and rep.max_logit_err_verify <= 1e-5
