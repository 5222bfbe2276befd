"""Which GEMM kernel a forward runs on its matrices (host only: the rules, not the kernels)."""
import dataclasses

import pytest

import s2d2_inputs as I
from paper_2603_25702_amd.binding import S2D2Error, s2d2_gemm_choice

LAYER = ("qkv", "o", "gateup", "down")
DENSE = [I.CONFIGS[k].cfg for k in (2, 3, 4)]


@pytest.mark.parametrize("cfg", DENSE, ids=lambda c: c.name)
@pytest.mark.parametrize("shifted", [0, 1])
def test_windows_of_few_rows_do_not_pay_for_tiles_of_128(cfg, shifted):
    """Up to 48 expected rows the streaming or the mid-size kernel has a layer's matrices, whatever rows are possible: 11 to 16 masked
    positions of a right-shifted model have a verifier of as many rows and room for three times that."""
    cfg = dataclasses.replace(cfg, right_shifted=bool(shifted))
    for N in range(1, 49):
        for B in range(1, 48 // N + 1):
            for forward in ("draft", "verify"):
                rows = N * B * (2 if forward == "verify" and not shifted else 1)
                if rows <= 48:
                    for m in LAYER:
                        assert s2d2_gemm_choice(cfg, forward, N, B, m)[0] in ("stream", "mid"), (N, B, forward, m)


@pytest.mark.parametrize("cfg", DENSE + [I.CONFIGS[5].cfg], ids=lambda c: c.name)
def test_unembedding_of_more_than_16_rows_goes_through_lds(cfg):
    for N, B in ((1, 4), (1, 16), (4, 4), (1, 17), (5, 7), (16, 16), (32, 32)):
        for forward in ("draft", "verify"):
            assert s2d2_gemm_choice(cfg, forward, N, B, "unembed")[0] == ("lds" if N * B > 16 else "stream"), (N, B, forward)


@pytest.mark.parametrize("d,kernel", [(256, "lds"), (288, "tile"), (320, "lds"), (352, "tile")])
def test_unembedding_whose_columns_are_no_multiple_of_64_is_tiled(d, kernel):
    cfg = I.ModelCfg("columns", 1, d, 8, 4, 128, 512, 2048)
    assert s2d2_gemm_choice(cfg, "draft", 3, 43, "unembed")[0] == kernel
    assert s2d2_gemm_choice(cfg, "draft", 3, 43, "unembed", act_planes=2)[0] == "tile"   # (two planes: 16-bit halves only)


@pytest.mark.parametrize("d,vocab,rows,kernel", [
    (2048, 8192, 32, "mid"), (2048, 8192, 64, "mid"), (2048, 8192, 128, "lds"), (2048, 8192, 256, "tile"), (2048, 16384, 512, "tile"), (4096, 8192, 128, "tile"),
    (2048, 32000, 32, "lds"), (2048, 24576, 64, "lds"), (2048, 36864, 256, "lds"), (4096, 20480, 256, "lds"), (2048, 20480, 512, "lds"), (4096, 36864, 320, "tile"),
])
def test_unembedding_of_small_vocabularies_leaves_the_kernel_through_lds(d, vocab, rows, kernel):
    """Its workgroups take as long for one feature tile as for 16: two tiles a workgroup, 8192 features of 2048 columns and 256 rows, took 17 us longer."""
    assert s2d2_gemm_choice(I.ModelCfg("vocab", 1, d, 16, 8, 128, 1024, vocab), "draft", rows // 16, 16, "unembed")[0] == kernel


def test_gate_up_through_lds_for_large_matrices_of_many_rows():
    """Which of the kernels has gate / up is seen from outside: the one through LDS is not reported as the tiled one."""
    for cfg, forward, N, B, kernel in ((DENSE[2], "draft", 16, 16, "lds"), (DENSE[2], "verify", 16, 16, "lds"), (DENSE[0], "prefill", 4, 192, "lds"),
                                       (DENSE[2], "draft", 4, 16, "block"), (DENSE[1], "verify", 8, 8, "block"), (DENSE[0], "draft", 1, 4, "stream")):
        assert s2d2_gemm_choice(cfg, forward, N, B, "gateup")[0] == kernel, (cfg.name, forward, N, B)
    for d, f in ((736, 65536), (704, 12288), (2080, 6144), (2048, 2016), (1024, 4064)):   # fewer than 768 columns or no multiple of 64, matrices of less than 16 MB
        for rows in range(1, 65):
            assert s2d2_gemm_choice(I.ModelCfg("small", 1, d, 8, 4, 128, f, 2048), "draft", 16, rows, "gateup")[0] != "lds", (d, f, rows)
    for d, f, N, B in ((768, 6144, 13, 59), (1024, 4096, 41, 25), (1536, 4608, 31, 33)):
        assert s2d2_gemm_choice(I.ModelCfg("mid", 1, d, 8, 4, 128, f, 2048), "draft", N, B, "gateup")[0] == "lds", (d, f)


@pytest.mark.parametrize("cfg", DENSE, ids=lambda c: c.name)
def test_gate_up_has_its_kernel_whatever_the_other_matrices_have(cfg):
    """The kernel through LDS wants its operands in fragment order: they come so where it is the only one that does (8B, 832 rows and more:
    the other three matrices are tiled).  Fewer heads leave gate / up the same and give the others to other kernels."""
    few = dataclasses.replace(cfg, n_q_heads=8, n_kv_heads=4)
    for N in (1, 5, 8, 13, 16, 22, 26, 28, 32, 40, 48):
        for B in range(1, 65):
            for forward in ("draft", "verify"):
                if N * B * (2 if forward == "verify" else 1) > 48:
                    assert s2d2_gemm_choice(cfg, forward, N, B, "gateup") == s2d2_gemm_choice(few, forward, N, B, "gateup"), (N, B, forward)


def test_arguments_are_checked():
    cfg = DENSE[0]
    for args in (("draft", 0, 4, "qkv"), ("verify", 1, 65, "o"), ("prefill", 1, 193, "o"), ("prefill", 4, 60, "unembed")):
        with pytest.raises(S2D2Error):
            s2d2_gemm_choice(cfg, *args)
    with pytest.raises(S2D2Error):
        s2d2_gemm_choice(I.CONFIGS[5].cfg, "draft", 4, 4, "down")
    with pytest.raises(S2D2Error):
        s2d2_gemm_choice(I.CONFIGS[1].cfg, "draft", 1, 4, "qkv")
