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


def test_arguments_are_checked():
    cfg = DENSE[0]
    for args in (("draft", 0, 4, "qkv"), ("verify", 1, 65, "o"), ("prefill", 1, 193, "o"), ("prefill", 4, 60, "unembed")):
        with pytest.raises(S2D2Error):
            s2d2_gemm_choice(cfg, *args)
    with pytest.raises(S2D2Error):
        s2d2_gemm_choice(I.CONFIGS[5].cfg, "draft", 4, 4, "down")
    with pytest.raises(S2D2Error):
        s2d2_gemm_choice(I.CONFIGS[1].cfg, "draft", 1, 4, "qkv")
