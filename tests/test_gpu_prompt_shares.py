"""The products of a prompt chunk that are cut into the eight shares of the reduction length, against the token-by-token pass: the same bits, at shares of
less than one, of one and of several phases of 8 blocks, with shares that are shorter or empty, and numbers of weight tiles that leave
waves of the last workgroup without one (two, four and eight waves)."""
import numpy as np
import pytest

import ppd_inputs as pi
from gpu_common import gpu_generate
from helpers import small_cfg
from paper_2307_05908_amd import binding

pytestmark = pytest.mark.gpu

SHAPES = [("opt", 64, 40), ("opt", 192, 256), ("opt", 832, 2048), ("opt", 1600, 2056), ("llama", 1664, 4096), ("llama", 2432, 4104), ("opt", 3136, 4360)]


@pytest.mark.parametrize("family,d_model,d_ff", SHAPES)
def test_shares_of_the_reduction_are_the_token_by_token_pass_bit_exact(family, d_model, d_ff, monkeypatch):
    heads = d_model // (128 if family == "llama" else 64)
    cfg = small_cfg(family, d_model=d_model, n_heads=heads, head_dim=d_model // heads, d_ff=d_ff, n_layers=3, exit_layer=2, max_ctx=60, n_gen=3, vocab=700)
    dev = binding.upload_model(pi.make_model(cfg))
    got = []
    for chunk in (None, "1"):
        if chunk:
            monkeypatch.setenv("PPD_PREFILL_CHUNK", chunk)
        P = binding.PPD(cfg, dev, k=2)
        got.append([gpu_generate(P, pi.make_prompt(cfg, n), cfg.n_gen, mode) for n in (9, 10, 16, 17, 18, 31, 32) for mode in ("ppd", "plain")])
        P.close()
    for a, b in zip(*got):
        np.testing.assert_array_equal(a[0], b[0])
        np.testing.assert_array_equal(a[1].view(np.uint32), b[1].view(np.uint32))
        assert a[2] == b[2]
