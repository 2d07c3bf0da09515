"""Captured rounds belong to a kind, a grid of the attention and the kernels of a length (up to two chunks of positions, up to
eight, more).  Sequences of three tokens, short ones and long ones in turn on one context, meet every change in the middle:
the same bits as with every round issued launch by launch (PPD_GRAPHS=2)."""
import numpy as np
import pytest

import ppd_inputs as pi
from gpu_common import gpu_generate
from helpers import small_cfg
from paper_2307_05908_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("family,width", [("tiny", 256), ("opt", 192), ("opt", 384), ("llama", 1152)])
@pytest.mark.parametrize("alpha", [1.0, 0.02])
def test_replayed_rounds_are_the_issued_ones_bit_exact(family, width, alpha, monkeypatch):
    cfg = small_cfg(family, n_layers=4, exit_layer=2, d_model=width, n_heads=width // (128 if family == "llama" else 64), alpha=alpha, max_ctx=700, n_gen=3)
    dev = binding.upload_model(pi.make_model(cfg))
    prompts = [pi.make_prompt(cfg, n) for n in (5, 126, 40, 190, 510, 254, 9, 600, 140, 512)]
    got = []
    for graphs in ("1", "2"):
        monkeypatch.setenv("PPD_GRAPHS", graphs)
        P = binding.PPD(cfg, dev, k=3)
        got.append([gpu_generate(P, p, cfg.n_gen, mode) for _ in range(3) for p in prompts for mode in ("ppd", "plain")])
        P.close()
    for a, b in zip(*got):
        np.testing.assert_array_equal(a[0], b[0])
        np.testing.assert_array_equal(a[1].view(np.uint32), b[1].view(np.uint32))
        assert a[2] == b[2]
