"""Products of narrow models have a kernel of their own whose arithmetic and order of additions are the streaming kernel's:
the same tokens and logits, bit for bit, with the streaming kernel everywhere (PPD_MGPASSES=2) over widths at the edges of
its rules: blocks of a wave's share, 512-element pieces of the statistics, tiles per workgroup, rows per wave."""
import numpy as np
import pytest

import ppd_inputs as pi
from gpu_common import gpu_generate
from helpers import small_cfg
from paper_2307_05908_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("family,d_model,d_ff,k", [
    ("opt", 64, 8, 1), ("opt", 512, 1032, 3), ("opt", 576, 4096, 8), ("opt", 1024, 4104, 4),
    ("llama", 128, 2048, 8), ("llama", 1024, 2752, 5), ("llama", 1152, 3080, 3), ("llama", 2048, 5504, 8), ("llama", 2176, 4096, 2)])
def test_narrow_products_are_the_streaming_kernels_bit_exact(family, d_model, d_ff, k, monkeypatch):
    hd = 64 if family == "opt" else 128
    cfg = small_cfg(family, d_model=d_model, n_heads=d_model // hd, head_dim=hd, d_ff=d_ff, n_layers=2, exit_layer=1, alpha=0.1, n_gen=6)
    dev = binding.upload_model(pi.make_model(cfg))
    prompt = pi.make_prompt(cfg)
    got = []
    for passes in (None, "2"):
        if passes:
            monkeypatch.setenv("PPD_MGPASSES", passes)
        P = binding.PPD(cfg, dev, k=k)
        got.append([gpu_generate(P, prompt, cfg.n_gen, mode) for mode in ("plain", "ppd")])
        P.close()
    for a, b in zip(*got):
        np.testing.assert_array_equal(a[0], b[0])
        np.testing.assert_array_equal(a[1].view(np.uint32), b[1].view(np.uint32))
        assert a[2] == b[2]


@pytest.mark.parametrize("family,d_model,k", [("opt", 128, 8), ("opt", 576, 3), ("opt", 1024, 8), ("llama", 256, 8), ("llama", 1152, 3), ("llama", 1152, 8)])
@pytest.mark.parametrize("n_prompt", [125, 189, 252, 318, 506])
def test_partials_merged_in_the_output_projection_bit_exact(family, d_model, k, n_prompt, monkeypatch):
    """Up to eight chunks of positions, across their boundaries and across the first position beyond them: the merge's own launch
    and order on the other side."""
    hd = 64 if family == "opt" else 128
    cfg = small_cfg(family, d_model=d_model, n_heads=d_model // hd, head_dim=hd, d_ff=520, vocab=700, n_layers=2, exit_layer=1, alpha=0.1,
                    max_ctx=560, n_prompt=n_prompt, n_gen=10)
    dev = binding.upload_model(pi.make_model(cfg))
    prompt = pi.make_prompt(cfg)
    got = []
    for passes in (None, "2"):
        if passes:
            monkeypatch.setenv("PPD_MGPASSES", passes)
        P = binding.PPD(cfg, dev, k=k)
        got.append([gpu_generate(P, prompt, cfg.n_gen, mode) for mode in ("plain", "ppd")])
        P.close()
    for a, b in zip(*got):
        np.testing.assert_array_equal(a[0], b[0])
        np.testing.assert_array_equal(a[1].view(np.uint32), b[1].view(np.uint32))
        assert a[2] == b[2]


@pytest.mark.parametrize("family,d_model,d_ff,k", [
    ("opt", 64, 4096, 2), ("opt", 128, 1024, 8), ("opt", 128, 1032, 8), ("opt", 1024, 1032, 3), ("opt", 1088, 1032, 3), ("llama", 2048, 4096, 4), ("llama", 2176, 1032, 1)])
def test_half_tiles_are_the_streaming_kernels_bit_exact(family, d_model, d_ff, k, monkeypatch):
    """Two workgroups to a tile: shares of 4 and of 5 blocks, the most tiles of one and of two groups and more, with and without the merge of partials."""
    hd = 64 if family == "opt" else 128
    cfg = small_cfg(family, d_model=d_model, n_heads=d_model // hd, head_dim=hd, d_ff=d_ff, n_layers=3, exit_layer=2, alpha=0.1, n_prompt=63, n_gen=6)
    dev = binding.upload_model(pi.make_model(cfg))
    got = []
    for passes in (None, "2"):
        if passes:
            monkeypatch.setenv("PPD_MGPASSES", passes)
        P = binding.PPD(cfg, dev, k=k)
        got.append([gpu_generate(P, pi.make_prompt(cfg), cfg.n_gen, mode) for mode in ("plain", "ppd")])
        P.close()
    for a, b in zip(*got):
        np.testing.assert_array_equal(a[0], b[0])
        np.testing.assert_array_equal(a[1].view(np.uint32), b[1].view(np.uint32))
        assert a[2] == b[2]
