"""Up to two chunks of 64 positions a head's attention and its merge are one launch: the same bits as the chunk kernels and
the merge over the boundaries of the chunks.  The one-launch chain of layers and prompt chunks have the chunk kernels'
arithmetic; rows that a match adopts come out of k rows at a time."""
import numpy as np
import pytest

import ppd_inputs as pi
from gpu_common import gpu_generate
from helpers import small_cfg
from paper_2307_05908_amd import binding

pytestmark = pytest.mark.gpu


def same(a, b):
    np.testing.assert_array_equal(a[0], b[0])
    np.testing.assert_array_equal(a[1].view(np.uint32), b[1].view(np.uint32))


@pytest.mark.parametrize("family,head_dim", [("opt", 64), ("llama", 128), ("tiny", 64)])
@pytest.mark.parametrize("n_prompt", [1, 57, 121])
def test_short_sequences_are_the_chunk_kernels_bit_exact(family, head_dim, n_prompt, monkeypatch):
    cfg = small_cfg(family, n_layers=2, exit_layer=1, alpha=0.02, n_heads=2, head_dim=head_dim, d_model=2 * head_dim, max_ctx=160,
                    n_prompt=n_prompt, n_gen=14)
    dev = binding.upload_model(pi.make_model(cfg))
    prompt = pi.make_prompt(cfg)
    P = binding.PPD(cfg, dev, k=8)
    plain = gpu_generate(P, prompt, cfg.n_gen, "plain")
    ppd = gpu_generate(P, prompt, cfg.n_gen, "ppd")
    long = pi.make_prompt(cfg, 140)
    gpu_generate(P, long, 4, "ppd")                               # (the graphs of longer sequences are others)
    again = gpu_generate(P, prompt, cfg.n_gen, "ppd")
    P.close()
    assert sum(m for m, _, _ in ppd[2]) > 0
    same(plain, ppd)
    same(ppd, again)
    # bf16: one launch per step in place of the chain; fp32: the prompt one row at a time in place of rows of 8
    monkeypatch.setenv("PPD_FUSED", "2")
    if family == "tiny":
        monkeypatch.setenv("PPD_PREFILL_CHUNK", "1")
    P = binding.PPD(cfg, dev, k=8)
    other = gpu_generate(P, prompt, cfg.n_gen, "plain")
    P.close()
    same(plain, other)
