"""Prompts of up to 32 rows of a bf16 model in one pass over the weights against the token-by-token pass
(PPD_PREFILL_CHUNK=1): the same bits, at the edges of the two 16-row tiles, over feed-forward widths that give a
workgroup one to more than eight weight tiles, ragged last tiles and columns, and across the 64-position chunks."""
import numpy as np
import pytest

import ppd_inputs as pi
from gpu_common import gpu_generate
from helpers import small_cfg
from paper_2307_05908_amd import binding

pytestmark = pytest.mark.gpu

SMALL = dict(n_layers=3, exit_layer=2, max_ctx=160, n_gen=5)
CASES = {
    "llama_2_tiles": small_cfg("llama", d_ff=2056, **SMALL),       # gate and up: 8 outputs per tile, 256 workgroups
    "llama_4_tiles": small_cfg("llama", d_ff=6200, **SMALL),
    "llama_6_tiles": small_cfg("llama", d_ff=10248, **SMALL),
    "llama_9_tiles": small_cfg("llama", d_ff=16392, **SMALL),      # more than fit a workgroup: more workgroups
    "opt": small_cfg("opt", **SMALL),
    "opt_ragged": small_cfg("opt", d_ff=8200, **SMALL),            # three tiles per workgroup, 8 columns in the last block
    "opt_wide": small_cfg("opt", d_model=2112, n_heads=33, head_dim=64, d_ff=200, **SMALL),
}


# where a few rows go through the decode step's launches: up to 4, 5 and (the rows have to fit LDS whole) 3 of them
WIDE = {"4_rows": (2048, 16), "5_rows": (4224, 33), "3_rows": (8192, 64)}


@pytest.mark.parametrize("name", list(WIDE))
def test_few_prompt_rows_are_the_token_by_token_pass_bit_exact(name, monkeypatch):
    d_model, heads = WIDE[name]
    cfg = small_cfg("llama", d_model=d_model, n_heads=heads, head_dim=128, d_ff=1096, n_layers=2, exit_layer=1, max_ctx=80, n_gen=3)
    dev = binding.upload_model(pi.make_model(cfg))
    runs = []
    for env in (("PPD_PREFILL_TILED", "2"), ("PPD_PREFILL_CHUNK", "1")):
        monkeypatch.setenv(*env)
        P = binding.PPD(cfg, dev, k=1)
        runs.append([gpu_generate(P, pi.make_prompt(cfg, n), cfg.n_gen, "plain")[:2] for n in (3, 4, 5, 6, 7, 36, 37, 69)])
        P.close()
        monkeypatch.delenv(env[0])
    for (tok, z), (rtok, rz) in zip(*runs):
        np.testing.assert_array_equal(tok, rtok)
        np.testing.assert_array_equal(np.asarray(z).view(np.uint32), np.asarray(rz).view(np.uint32))


@pytest.mark.parametrize("name", list(CASES))
def test_prompt_rows_are_the_token_by_token_pass_bit_exact(name, monkeypatch):
    cfg = CASES[name]
    dev = binding.upload_model(pi.make_model(cfg))

    def run(n_prompt):
        P = binding.PPD(cfg, dev, k=3)
        out = [gpu_generate(P, pi.make_prompt(cfg, n_prompt), cfg.n_gen, mode)[:2] for mode in ("plain", "ppd")]
        P.close()
        return out

    lengths = [3, 5, 6, 16, 17, 18, 32, 33, 34, 35, 100]     # one row fewer goes through the layers
    monkeypatch.setenv("PPD_PREFILL_TILED", "2")             # (the default from 32 rows on is the compute-bound pass)
    got = {n: run(n) for n in lengths}
    monkeypatch.setenv("PPD_PREFILL_CHUNK", "1")
    for n in lengths:
        for (tok, z), (rtok, rz) in zip(got[n], run(n)):
            np.testing.assert_array_equal(tok, rtok)
            np.testing.assert_array_equal(np.asarray(z).view(np.uint32), np.asarray(rz).view(np.uint32))
