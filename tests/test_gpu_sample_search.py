"""The draw's search: every drawn token against the oracle's sampler on the GPU's own logits, over vocabularies and spreads
of the logits that put the edge of the kept set, and the draw, between the collected thresholds, beyond the last of them,
and among more tokens than are collected."""
import numpy as np
import pytest

import oracle
import ppd_inputs as pi
from helpers import small_cfg
from paper_2307_05908_amd import binding

pytestmark = pytest.mark.gpu

SEED = 77


def scaled_head(m, factor):
    h = m.g["lm_head"]
    v = (pi.to_float64(h) * factor).astype(np.float32)
    u = v.view(np.uint32).astype(np.uint64)
    m.g["lm_head"] = np.ascontiguousarray(((u + 0x7FFF + ((u >> 16) & 1)) >> 16).astype(np.uint16))


@pytest.mark.parametrize("vocab,factor", [(3, 1.0), (1023, 8.0), (1025, 30.0), (32769, 0.02), (32769, 1.0), (50272, 1.0), (50272, 14.0), (50272, 60.0)])
@pytest.mark.parametrize("mode,ks,p", [(oracle.TOP_P, 0, 0.95), (oracle.TOP_P, 0, 1.0), (oracle.TOP_K, 40, 1.0)])
def test_draw_is_the_oracles(vocab, factor, mode, ks, p):
    cfg = small_cfg("opt", vocab=vocab, n_layers=2, exit_layer=1, n_gen=6)
    m = pi.make_model(cfg)
    scaled_head(m, factor)
    P = binding.PPD(cfg, binding.upload_model(m), k=min(3, vocab))
    P.ppd_set_sampling(mode, ks, p, SEED)
    prompt = [int(x) for x in pi.make_prompt(cfg)]
    P.ppd_prefill(prompt)
    for t in range(cfg.n_gen):
        tok = P.plain_greedy_step()
        z = P.ppd_get_logits().astype(np.float64)
        u = oracle.uniform(SEED, len(prompt) + t)
        assert tok == oracle.sample(z, mode, ks, p, u), (t, u)
    P.close()


@pytest.mark.parametrize("vocab,factor", [(6145, 0.0), (50272, 0.0), (9000, 0.02), (16000, 20.0), (32000, 1.0), (128256, 0.3), (128256, 14.0), (128256, 40.0)])
@pytest.mark.parametrize("mode,ks,p", [(oracle.TOP_P, 0, 1.0), (oracle.TOP_P, 0, 0.999), (oracle.TOP_P, 0, 0.3), (oracle.TOP_K, 7000, 1.0)])
def test_draw_among_more_tokens_than_are_collected(vocab, factor, mode, ks, p):
    """Equal logits, flat softmaxes and long tails: the range in question holds more tokens than LDS does."""
    test_draw_is_the_oracles(vocab, factor, mode, min(ks, vocab - 1), p)


@pytest.mark.parametrize("p", [1 - 2.0 ** -53, 1 - 2.0 ** -52])
@pytest.mark.parametrize("vocab,factor", [(1000, 1.0), (5003, 3.6), (32000, 1.0), (50272, 3.6)])
def test_nearly_all_of_a_flat_softmax_is_kept(vocab, factor, p):
    """No token lies below the last threshold, and the mass asked for is an ulp from that of all tokens: the sums on both sides
    of the comparison have to be the same sum.  (Every position's logits are another rounding of it; the token that the oracle
    draws does not depend on the last bits of the kept mass, of which the draw leaves 2^-24 at least.)"""
    cfg = small_cfg("opt", vocab=vocab, n_layers=2, exit_layer=1, n_gen=80)
    m = pi.make_model(cfg)
    scaled_head(m, factor)
    P = binding.PPD(cfg, binding.upload_model(m))
    P.ppd_set_sampling(oracle.TOP_P, 0, p, SEED)
    prompt = [int(x) for x in pi.make_prompt(cfg)]
    P.ppd_prefill(prompt)
    wrong = []
    for t in range(cfg.n_gen):
        tok = P.plain_greedy_step()
        z = P.ppd_get_logits().astype(np.float64)
        assert z.max() - z.min() < 11.75                 # (the last threshold lies 11.75 below the largest logit)
        want = oracle.sample(z, oracle.TOP_P, 0, p, oracle.uniform(SEED, len(prompt) + t))
        if tok != want:
            wrong.append((t, tok, want))
    P.close()
    assert not wrong
