"""The main token's layers in one launch against one launch per step of a layer: the same bits, over layer shapes whose
tiles, blocks and attention items do not divide evenly among the workgroups and waves; and a launch that has to give up
waiting (a spin limit of one tick, set from the host) is run again one launch per step."""
import threading
import time

import numpy as np
import pytest

import ppd_inputs as pi
from gpu_common import gpu_generate
from helpers import small_cfg
from paper_2307_05908_amd import binding

pytestmark = pytest.mark.gpu

CASES = {
    "llama": small_cfg("llama"),                                   # head_dim as configured, one attention item per head
    "opt": small_cfg("opt"),                                       # LayerNorm, biases, learned positions
    "llama_300": small_cfg("llama", max_ctx=420, n_prompt=300, n_gen=12),     # several items per head, odd number of chunks
    "opt_250": small_cfg("opt", max_ctx=300, n_prompt=250, n_gen=12),
    # more 16-row tiles than workgroups in every product, ragged feed-forward width, more attention items than workgroups
    "wide": small_cfg("llama", d_model=4224, n_heads=33, head_dim=128, d_ff=11000, vocab=700, n_layers=2, exit_layer=1,
                      max_ctx=1300, n_prompt=1215, n_gen=4),
    "wide_ln": small_cfg("opt", d_model=2112, n_heads=33, head_dim=64, d_ff=8456, vocab=700, n_layers=2, exit_layer=1,
                         max_ctx=200, n_prompt=127, n_gen=4),
}


def run(cfg, dev, prompt, monkeypatch, rounds=None, **env):
    """Tokens, logits and rounds of both modes; rounds: receives the chain's counters."""
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    P = binding.PPD(cfg, dev)
    out = [gpu_generate(P, prompt, cfg.n_gen, mode) for mode in ("plain", "ppd")]
    if rounds is not None:
        rounds.append(P.ppd_get_chain_rounds())
    P.close()
    for k in env:
        monkeypatch.delenv(k)
    return out


@pytest.mark.parametrize("name", list(CASES))
def test_one_launch_is_one_launch_per_step_bit_exact(name, monkeypatch):
    cfg = CASES[name]
    dev = binding.upload_model(pi.make_model(cfg))
    prompt = pi.make_prompt(cfg)
    rounds = []
    one = run(cfg, dev, prompt, monkeypatch, rounds)
    steps = run(cfg, dev, prompt, monkeypatch, rounds, PPD_FUSED="2")
    # every plain step, and the PPD rounds that do not begin at the exit layer (here: those behind no match)
    behind = [m for m, _, _ in one[1][2]][:-1]
    assert rounds == [(2 * cfg.n_gen - sum(behind), 0), (0, 0)]
    for a, b in zip(one, steps):
        np.testing.assert_array_equal(a[0], b[0])
        np.testing.assert_array_equal(a[1], b[1])
        assert a[2] == b[2]


@pytest.mark.parametrize("family", ["llama", "opt"])
def test_a_chain_that_begins_behind_a_match_bit_exact(family, monkeypatch):
    """An exit layer above the middle and a late part that changes little: rounds behind a match go through the layers
    between in one launch, too."""
    n = {"llama": 6, "opt": 4}[family]
    cfg = small_cfg(family, n_layers=n, exit_layer=n - 1, alpha=0.02, max_ctx=160, n_prompt=70, n_gen=30)
    dev = binding.upload_model(pi.make_model(cfg))
    prompt = pi.make_prompt(cfg)
    rounds = []
    one = run(cfg, dev, prompt, monkeypatch, rounds)
    steps = run(cfg, dev, prompt, monkeypatch, PPD_FUSED="2")
    assert sum(m for m, _, _ in one[1][2][:-1]) > 0 and rounds == [(2 * cfg.n_gen, 0)]
    for a, b in zip(one, steps):
        np.testing.assert_array_equal(a[0], b[0])
        np.testing.assert_array_equal(a[1], b[1])
        assert a[2] == b[2]


@pytest.mark.parametrize("name", ["llama_300", "opt"])
def test_a_launch_that_gives_up_is_run_again(name, monkeypatch):
    cfg = CASES[name]
    dev = binding.upload_model(pi.make_model(cfg))
    prompt = pi.make_prompt(cfg)
    rounds = []
    gave_up = run(cfg, dev, prompt, monkeypatch, rounds, PPD_SPIN_TICKS="1")
    steps = run(cfg, dev, prompt, monkeypatch, PPD_FUSED="2")
    assert rounds == [(1, 1)]          # the first round; those after it go without
    for a, b in zip(gave_up, steps):
        np.testing.assert_array_equal(a[0], b[0])
        np.testing.assert_array_equal(a[1], b[1])
        assert a[2] == b[2]


@pytest.mark.parametrize("family", ["llama", "opt"])
def test_a_round_behind_a_match_is_run_again(family, monkeypatch):
    """The chain of such a round begins behind the layers that the matching candidate has been through: their keys and
    values at the round's position stay, and every later token attends to them."""
    n = {"llama": 6, "opt": 4}[family]
    cfg = small_cfg(family, n_layers=n, exit_layer=n - 1, alpha=0.02, max_ctx=160, n_prompt=40, n_gen=30)
    dev = binding.upload_model(pi.make_model(cfg))
    prompt = pi.make_prompt(cfg)
    ref = run(cfg, dev, prompt, monkeypatch, PPD_FUSED="2")[1]
    match = [m for m, _, _ in ref[2]]
    first = match.index(1)
    assert first < cfg.n_gen // 2
    P = binding.PPD(cfg, dev)
    P.ppd_prefill(prompt)
    for t in range(cfg.n_gen):
        if t == first + 1:
            assert P.ppd_get_chain_rounds() == (first + 1, 0)
            P.ppd_set_chain_wait(1)
        tok, info = P.ppd_step()
        if t == first + 1:
            assert P.ppd_get_chain_rounds() == (first + 2, 1)
        assert tok == ref[0][t], t
        assert (info.matched, info.match_idx, list(info.cand)) == ref[2][t], t
        np.testing.assert_array_equal(P.ppd_get_logits(), ref[1][t])
    P.close()


def test_contexts_at_work_together_go_launch_by_launch():
    """Two contexts that one thread uses in turn take the one-launch chain every round; from two threads they meet, and go
    launch by launch then.  The tokens and logits stay the same."""
    cfg = small_cfg("llama", max_ctx=260, n_prompt=40, n_gen=200)
    dev = binding.upload_model(pi.make_model(cfg))
    prompt = pi.make_prompt(cfg)
    P = [binding.PPD(cfg, dev) for _ in range(2)]
    time.sleep(0.1)                                   # (a meeting with an earlier test's contexts is over)
    ref = gpu_generate(P[0], prompt, cfg.n_gen, "plain")
    assert P[0].ppd_get_chain_rounds() == (cfg.n_gen, 0)
    for p in P:
        p.ppd_prefill(prompt)
    for t in range(20):
        for p in P:
            assert p.plain_greedy_step() == ref[0][t]
    assert [p.ppd_get_chain_rounds() for p in P] == [(cfg.n_gen + 20, 0), (20, 0)]
    got, gate = [None, None], threading.Barrier(2)

    def work(i):
        gate.wait()
        got[i] = gpu_generate(P[i], prompt, cfg.n_gen, "plain")

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for g in got:
        np.testing.assert_array_equal(g[0], ref[0])
        np.testing.assert_array_equal(g[1], ref[1])
    rounds = [p.ppd_get_chain_rounds() for p in P]
    assert rounds[0][0] + rounds[1][0] < 3 * cfg.n_gen + 40 and rounds[0][1] + rounds[1][1] == 0
    for p in P:
        p.close()


def test_the_chain_comes_back_after_a_launch_gave_up(monkeypatch):
    """64 rounds go without the chain then, 128 after the second time; its attention partials (several per head here) are
    in order again."""
    cfg = small_cfg("llama", max_ctx=560, n_prompt=300, n_gen=230)
    dev = binding.upload_model(pi.make_model(cfg))
    prompt = pi.make_prompt(cfg)
    ref = run(cfg, dev, prompt, monkeypatch, PPD_FUSED="2")[0]
    P = binding.PPD(cfg, dev)
    P.ppd_prefill(prompt)
    count = []
    for t in range(cfg.n_gen):
        if t in (5, 80):
            P.ppd_set_chain_wait(1)
        assert P.plain_greedy_step() == ref[0][t], t
        np.testing.assert_array_equal(P.ppd_get_logits(), ref[1][t])
        if t in (5, 80):
            P.ppd_set_chain_wait(0)
        count.append(P.ppd_get_chain_rounds())
    P.close()
    assert count[5] == (6, 1) and count[69] == (6, 1) and count[70] == (7, 1)
    assert count[80] == (17, 2) and count[208] == (17, 2) and count[229] == (38, 2)


@pytest.mark.parametrize("heads,head_dim,limit", [(2, 128, 48 * 64), (3, 64, 72 * 64)])
def test_long_sequences_leave_the_chain(heads, head_dim, limit, monkeypatch):
    """Past 24 chunks of positions per head the rounds go launch by launch: the same tokens and logits across the line."""
    cfg = small_cfg("llama", n_layers=2, exit_layer=1, n_heads=heads, head_dim=head_dim, d_model=heads * head_dim, max_ctx=limit + 64, n_prompt=limit - 3, n_gen=8)
    dev = binding.upload_model(pi.make_model(cfg))
    prompt = pi.make_prompt(cfg)
    ref = run(cfg, dev, prompt, monkeypatch, PPD_FUSED="2")[0]
    P = binding.PPD(cfg, dev)
    got = gpu_generate(P, prompt, cfg.n_gen, "plain")
    np.testing.assert_array_equal(got[0], ref[0])
    np.testing.assert_array_equal(got[1], ref[1])
    assert P.ppd_get_chain_rounds() == (4, 0)        # positions limit - 4 .. limit - 1
    P.close()
