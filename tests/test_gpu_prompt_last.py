"""x_0, the prompt's last token, goes through all layers but the last with the prompt's other rows; PPD_PREFILL_LAST=2 leaves it to
the first round.  Prompts whose rows take the decode step's arithmetic (one chunk of a bf16 model): the same bits, tokens,
candidates and counters, over exit layers, numbers of candidates, and prompts of which x_0 is the last of a few rows, of a tile and of the chunk.  Prompts that
leave x_0 to the first round (several chunks, fp32 models) are among them as they stood before.  Longer prompts of bf16 models: close
logits, and PPD == plain greedy bit for bit.  Which of these prompts take x_0 along is what test_host_rounds.py checks, without a GPU."""
import numpy as np
import pytest

import ppd_inputs as pi
from gpu_common import TOL, gpu_generate
from helpers import small_cfg
from paper_2307_05908_amd import binding

pytestmark = pytest.mark.gpu

CASES = {
    "tiny_2_layers": small_cfg("tiny", n_layers=2, exit_layer=1, n_gen=3),
    "tiny": small_cfg("tiny", n_gen=4, alpha=0.05),
    "opt": small_cfg("opt", n_gen=4, max_ctx=160, alpha=0.05),
    "opt_wider": small_cfg("opt", d_model=384, n_heads=6, n_gen=4, max_ctx=160),             # launch by launch
    "llama_2_layers": small_cfg("llama", n_layers=2, exit_layer=1, n_gen=3, max_ctx=160),
    "llama": small_cfg("llama", n_gen=4, max_ctx=160),
    "llama_late": small_cfg("llama", exit_layer=5, alpha=0.02, n_gen=4, max_ctx=160),
}
ONE_CHUNK = (1, 2, 3, 8, 9, 16, 17, 32)
LONG = (33, 34, 63, 64, 65, 66, 100, 128, 129, 257, 590)      # (in the compute-bound pass; several chunks with PPD_PREFILL_TILED=2)


def generate(cfg, dev, prompts, k, monkeypatch, **env):
    for name, v in env.items():
        monkeypatch.setenv(name, v)
    P = binding.PPD(cfg, dev, k=k)
    out = []
    for n in prompts:
        prompt = pi.make_prompt(cfg, n)
        a = gpu_generate(P, prompt, cfg.n_gen, "ppd")
        st = P.ppd_get_stats()
        b = gpu_generate(P, prompt, 2, "plain")
        P.ppd_prefill(prompt)
        P.ppd_step()
        out.append((a, b, P.ppd_get_early_logits(), [st[f] for f in ("rounds", "matches", "runs", "main_layer_rows", "branch_layer_rows")]))
    P.close()
    for name in env:
        monkeypatch.delenv(name)
    return out


@pytest.mark.parametrize("k", [1, 3, 8])
@pytest.mark.parametrize("name", list(CASES))
def test_x0_with_the_prompt_is_x0_by_itself_bit_exact(name, k, monkeypatch):
    cfg = CASES[name]
    dev = binding.upload_model(pi.make_model(cfg))
    prompts = ONE_CHUNK + ((33, 34, 64, 65, 66, 100) if cfg.max_ctx >= 120 else ())
    env = dict(PPD_PREFILL_TILED="2")
    got = generate(cfg, dev, prompts, k, monkeypatch, **env)
    ref = generate(cfg, dev, prompts, k, monkeypatch, PPD_PREFILL_LAST="2", **env)
    eager = generate(cfg, dev, prompts, k, monkeypatch, PPD_SPIN_TICKS="1", PPD_GRAPHS="2", **env)     # (a chain gives up in its first round)
    for n, g, r, e in zip(prompts, got, ref, eager):
        for x in (g, e):
            for a, b in zip(x[:2], r[:2]):
                np.testing.assert_array_equal(a[0], b[0], err_msg=str(n))
                np.testing.assert_array_equal(a[1].view(np.uint32), b[1].view(np.uint32), err_msg=str(n))
                assert a[2] == b[2], n
            np.testing.assert_array_equal(x[2].view(np.uint32), r[2].view(np.uint32), err_msg=str(n))
            assert x[3] == r[3], n


@pytest.mark.parametrize("name", ["opt", "opt_wider", "llama", "llama_late"])
def test_x0_with_a_long_prompt(name, monkeypatch):
    cfg = CASES[name].replace(max_ctx=600, n_gen=5)
    dev = binding.upload_model(pi.make_model(cfg))
    prompts = (33, 63, 64, 65, 128, 129, 257, 590)
    got = generate(cfg, dev, prompts, 3, monkeypatch)
    ref = generate(cfg, dev, prompts, 3, monkeypatch, PPD_PREFILL_LAST="2")
    for n, g, r in zip(prompts, got, ref):
        np.testing.assert_array_equal(g[0][0][:2], g[1][0])                               # PPD == plain greedy
        np.testing.assert_array_equal(g[0][1][:2].view(np.uint32), g[1][1].view(np.uint32))
        # (either way every logit is within the oracle's tolerance; measured distances are some 1e-5)
        assert np.abs(g[1][1][0] - r[1][1][0]).max() <= TOL[cfg.wdtype] / 100, n
        assert np.abs(g[2] - r[2]).max() <= TOL[cfg.wdtype] / 100, n


@pytest.mark.parametrize("mode,ks,p", [(1, 3, 1.0), (2, 0, 0.95)])
@pytest.mark.parametrize("name", ["opt", "opt_wider", "llama", "llama_late"])
def test_a_seed_draws_what_it_draws_with_x0_by_itself(name, mode, ks, p, monkeypatch):
    """Sampling switched on before or behind the prompt, and with PPD_PREFILL_LAST=2: the same tokens, logits and early logits."""
    cfg = CASES[name].replace(max_ctx=200, n_gen=4)
    dev = binding.upload_model(pi.make_model(cfg))

    def draw(P, n, behind, plain):
        P.ppd_set_sampling(0)
        if not behind:
            P.ppd_set_sampling(mode, ks, p, 20230713)
        P.ppd_prefill(pi.make_prompt(cfg, n))
        if behind:
            P.ppd_set_sampling(mode, ks, p, 20230713)
        out = []
        for t in range(cfg.n_gen):
            out.append(np.float32(P.plain_greedy_step() if plain else P.ppd_step()[0]))
            out.extend(P.ppd_get_logits())
            if not plain:
                out.extend(P.ppd_get_early_logits())
        return np.array(out, np.float32)

    P = binding.PPD(cfg, dev, k=3)
    monkeypatch.setenv("PPD_PREFILL_LAST", "2")
    Q = binding.PPD(cfg, dev, k=3)
    for n in (20, 33, 64, 128, 177):
        for plain in (False, True):
            ref = draw(Q, n, False, plain)
            for X, behind in ((P, False), (P, True), (Q, True)):
                np.testing.assert_array_equal(draw(X, n, behind, plain).view(np.uint32), ref.view(np.uint32), err_msg=f"{n} {behind} {plain}")
    P.close()
    Q.close()


def test_a_prompt_that_fills_the_context_window():
    cfg = small_cfg("llama", max_ctx=70)
    dev = binding.upload_model(pi.make_model(cfg))
    P = binding.PPD(cfg, dev, k=3)
    prompt = pi.make_prompt(cfg, 70)
    P.ppd_prefill(prompt)
    with pytest.raises(binding.PPDError) as ei:
        P.ppd_step()                                  # the candidates have no position left
    assert ei.value.code == -3
    tok = P.plain_greedy_step()
    z = P.ppd_get_logits()
    assert tok == int(np.argmax(z))
    with pytest.raises(binding.PPDError):
        P.plain_greedy_step()
    P.close()
