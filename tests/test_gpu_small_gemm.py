"""Short reduction lengths with fp32 weights have a kernel of their own whose additions are the streaming kernel's: the
logits of a vocabulary small enough for it against those of a larger one (which the streaming kernel takes) on the same
rows, bit for bit, at the edges of the 256-element blocks; and the ids are the top of these logits."""
import numpy as np
import pytest
import torch

import oracle
import ppd_inputs as pi
from gpu_common import TOL, gpu_generate, run_against_oracle
from helpers import small_cfg
from paper_2307_05908_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [8, 248, 256, 264, 512, 520, 768, 1016, 1024])
@pytest.mark.parametrize("norm", [0, 1])
def test_short_rows_are_the_streaming_kernels_bit_exact(K, norm):
    gen = torch.Generator().manual_seed(K + norm)
    head = torch.randn(8200, K, generator=gen).cuda()          # 2050 sets of 4 rows: more than 512 workgroups of 4 waves
    h = (3 * torch.randn(K, generator=gen) + 1).cuda()
    g = (1 + 0.1 * torch.randn(K, generator=gen)).cuda()
    b = (0.1 * torch.randn(K, generator=gen)).cuda() if norm == 0 else None
    _, _, big = binding.ppd_early_topk(h, g, b, head, 8, norm, 1e-5, want_logits=True)
    big = np.asarray(big.cpu() if torch.is_tensor(big) else big)
    for vocab in (8, 9, 1001, 8189):
        ids, vals, z = binding.ppd_early_topk(h, g, b, head[:vocab].contiguous(), 8, norm, 1e-5, want_logits=True)
        z = np.asarray(z.cpu() if torch.is_tensor(z) else z)
        ids = np.asarray(ids.cpu() if torch.is_tensor(ids) else ids)
        np.testing.assert_array_equal(z.view(np.uint32), big[:vocab].view(np.uint32))
        np.testing.assert_array_equal(ids, np.argsort(-z, kind="stable")[:8])


def fp32_cfg(act, d_model, d_ff, **kw):
    """GELU / ReLU models with LayerNorm, biases and learned positions, SwiGLU ones with RMSNorm and RoPE."""
    base = dict(act=act, d_model=d_model, n_heads=d_model // 64, d_ff=d_ff, vocab=1201, n_layers=2, exit_layer=1, max_ctx=64, n_prompt=19, n_gen=8)
    if act == pi.ACT_SWIGLU:
        base.update(norm=pi.NORM_RMS, pos=pi.POS_ROPE, has_bias=0)
    base.update(kw)
    return small_cfg("tiny", **base)


def padded(cfg, extra):
    """The same model with `extra` more feed-forward columns that come out as zero."""
    n = pi.make_model(cfg)
    L = n.layers
    for l in range(cfg.n_layers):
        for name in ("w_in", "w_up", "b_in"):
            if L[name][l] is not None:
                a = L[name][l]
                L[name][l] = np.concatenate([a, np.zeros((extra,) + a.shape[1:], a.dtype)])
        L["w_out"][l] = np.ascontiguousarray(np.concatenate([L["w_out"][l], np.ones((cfg.d_model, extra), np.float32)], axis=1))
    return n


@pytest.mark.parametrize("act", [pi.ACT_GELU, pi.ACT_RELU, pi.ACT_SWIGLU])
@pytest.mark.parametrize("d_model,k", [(64, 3), (320, 1), (512, 4), (768, 3), (1024, 8)])
def test_feed_forward_in_is_the_streaming_kernels_bit_exact(act, d_model, k):
    """4096 feed-forward columns are the most the short-row kernel takes; with eight more, all zero, the streaming kernel
    has the same rows: one row, k rows and prompt rows, with norm, bias and activation, pairs of matrices."""
    cfg = fp32_cfg(act, d_model, 4096)
    m = pi.make_model(cfg)
    prompt = pi.make_prompt(cfg)
    got = []
    for c, mm in ((cfg, m), (cfg.replace(d_ff=4104), padded(cfg, 8))):
        P = binding.PPD(c, binding.upload_model(mm), k=k)
        got.append([gpu_generate(P, prompt, cfg.n_gen, mode)[:2] for mode in ("plain", "ppd")])
        P.close()
    for (tok, z), (rtok, rz) in zip(*got):
        np.testing.assert_array_equal(tok, rtok)
        np.testing.assert_array_equal(z.view(np.uint32), rz.view(np.uint32))


@pytest.mark.parametrize("act", [pi.ACT_GELU, pi.ACT_SWIGLU])
@pytest.mark.parametrize("d_model", [256, 576, 1024])
def test_prompt_rows_are_the_one_row_pass_bit_exact(act, d_model, monkeypatch):
    """2 to 8 rows of a prompt chunk against one row at a time (queries, keys and values, residuals)."""
    cfg = fp32_cfg(act, d_model, 1000)
    dev = binding.upload_model(pi.make_model(cfg))
    runs = []
    for chunk in (None, "1"):
        if chunk:
            monkeypatch.setenv("PPD_PREFILL_CHUNK", chunk)
        P = binding.PPD(cfg, dev, k=3)
        runs.append([gpu_generate(P, pi.make_prompt(cfg, n), 3, "plain")[1] for n in (3, 5, 6, 9, 10, 19)])
        P.close()
    for z, rz in zip(*runs):
        np.testing.assert_array_equal(z.view(np.uint32), rz.view(np.uint32))


@pytest.mark.parametrize("act,d_model,d_ff", [(pi.ACT_SWIGLU, 256, 1000), (pi.ACT_GELU, 1024, 1024), (pi.ACT_SWIGLU, 640, 4104), (pi.ACT_GELU, 1088, 1032)])
def test_chunks_of_32_rows_are_the_one_row_pass_bit_exact(act, d_model, d_ff, monkeypatch):
    """Prompts around 8, 16, 24 and 32 rows, eight to a workgroup: all products in the short-row kernel, at its longest rows, and some or
    all of them in the streaming one, against one row and eight rows at a time."""
    cfg = fp32_cfg(act, d_model, d_ff).replace(max_ctx=80)
    dev = binding.upload_model(pi.make_model(cfg))
    runs = []
    for chunk in (None, "1", "8"):
        if chunk:
            monkeypatch.setenv("PPD_PREFILL_CHUNK", chunk)
        P = binding.PPD(cfg, dev, k=3)
        runs.append([gpu_generate(P, pi.make_prompt(cfg, n), 2, mode)[1] for n in (9, 10, 17, 18, 25, 32, 33, 34, 42, 67) for mode in ("ppd", "plain")])
        P.close()
    for z, *others in zip(*runs):
        for rz in others:
            np.testing.assert_array_equal(z.view(np.uint32), rz.view(np.uint32))


@pytest.mark.parametrize("act,d_model,d_ff,k", [(pi.ACT_SWIGLU, 192, 520, 3), (pi.ACT_SWIGLU, 640, 1016, 8), (pi.ACT_GELU, 1024, 1024, 5), (pi.ACT_RELU, 448, 2048, 1)])
def test_short_rows_match_the_oracle(act, d_model, d_ff, k):
    cfg = fp32_cfg(act, d_model, d_ff)
    m = pi.make_model(cfg)
    prompt = pi.make_prompt(cfg)
    ro = oracle.Oracle(m).ppd(prompt, cfg.n_gen, k, cfg.exit_layer, want_logits=True)
    P = binding.PPD(cfg, binding.upload_model(m), k=k)
    run_against_oracle(P, prompt, "ppd", ro["tokens"], ro["final_logits"], ro["early_logits"], tol=TOL[cfg.wdtype])
    P.close()
