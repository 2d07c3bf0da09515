"""What the host launches for a round, on the CPU: the library over a stand-in for the HIP runtime that writes the calls down
(hip_stand_in.c), in a process of its own."""
import os
import subprocess
import sys

import pytest

import ppd_inputs as pi
from test_gpu_prompt_last import CASES, LONG, ONE_CHUNK

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("si") / "hip_stand_in.so")
    subprocess.check_call(["gcc", "-O1", "-Wall", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "hip_stand_in.c")])
    return so


def run(stand_in, body, **env):
    from paper_2307_05908_amd import binding
    binding.load_library()                                     # (built if nothing is)
    e = {k: v for k, v in os.environ.items() if not k.startswith("PPD_")}
    r = subprocess.run([sys.executable, "-c", "from host_rounds import *\n" + body, stand_in], cwd=HERE, env=dict(e, **env),
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-4000:]


def dims(cfg):
    return {n: getattr(cfg, n) for n in ("n_layers", "d_model", "n_heads", "head_dim", "d_ff", "vocab", "max_ctx", "norm", "act", "pos", "has_bias", "wdtype")}


# The first round's attention launches.  Where x_0 went along, one for it, elsewhere one a layer (a PPD round: up to the exit layer E); and one
# for each layer of the candidates, with or without x_0.
ALONG = """
def attentions(C, n, plain):
    C.prefill(n)
    return sum(k.startswith("attn_kernel") or k.startswith("attn_whole") for k in C.step(plain)[1])
def along(C, n):
    plain, ppd = attentions(C, n, True), attentions(C, n, False) - (L - E)
    assert (plain, ppd) in ((1, 1), (L, E)), (plain, ppd)
    return plain == 1
"""


@pytest.mark.parametrize("name", list(CASES))
def test_where_x0_goes_with_the_prompt(stand_in, name):
    """The prompts of test_gpu_prompt_last.py take the path that it compares: x_0 goes along behind one chunk and in the compute-bound
    pass, not in fp32 models, not where several chunks go through the decode step's kernels, and not with PPD_PREFILL_LAST=2."""
    cfg = CASES[name].replace(max_ctx=600)
    body = f"""
L, E, bf16 = {cfg.n_layers}, {cfg.exit_layer}, {cfg.wdtype == pi.WD_BF16}
C = Context(3, {cfg.exit_layer}, **{dims(cfg)})
{ALONG}
for n in {ONE_CHUNK}:
    assert along(C, n) == (ONE_CHUNK and bf16 and n > 1), n
for n in {LONG}:
    assert along(C, n) == (TILED and bf16), n
C.close()
"""
    run(stand_in, "ONE_CHUNK = TILED = True\n" + body, PPD_FUSED="2")
    run(stand_in, "ONE_CHUNK, TILED = True, False\n" + body, PPD_FUSED="2", PPD_PREFILL_TILED="2")
    run(stand_in, "ONE_CHUNK = TILED = False\n" + body, PPD_FUSED="2", PPD_PREFILL_LAST="2")
    run(stand_in, "ONE_CHUNK = TILED = False\n" + body, PPD_FUSED="2", PPD_PREFILL_CHUNK="1")


def test_a_further_row_of_tiles_costs_wide_models_more_than_the_step(stand_in):
    cfg = pi.CONFIGS["llama7b"].replace(n_layers=4, exit_layer=2, vocab=512, max_ctx=640)
    run(stand_in, f"""
L, E = {cfg.n_layers}, {cfg.exit_layer}
C = Context(3, {cfg.exit_layer}, **{dims(cfg)})
{ALONG}
assert [n for n in (2, 32, 33, 64, 65, 128, 129, 256, 257, 258, 512, 513, 514) if not along(C, n)] == [257, 513]
C.close()
""", PPD_FUSED="2")


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("plain", [False, True])
def test_sampling_switched_on_behind_a_long_prompt_starts_from_the_embedding(stand_in, mode, plain):
    """A seed's tokens do not depend on whether ppd_set_sampling comes before or behind ppd_prefill: x_0 goes through all layers by
    itself either way."""
    run(stand_in, f"""
mode, plain = {mode}, {plain}
C = Context()
C.prefill(64)
_, taken = C.step(plain)                                       # (the arg max: x_0 went with the prompt)
C.sample(mode, 3, 0.9, 7)
C.prefill(64)
_, alone = C.step(plain)
assert len(alone) > len(taken)
C.sample(0)
C.prefill(64)
assert C.step(plain)[1] == taken
C.prefill(64)
C.sample(mode, 3, 0.9, 7)
before, late = C.step(plain)
assert late == alone, (late, alone)
assert [k for k in before if k.startswith("embed_kernel")], before
C.sample(0)
C.prefill(20)                                                  # one chunk: the decode step's bits, x_0 stays with the prompt
C.sample(mode, 3, 0.9, 7)
assert len(C.step(plain)[1]) < len(alone)
C.close()
""", PPD_FUSED="2")


@pytest.mark.parametrize("last", ["1", "2"])
def test_the_first_rounds_counters_fit_each_other(stand_in, last):
    """Bytes and layer rows of a first round count the same layers, whether x_0 went with the prompt or not: what the bytes hold over
    the rows' weights is whole passes over the LM head, keys and values are those of the rows."""
    run(stand_in, """
nb, wl, wh, kv = 3, 2 * (4 * 256 * 256 + 3 * 256 * 696), 2 * 1237 * 256, 2 * 256 * 4
C = Context()
for n in (1, 20, 64):
    C.prefill(n)
    C.step()
    s = C.stats()
    assert s["main_layer_rows"] == 6 and s["branch_layer_rows"] == 3 * nb
    assert s["weight_bytes"] == (6 + nb) * wl + 2 * wh, (n, s)
    assert s["kv_bytes"] == (6 * (n - 1) + nb * n) * kv, (n, s)
    C.prefill(n)
    C.step(plain=True)
    s = C.stats()
    assert s["weight_bytes"] == 6 * wl + wh and s["kv_bytes"] == 6 * (n - 1) * kv, (n, s)
C.close()
""", PPD_FUSED="2", PPD_PREFILL_LAST=last)


def test_a_round_is_waited_for_before_its_graph_goes(stand_in):
    """A round returns on the word of its last kernel, which may still run: a captured round that is captured anew for a longer
    sequence, or dropped with the rule it was captured for, is destroyed only once the stream has been waited for."""
    run(stand_in, """
for plain in (False, True):
    C = Context(max_ctx=2100)
    for n in (506, 1018, 2042):
        C.prefill(n)
        for t in range(12):                                        # (512, 1024 and 2048 positions: another grid of the attention)
            C.step(plain, match=t % 3 - 1)
    C.sample(1, 3, 1.0, 7)
    assert counter("si_destroyed") > 0
    assert counter("si_destroyed_under_way") == 0
    C.close()
""", PPD_FUSED="2")
