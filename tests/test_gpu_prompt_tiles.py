"""The products of the compute-bound prompt pass with every tile shape and with the reduction length cut into parts
(PPD_PG_TILE, PPD_PG_PARTS), whatever the rule would choose: ragged tiles in both directions, parts of unequal length and
of a single 32-column block, every epilogue (bias, ReLU, SwiGLU, residual, packed outputs)."""
import numpy as np
import pytest

import ppd_inputs as pi
from gpu_common import gpu_generate
from helpers import small_cfg
from paper_2307_05908_amd import binding

pytestmark = pytest.mark.gpu

CFG = {
    "llama": small_cfg("llama", max_ctx=320, n_layers=2, exit_layer=1),
    "opt": small_cfg("opt", max_ctx=320, n_layers=2, exit_layer=1, d_ff=776),
}
LENGTHS = (34, 66, 131, 291)       # one row fewer goes through the layers
_ref = {}


def _generate(P):
    return [gpu_generate(P, pi.make_prompt(P.cfg, n), 3, "plain")[1] for n in LENGTHS]


def _reference(name, monkeypatch):
    """The same prompts a chunk of rows at a time, on the decode step's kernels."""
    if name not in _ref:
        dev = binding.upload_model(pi.make_model(CFG[name]))
        monkeypatch.setenv("PPD_PREFILL_TILED", "2")
        P = binding.PPD(CFG[name], dev, k=1)
        _ref[name] = dev, _generate(P)
        P.close()
        monkeypatch.delenv("PPD_PREFILL_TILED")
    return _ref[name]


@pytest.mark.parametrize("name", list(CFG))
@pytest.mark.parametrize("tile", range(1, 8))
@pytest.mark.parametrize("parts", [1, 3, 8])
def test_every_tile_and_cut_agrees_with_the_row_chunks(name, tile, parts, monkeypatch):
    dev, ref = _reference(name, monkeypatch)
    monkeypatch.setenv("PPD_PG_TILE", str(tile))
    monkeypatch.setenv("PPD_PG_PARTS", str(parts))
    P = binding.PPD(CFG[name], dev, k=1)
    got, again = _generate(P), _generate(P)
    P.close()
    for z, z2, r in zip(got, again, ref):
        # (rows in two bf16 terms on both sides, |x - hi - lo| <= 2^-17 |x|; other orders of the same fp32 sums: the row-chunk
        # tests of longer prompts have the same bound)
        assert np.abs(z - r).max() <= 1e-4
        np.testing.assert_array_equal(z.view(np.uint32), z2.view(np.uint32))     # the parts are added in their order


@pytest.mark.parametrize("name", list(CFG))
def test_products_stay_whole_where_the_parts_sums_cannot_be_allocated(name, monkeypatch):
    """(PPD_PG_WS=2 asks for more memory than a GPU has.)  The prompt runs as with PPD_PG_PARTS=1, bit for bit, the calls behind
    it find no error left over, and so does the rule's own choice, which cuts some of these products."""
    dev, _ = _reference(name, monkeypatch)
    got = []
    for env in ({"PPD_PG_PARTS": "1"}, {"PPD_PG_PARTS": "3", "PPD_PG_WS": "2"}, {"PPD_PG_WS": "2"}):
        for k, v in env.items():
            monkeypatch.setenv(k, v)
        P = binding.PPD(CFG[name], dev, k=1)
        got.append(_generate(P))
        P.close()
        for k in env:
            monkeypatch.delenv(k)
    for z, z2, z3 in zip(*got):
        np.testing.assert_array_equal(z.view(np.uint32), z2.view(np.uint32))
        assert np.abs(z - z3).max() <= 1e-4                  # (another tile may be the better one; the bound is the one above)
