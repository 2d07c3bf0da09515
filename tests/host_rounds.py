"""One decoding context over the stand-in for the HIP runtime (hip_stand_in.c).  Imported in a process of its own: the stand-in has to
be there before libppd.so, and torch must not be."""
import ctypes
import os
import re
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.dirname(HERE))

SI = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)

from paper_2307_05908_amd import binding                       # noqa: E402
from paper_2307_05908_amd.build import LIB_PATH                # noqa: E402

LIB = ctypes.CDLL(LIB_PATH)
LIB.ppd_set_sampling.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_double, ctypes.c_uint64]


class Context:
    def __init__(self, k=3, exit_layer=3, **dims):
        base = dict(n_layers=6, d_model=256, n_heads=2, head_dim=128, d_ff=696, vocab=1237, max_ctx=1200, norm=1, act=2, pos=1,
                    has_bias=0, wdtype=1, norm_eps=1e-5, rope_theta=1e4, eos_id=-1)
        base.update(dims)
        d = binding.ModelDims(**base)
        self.dummy = ctypes.create_string_buffer(4096)             # (no kernel runs: never read)
        at = ctypes.cast(self.dummy, ctypes.c_void_p).value
        w = binding.Weights()
        for n in ("tok_emb", "pos_emb", "lnf_g", "lnf_b", "lm_head"):
            setattr(w, n, at)
        self.tabs = []
        for n in binding._W_LAYER_ORDER:
            self.tabs.append((ctypes.c_void_p * d.n_layers)(*[at] * d.n_layers))
            setattr(w, n, self.tabs[-1])
        self.h = ctypes.c_void_p()
        assert LIB.ppd_create(ctypes.byref(d), ctypes.byref(w), k, exit_layer, None, ctypes.byref(self.h)) == 0

    def prefill(self, n):
        assert LIB.ppd_prefill(self.h, (ctypes.c_int32 * n)(), n) == 0

    def sample(self, mode, top_k=0, top_p=1.0, seed=0):
        assert LIB.ppd_set_sampling(self.h, mode, top_k, top_p, seed) == 0

    def step(self, plain=False, match=-1):
        """One token; what the host launched for it: (before the replayed round, in it)."""
        tok = (ctypes.c_int32 * 1)()
        ctypes.c_int32.in_dll(SI, "si_match").value = match
        SI.si_clear()
        rc = LIB.plain_greedy_step(self.h, tok) if plain else LIB.ppd_step(self.h, tok, 1, None)
        assert rc == 1, rc
        before, _, inside = log().partition("G \n")
        return kernels(before), kernels(inside)

    def stats(self):
        s = binding.Stats()
        assert LIB.ppd_get_stats(self.h, ctypes.byref(s)) == 0
        return {n: int(getattr(s, n)) for n, _ in s._fields_}

    def close(self):
        LIB.ppd_destroy(self.h)


def log():
    return ctypes.c_char_p(ctypes.addressof(ctypes.c_char.in_dll(SI, "si_log"))).value.decode()


def kernels(text):
    return [re.sub(r"^_ZN3ppd\d+|^_ZN12_GLOBAL__N_1\d+", "", l[2:]) for l in text.splitlines() if l.startswith("K ")]


def counter(name):
    return ctypes.c_int.in_dll(SI, name).value
