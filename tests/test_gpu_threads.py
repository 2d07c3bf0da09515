"""Contexts of several threads: rounds that one thread captures for replay beside every other kind of call of another."""
import threading
import time

import numpy as np
import pytest

import ppd_inputs as pi
from gpu_common import gpu_generate
from helpers import small_cfg
from paper_2307_05908_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("family", ["tiny", "llama"])
def test_captures_beside_another_threads_calls(family):
    """ppd_set_sampling drops the captured rounds, so one thread captures again and again; the other creates contexts, fills
    them and reads logits.  Neither fails, and both have the results they have alone."""
    cfg = small_cfg(family, n_layers=4, exit_layer=2, max_ctx=200, n_gen=12)
    dev = binding.upload_model(pi.make_model(cfg))
    prompt, other = pi.make_prompt(cfg, 20), pi.make_prompt(cfg, 60)
    P = binding.PPD(cfg, dev)
    Q = binding.PPD(cfg, dev)
    ref = gpu_generate(P, prompt, cfg.n_gen, "ppd")
    ref_q = gpu_generate(Q, other, cfg.n_gen, "plain")
    Q.close()
    errors, rounds, done = [], [], threading.Event()

    def capture():
        try:
            for _ in range(20):
                P.ppd_set_sampling(0)
                rounds.append(gpu_generate(P, prompt, cfg.n_gen, "ppd"))
        except Exception as e:       # (asserted on below, in the test's own thread)
            errors.append(e)
        done.set()

    t = threading.Thread(target=capture)
    t.start()
    got = []
    try:
        while not done.is_set() or not got:
            R = binding.PPD(cfg, dev)
            got.append(gpu_generate(R, other, cfg.n_gen, "plain"))
            R.close()
    except Exception as e:
        errors.append(e)
    t.join()
    P.close()
    time.sleep(0.1)                  # (later tests count the rounds of contexts that are alone)
    assert not errors
    for a in rounds:
        np.testing.assert_array_equal(a[0], ref[0])
        np.testing.assert_array_equal(a[1].view(np.uint32), ref[1].view(np.uint32))
    for a in got:
        np.testing.assert_array_equal(a[0], ref_q[0])
        np.testing.assert_array_equal(a[1].view(np.uint32), ref_q[1].view(np.uint32))


def test_rounds_whose_captures_are_lost_are_run_all_the_same():
    """The caller's own thread synchronises the device beside a decoding one: HIP takes the capture with it (that call may
    fail, which is the caller's to see), the rounds go on."""
    import torch
    cfg = small_cfg("tiny", n_layers=4, exit_layer=2, max_ctx=200, n_gen=12)
    P = binding.PPD(cfg, binding.upload_model(pi.make_model(cfg)))
    prompt = pi.make_prompt(cfg, 20)
    ref = gpu_generate(P, prompt, cfg.n_gen, "ppd")
    done, refused = threading.Event(), [0]

    def synchronise():
        while not done.is_set():
            try:
                torch.cuda.synchronize()
            except RuntimeError:
                refused[0] += 1

    t = threading.Thread(target=synchronise)
    t.start()
    try:
        for i in range(400):
            if i >= 20 and refused[0] >= 3:
                break
            P.ppd_set_sampling(0)
            got = gpu_generate(P, prompt, cfg.n_gen, "ppd")
            np.testing.assert_array_equal(got[0], ref[0])
            np.testing.assert_array_equal(got[1].view(np.uint32), ref[1].view(np.uint32))
    finally:
        done.set()
        t.join()
        P.close()
        time.sleep(0.1)
    assert refused[0] > 0            # (a capture was lost)
