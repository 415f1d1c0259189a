"""Logits buffers.  Memory of the engine's device receives the kernels' own
stores, wherever in a larger buffer it begins; anything else (pinned host
memory) gets the same values by a copy.  The captured decode graph stores
through an address that each call uploads, so buffers of every kind follow one
another on one engine, and a later call leaves an earlier call's buffer alone."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2608_14376_amd import corun
from paper_2608_14376_amd import workload as wl
from tests.gpu_helpers import DEV, to_device

pytestmark = pytest.mark.gpu


def test_prefill_logits_in_pinned_host_memory():
    cfg = wl.config("tiny")
    K, V = wl.make_kv_contiguous(cfg, 2, 64, seed=1, device=DEV)
    eng = corun.Engine(cfg, to_device(wl.make_weights(cfg, seed=0)), 2, K, V,
                       opt=corun.options(max_prefill_len=48))
    prompt = wl.make_prompt(cfg["vocab"], 33, seed=2)
    dev = torch.empty(cfg["vocab"], dtype=torch.float32, device=DEV)
    host = torch.zeros(cfg["vocab"], dtype=torch.float32, pin_memory=True)
    assert eng.prefill(prompt, 0, dev) == eng.prefill(prompt, 1, host)
    assert torch.equal(dev.cpu(), host)
    eng.close()


def test_batched_prefill_logits_in_pinned_host_memory():
    cfg = wl.config("small128")
    K, V = wl.make_kv_contiguous(cfg, 3, 96, seed=3, device=DEV)
    eng = corun.Engine(cfg, to_device(wl.make_weights(cfg, seed=4)), 3, K, V,
                       opt=corun.options(max_prefill_len=200, bi_prefill=True))
    prompts = [wl.make_prompt(cfg["vocab"], n, seed=5 + n) for n in (70, 9, 33)]
    slots = np.array([2, 0, 1], np.int32)
    dev = torch.empty((3, cfg["vocab"]), dtype=torch.float32, device=DEV)
    host = torch.zeros((3, cfg["vocab"]), dtype=torch.float32, pin_memory=True)
    assert np.array_equal(eng.prefill_batch(prompts, slots, dev), eng.prefill_batch(prompts, slots, host))
    assert torch.equal(dev.cpu(), host)
    eng.close()


# lm_head on the pipelined 32- and 64-row tiles, the wide tile, and split
# (the split-K test aid, whose logits are reduced into the engine's buffer)
@pytest.mark.parametrize("B,opt", [(4, {}), (40, {}), (130, {}), (4, dict(split_k_override=2)), (4, dict(no_graph=True))])
def test_decode_logits_buffers_in_turn(B, opt):
    cfg = wl.config("small128")
    V_ = cfg["vocab"]
    K, V = wl.make_kv_contiguous(cfg, B, 32, seed=6, device=DEV)
    eng = corun.Engine(cfg, to_device(wl.make_weights(cfg, seed=7)), B, K, V, opt=corun.options(**opt))
    rng = np.random.default_rng(8)
    tok = rng.integers(0, V_, B).astype(np.int32)
    valid = np.ones(B, np.uint8)
    valid[1] = 0
    pos = np.full(B, 11, np.int32)      # the same step again: each appends the same k, v
    live = torch.from_numpy(valid.astype(bool))
    nxt = np.empty(B, np.int32)

    def step(ptr):
        st = eng._L.corun_decode_step(eng._h, tok.ctypes.data, valid.ctypes.data, pos.ctypes.data, nxt.ctypes.data,
                                      C.c_void_p(ptr))
        assert st == 0, corun.last_error()
        return nxt.copy()

    poison = -12345.0
    first = torch.full((B, V_), poison, device=DEV)
    host = torch.full((B, V_), poison, pin_memory=True)
    odd = torch.full((B * V_ + 9,), poison, device=DEV)   # logits from its second float on
    last = torch.full((B, V_), poison, device=DEV)
    n0 = step(first.data_ptr())
    want = first.cpu()[live]
    assert torch.isfinite(want).all() and (want != poison).any(1).all()
    for buf, ptr in ((first, first.data_ptr()), (host, host.data_ptr()), (None, None), (odd, odd.data_ptr() + 4),
                     (None, None), (last, last.data_ptr())):
        first.fill_(poison)
        torch.cuda.synchronize()
        assert np.array_equal(step(ptr), n0)
        if buf is odd:
            got = odd.cpu()
            assert got[0] == poison and (got[1 + B * V_:] == poison).all()
            assert torch.equal(got[1:1 + B * V_].view(B, V_)[live], want)
        elif buf is not None:
            assert torch.equal(buf.cpu()[live], want)
        if buf is not first:
            assert (first == poison).all()
    eng.decode_run(3, tok, valid, pos)
    assert (first == poison).all() and torch.equal(last.cpu()[live], want)
    eng.close()
