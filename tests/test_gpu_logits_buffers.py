"""Logits buffers that are not memory of the engine's device (pinned host
memory) receive the same values as a device buffer, by a copy."""
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
