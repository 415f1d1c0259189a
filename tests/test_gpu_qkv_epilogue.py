"""The QKV epilogue inside the wide projection tiles (heads of 128, more than
64 rows, no split-K): q rotated, k and v placed in the cache by the projection.

Every path runs the same arithmetic on the same fp32 sums, so a prompt gives
bit-identical keys, values and logits whether its cache is contiguous or paged
(pages in a random order), at the row counts around the tiles' edges, and
whether it is prefilled alone or among others; 64 rows, on the separate
epilogue kernel, agree with the same positions of the longer prompts.
"""
import numpy as np
import pytest
import torch

from paper_2608_14376_amd import corun
from paper_2608_14376_amd import workload as wl
from tests.gpu_helpers import DEV, to_device

pytestmark = pytest.mark.gpu
PAGE, CAP, SLOTS = 16, 400, 3


def _bits(t):
    return t.contiguous().view(torch.int16)


@pytest.mark.parametrize("n", [64, 65, 128, 129, 257, 321, 385])
def test_paged_and_batched_against_contiguous(n):
    cfg = wl.config("small128")
    W = to_device(wl.make_weights(cfg, seed=91))
    opt = lambda rows: corun.options(max_prefill_len=rows, bi_prefill=True)
    prompts = [wl.make_prompt(cfg["vocab"], m, seed=92 + i) for i, m in enumerate((n, 33, 70))]
    alone, paged = (torch.empty(cfg["vocab"], dtype=torch.float32, device=DEV) for _ in range(2))
    batch = torch.empty((3, cfg["vocab"]), dtype=torch.float32, device=DEV)

    K, V = wl.make_kv_contiguous(cfg, SLOTS, CAP, seed=95, device=DEV)
    eng = corun.Engine(cfg, W, SLOTS, K, V, opt=opt(n))
    eng.prefill(prompts[0], 1, alone)
    eng.close()

    pages = np.random.default_rng(96).permutation(SLOTS * CAP // PAGE).astype(np.int32).reshape(SLOTS, -1)
    Kp, Vp = wl.make_kv_paged(cfg, pages.size, PAGE, 97, device=DEV)
    eng = corun.Engine(cfg, W, SLOTS, Kp, Vp, opt=opt(n), layout=corun.KV_PAGED, page_size=PAGE,
                       page_table=torch.from_numpy(pages).to(DEV))
    eng.set_page_table_host(pages)
    eng.prefill(prompts[0], 2, paged)
    eng.close()
    assert torch.equal(alone, paged)
    row = torch.from_numpy(pages[2]).to(DEV).long()
    for a, b in zip(K + V, Kp + Vp):
        flat = b[row].transpose(0, 1).reshape(cfg["n_kv_heads"], -1, cfg["head_dim"])
        assert torch.equal(_bits(a[1, :, :n]), _bits(flat[:, :n]))

    Kb, Vb = wl.make_kv_contiguous(cfg, SLOTS, CAP, seed=98, device=DEV)
    eng = corun.Engine(cfg, W, SLOTS, Kb, Vb, opt=opt(n + 103))
    eng.prefill_batch(prompts, np.array([2, 0, 1], np.int32), batch)
    eng.close()
    assert torch.equal(alone, batch[0])
    for a, b in zip(K + V, Kb + Vb):
        assert torch.equal(_bits(a[1, :, :n]), _bits(b[2, :, :n]))
