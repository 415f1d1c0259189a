"""The wide projection tiles (more than 64 rows) and the prefill expert tiles
at their edges.

With batch-invariant prefill every projection output is one MFMA chain over K
in order, whatever tile it is computed in, and causal attention gives a
position the same bits whatever follows it.  So the k, v of a prompt's first n
positions are bit-identical whether the prompt is prefilled at n tokens or
longer.  The small models run the 64- and 128-row tiles and the expert tiles
(16, 64, 128 rows; two-launch dispatch above 2048 assignments) at row counts
around their edges; a model 4096 wide runs every tile, with one row or all but
one of its last row tile and half or a quarter of its last column tile.
Against the oracle: relative 2e-2 on the last logits.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_14376_amd import corun
from paper_2608_14376_amd import workload as wl
from tests.gpu_helpers import DEV, check_routing, host_model, oracle_kv, row_rel_err, to_device

pytestmark = pytest.mark.gpu
TOL = 2e-2
LENS = {"small128": (1, 64, 65, 127, 128, 129, 255, 256, 257, 319, 320, 321, 640, 641),
        "small_moe": (31, 32, 33, 95, 96, 97, 512, 513),
        # 64 experts of 4 assignments a row over 18 column tiles: 16-row expert
        # tiles to 128 rows (8 per expert), 64-row ones to 384, 128-row ones above
        "moe64": (33, 127, 128, 129, 200, 383, 384, 385, 513)}
CONFIGS = {"moe64": dict(n_experts=64, hidden=2048)}
LONGEST = 700


@pytest.mark.parametrize("name", sorted(LENS))
def test_prefix_bits_at_the_tile_edges(name):
    cfg = wl.config("small_moe", **CONFIGS[name]) if name in CONFIGS else wl.config(name)
    Wc = wl.make_weights(cfg, seed=81)
    Wg = to_device(Wc)
    K, V = wl.make_kv_contiguous(cfg, 2, 704, seed=82)
    Kd, Vd = [k.to(DEV) for k in K], [v.to(DEV) for v in V]
    eng = corun.Engine(cfg, Wg, 2, Kd, Vd, opt=corun.options(max_prefill_len=LONGEST, bi_prefill=True,
                                                             record_routing=cfg["n_experts"] > 0))
    prompt = wl.make_prompt(cfg["vocab"], LONGEST, seed=83)
    last = torch.empty(cfg["vocab"], dtype=torch.float32, device=DEV)
    eng.prefill(prompt, 0, last)
    for n in LENS[name]:
        for c in Kd + Vd:
            c[1].zero_()
        eng.prefill(prompt[:n], 1)
        for l in range(cfg["n_layers"]):
            for c in (Kd[l], Vd[l]):
                assert torch.equal(c[1, :, :n].view(torch.int16), c[0, :, :n].view(torch.int16)), (n, l)

    m = host_model(Wc)
    okv = oracle_kv(K, V)
    if cfg["n_experts"]:
        eng.prefill(prompt[:200], 1, last)
        sel, glog = eng.routing_trace(1)
        ref, _, rl, own = oracle.prefill_routed(m, okv, 1, prompt[:200], force=sel)
        for t in range(200):
            check_routing(sel[:, t], glog[:, t], rl[:, t], own[:, t], t)
    else:
        ref, _ = oracle.prefill(m, okv, 1, prompt[:321])
        eng.prefill(prompt[:321], 1, last)
    assert row_rel_err(last.cpu().numpy(), ref) <= TOL
    eng.close()


@pytest.mark.parametrize("n", [129, 257, 321, 500])
def test_default_plan_against_the_oracle(n):
    """The default prefill plan (split-K where the estimate asks for it) at
    lengths that pick different wide tiles."""
    cfg = wl.config("small128", n_layers=1, ffn=6144)
    Wc = wl.make_weights(cfg, seed=84)
    Wg = to_device(Wc)
    K, V = wl.make_kv_contiguous(cfg, 1, 512, seed=85)
    eng = corun.Engine(cfg, Wg, 1, [k.to(DEV) for k in K], [v.to(DEV) for v in V],
                       opt=corun.options(max_prefill_len=n))
    prompt = wl.make_prompt(cfg["vocab"], n, seed=86)
    last = torch.empty(cfg["vocab"], dtype=torch.float32, device=DEV)
    eng.prefill(prompt, 0, last)
    ref, _ = oracle.prefill(host_model(Wc), oracle_kv(K, V), 0, prompt)
    assert row_rel_err(last.cpu().numpy(), ref) <= TOL
    eng.close()


@pytest.mark.parametrize("ffn", [64, 128, 192, 256, 320])
def test_chains_shorter_than_the_ring(ffn):
    """The down projection over one to five 64-element stages, on rings of
    four (128 x 128), three (256 x 128) and two (256 x 256) stages: chains that
    end before the ring is full, with its last slot and one or two later.  The
    k, v of layer 1 carry layer 0's down products; the 64-row tile, another
    kernel, gives the bits."""
    cfg = wl.config("small128", hidden=2048, ffn=ffn)
    opt = corun.options(max_prefill_len=4100, bi_prefill=True)
    tiles = {64: (64, 128), 129: (128, 128), 2050: (256, 128), 4100: (256, 256)}
    for n, t in tiles.items():
        p = corun.describe_prefill_plan(cfg, n, opt)["down"]
        assert (p["m_tile"], p["n_tile"], p["split_k"]) == (*t, 1), (n, p)
    W = to_device(wl.make_weights(cfg, seed=87))
    K, V = wl.make_kv_contiguous(cfg, 2, 4112, seed=88, device=DEV)
    eng = corun.Engine(cfg, W, 2, K, V, opt=opt)
    prompt = wl.make_prompt(cfg["vocab"], 4100, seed=89)
    eng.prefill(prompt, 0)
    for n in (64, 129, 2050):
        for c in K + V:
            c[1].zero_()
        eng.prefill(prompt[:n], 1)
        for c in (K[1], V[1]):
            assert torch.equal(c[1, :, :n].view(torch.int16), c[0, :, :n].view(torch.int16)), n
    eng.close()


# rows: tile of qkv for heads of 128 and of 64, of o and down, of gate/up
WIDE = {64: ((64, 128), (64, 128), (64, 128), (64, 128)),
        65: ((128, 128), (128, 128), (128, 128), (128, 128)),
        257: ((128, 128), (128, 128), (128, 128), (256, 256)),
        641: ((256, 128), (128, 128), (128, 128), (256, 128)),
        897: ((256, 128), (256, 128), (128, 128), (256, 128)),
        1537: ((256, 256), (256, 256), (256, 128), (320, 256)),
        2049: ((256, 256), (256, 256), (256, 256), (320, 256)),
        2881: ((320, 256), (256, 256), (256, 256), (320, 256)),
        3199: ((320, 256), (320, 256), (256, 256), (320, 256)),
        4161: ((256, 128), (256, 128), (320, 256), (256, 256)),
        4479: ((256, 256), (256, 128), (320, 256), (320, 256))}


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("head_dim", [128, 64])
def test_every_wide_tile(head_dim, paged):
    """The QKV epilogue (heads of 128) or fp32 sums (64) over column counts of
    22.5 and 20.25 tiles of 256, SwiGLU over 86.5, fp32 sums of o and down: k, v
    of both layers against the longest prompt's, in another slot, paged on
    another cache layout, contiguous also as a batch of prompts."""
    heads = 15 if head_dim == 128 else 27
    cfg = wl.config("small128", hidden=4096, n_heads=heads, n_kv_heads=heads, head_dim=head_dim, ffn=11072)
    longest, cap, page = max(WIDE), 4480, 16
    opt = corun.options(max_prefill_len=longest, bi_prefill=True)
    for n, (qkv128, qkv64, odown, gu) in WIDE.items():
        p = corun.describe_prefill_plan(cfg, n, opt)
        want = {"qkv": qkv128 if head_dim == 128 else qkv64, "o": odown, "down": odown, "gate_up": gu}
        assert {k: (p[k]["m_tile"], p[k]["n_tile"]) for k in want} == want, n
    W = wl.make_weights(cfg, seed=104, device=DEV)
    prompt = wl.make_prompt(cfg["vocab"], longest, seed=105)
    K, V = wl.make_kv_contiguous(cfg, 4, cap, seed=106, device=DEV)
    eng = corun.Engine(cfg, W, 4, K, V, opt=opt)
    eng.prefill(prompt, 0)
    if not paged:   # 2881 rows of three prompts, each in its own slot
        lens = (1500, 881, 500)
        eng.prefill_batch([prompt[:n] for n in lens], np.array([2, 1, 3], np.int32))
        for n, slot in zip(lens, (2, 1, 3)):
            for c in K + V:
                assert torch.equal(c[slot, :, :n].view(torch.int16), c[0, :, :n].view(torch.int16)), (n, slot)
    else:
        eng.close()
        pages = np.random.default_rng(107).permutation(2 * cap // page).astype(np.int32).reshape(2, -1)
        Kp, Vp = wl.make_kv_paged(cfg, pages.size, page, 108, device=DEV)
        eng = corun.Engine(cfg, W, 2, Kp, Vp, opt=opt, layout=corun.KV_PAGED, page_size=page,
                           page_table=torch.from_numpy(pages).to(DEV))
        eng.set_page_table_host(pages)
        row = torch.from_numpy(pages[1]).to(DEV).long()
    for n in WIDE:
        for c in Kp + Vp if paged else [x[1] for x in K + V]:
            c.zero_()
        eng.prefill(prompt[:n], 1)
        for i, ref in enumerate(K + V):
            got = (Kp + Vp)[i][row].transpose(0, 1).reshape(heads, -1, head_dim) if paged else ref[1]
            assert torch.equal(got[:, :n].contiguous().view(torch.int16),
                               ref[0, :, :n].contiguous().view(torch.int16)), (n, i)
    eng.close()
