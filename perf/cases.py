"""The work that programs built on this package have it do, as measurable cases.

Every case goes through the package's own entry points (``corun.Engine``): one
padded decode step that also returns its logits (what a sampling server calls
once per token), an isolated prefill of a whole prompt or of one chunk of a
long one, a batched batch-invariant prefill, and a seeded sampler call.  Model
shapes are ``workload.CONFIGS``; the large ones run on a slice of their layers
(two or four), so that rounding differences do not grow with depth and a
case's inputs are quick to make.  Embedding, final norm and lm_head are whole.

Decode batches hold their live requests in the lowest slots, as the package's
scheduler does (it reuses the lowest free slot); the other slots are padding,
whose logits the entry point leaves unspecified, so the logits that come back
are the live rows'.  Greedy tokens are not part of the outputs: they are a
comparison of the logits that do come back, which rounding may tie.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2608_14376_amd import corun
from paper_2608_14376_amd import workload as wl

DEV = "cuda"
PAGE = 16


def listed() -> list:
    return [
        # the smallest call: four requests on the two-layer model that the
        # package's exhaustive tests use; launches and the host path count
        dict(name="decode_tiny_b4", kind="decode", model="tiny", layers=2, batch=4, live=3, lo=16, hi=128),
        # one user talking to an 8B-class model: every weight streamed for one row
        dict(name="decode_8b_b1", kind="decode", model="8b", layers=4, batch=1, live=1, lo=512, hi=4096),
        # a lightly loaded server
        dict(name="decode_8b_b16", kind="decode", model="8b", layers=4, batch=16, live=11, lo=512, hi=4096),
        # the paper's capture size, partly filled: the package's headline benchmark
        dict(name="decode_8b_b256", kind="decode", model="8b", layers=2, batch=256, live=162, lo=512, hi=4096),
        # long contexts on a 32B-class model with a paged cache
        dict(name="decode_32b_paged", kind="decode", model="32b", layers=2, batch=32, live=32, lo=1024, hi=32768,
             paged=True),
        # mixture-of-experts serving
        dict(name="decode_moe_b128", kind="decode", model="moe", layers=2, batch=128, live=81, lo=512, hi=4096),
        # an ordinary chat prompt
        dict(name="prefill_8b_600", kind="prefill", model="8b", layers=4, tokens=600, start=0),
        # a whole long document
        dict(name="prefill_8b_32768", kind="prefill", model="8b", layers=2, tokens=32768, start=0),
        # one fixed-size chunk deep in a long prompt (chunked prefill)
        dict(name="chunk_8b_2048", kind="prefill", model="8b", layers=2, tokens=2048, start=14336),
        # waiting prompts of ragged lengths prefilled in one batch-invariant pass
        dict(name="batch_8b_12", kind="prefill_batch", model="8b", layers=2, prompts=12, lo=100, hi=600),
        # a prompt on the mixture-of-experts model
        dict(name="prefill_moe_3000", kind="prefill", model="moe", layers=2, tokens=3000, start=0),
        # sampling the step's tokens for a full batch, part of it greedy
        dict(name="sample_b256", kind="sample", rows=256, live=162, vocab=151936),
    ]


def _logint(rng, lo: int, hi: int) -> int:
    return int(min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng) -> dict:
    kind = rng.choice(["decode_small", "decode", "decode", "decode_paged", "decode_moe", "prefill", "prefill", "chunk",
                       "batch", "prefill_moe", "sample"])
    if kind == "decode_small":
        b = _logint(rng, 1, 64)
        return dict(kind="decode", model=rng.choice(["tiny", "small128"]), layers=2, batch=b, live=rng.randint(1, b),
                    lo=16, hi=rng.randint(64, 512))
    if kind == "decode":
        b = _logint(rng, 1, 256)
        return dict(kind="decode", model="8b", layers=2, batch=b, live=rng.randint((b + 3) // 4, b), lo=512,
                    hi=rng.randint(1024, 4096))
    if kind == "decode_paged":
        b = rng.randint(4, 32)
        return dict(kind="decode", model="32b", layers=2, batch=b, live=b, lo=1024, hi=_logint(rng, 2048, 32768),
                    paged=True)
    if kind == "decode_moe":
        b = _logint(rng, 1, 128)
        return dict(kind="decode", model="moe", layers=2, batch=b, live=rng.randint((b + 3) // 4, b), lo=512,
                    hi=rng.randint(1024, 4096))
    if kind == "prefill":
        return dict(kind="prefill", model="8b", layers=2, tokens=_logint(rng, 33, 16384), start=0)
    if kind == "chunk":
        c = rng.choice([512, 1024, 2048, 4096])
        return dict(kind="prefill", model="8b", layers=2, tokens=rng.choice([c, rng.randint(c // 2, c)]),
                    start=c * rng.randint(1, 16384 // c - 1))
    if kind == "batch":
        n = rng.randint(2, 24)
        return dict(kind="prefill_batch", model="8b", layers=2, prompts=n, lo=16, hi=rng.randint(64, 8192 // n))
    if kind == "prefill_moe":
        return dict(kind="prefill", model="moe", layers=2, tokens=_logint(rng, 33, 8192), start=0)
    r = _logint(rng, 1, 256)
    return dict(kind="sample", rows=r, live=rng.randint((r + 1) // 2, r), vocab=rng.choice([1024, 151936, 152064]))


# --------------------------------------------------------------------------
# Inputs
# --------------------------------------------------------------------------

def _cfg(case: dict) -> dict:
    if case["kind"] == "sample":   # the sampler needs an engine of the vocabulary, not its layers
        return wl.config("tiny", n_layers=1, vocab=case["vocab"])
    return wl.config(case["model"], n_layers=case["layers"])


def _lens(case: dict, n: int, seed: int) -> np.ndarray:
    """Context or prompt lengths over [lo, hi] in a random order: one from
    each of n equal parts of the range (of its logarithm for the paged
    long-context batches), so that every seed has the same total."""
    lo, hi = case["lo"], case["hi"]
    u = (np.arange(n) + 0.5) / n
    lens = lo * (hi / lo) ** u if case.get("paged") else lo + (hi - lo) * u
    return np.random.default_rng(seed * 31 + 7).permutation(np.round(lens).astype(np.int64))


def _up(n: int, m: int) -> int:
    return (n + m - 1) // m * m


def prepare(case: dict, seed: int) -> dict:
    cfg = _cfg(case)
    rng = np.random.default_rng(seed)
    W = wl.make_weights(cfg, seed=seed, device=DEV)
    st = dict(case=case, cfg=cfg, W=W)
    if case["kind"] == "sample":
        rows, live = case["rows"], case["live"]
        K, V = wl.make_kv_contiguous(cfg, rows, 16, seed + 1, device=DEV)
        g = torch.Generator(device=DEV)
        g.manual_seed(seed)
        st["logits"] = torch.randn((rows, cfg["vocab"]), generator=g, device=DEV) * 2.5
        st["valid"] = (np.arange(rows) < live).astype(np.uint8)
        st["positions"] = rng.integers(1, 4096, rows).astype(np.int32)
        st["seeds"] = rng.integers(0, 2**63, rows).astype(np.uint64)
        st["temperature"] = rng.choice(np.array([0.0, 0.6, 0.6, 0.8, 1.0], np.float32), rows)
        st["eng"] = corun.Engine(cfg, W, rows, K, V)
        return st
    if case["kind"] == "decode":
        B, live = case["batch"], case["live"]
        lens = _lens(case, live, seed)
        st["tokens"] = rng.integers(0, cfg["vocab"], B).astype(np.int32)
        st["valid"] = (np.arange(B) < live).astype(np.uint8)
        st["seq_lens"] = np.zeros(B, np.int32)
        st["seq_lens"][:live] = lens
        st["logits"] = torch.empty((B, cfg["vocab"]), dtype=torch.float32, device=DEV)
        cap = _up(case["hi"] + 128, PAGE)   # room to generate
        if case.get("paged"):
            need = (st["seq_lens"] + 64 + PAGE - 1) // PAGE
            pages = rng.permutation(int(need.sum())).astype(np.int32)
            pt = np.zeros((B, cap // PAGE), np.int32)
            at = 0
            for b in range(B):
                pt[b, :need[b]] = pages[at:at + need[b]]
                at += need[b]
            st["K"], st["V"] = wl.make_kv_paged(cfg, pages.size, PAGE, seed + 1, device=DEV)
            st["pt"] = pt
            st["eng"] = corun.Engine(cfg, W, B, st["K"], st["V"], layout=corun.KV_PAGED, page_size=PAGE,
                                     page_table=torch.from_numpy(pt).to(DEV))
            st["eng"].set_page_table_host(pt)
        else:
            st["K"], st["V"] = wl.make_kv_contiguous(cfg, B, cap, seed + 1, device=DEV)
            st["eng"] = corun.Engine(cfg, W, B, st["K"], st["V"])
        return st
    if case["kind"] == "prefill":
        n, start = case["tokens"], case["start"]
        slots, cap, longest = 4, _up(start + n + 64, PAGE), n
        st["slot"] = int(rng.integers(0, slots))
        st["prompt"] = wl.make_prompt(cfg["vocab"], n, seed)
        st["logits"] = torch.empty(cfg["vocab"], dtype=torch.float32, device=DEV)
    else:
        lens = _lens(case, case["prompts"], seed)
        slots, cap, longest = case["prompts"], _up(case["hi"] + 64, PAGE), int(lens.sum())
        st["slots"] = rng.permutation(slots).astype(np.int32)
        st["prompts"] = [wl.make_prompt(cfg["vocab"], int(m), seed + 100 + i) for i, m in enumerate(lens)]
        st["logits"] = torch.empty((slots, cfg["vocab"]), dtype=torch.float32, device=DEV)
    # a chunk's earlier positions hold the cache of the prompt's earlier chunks
    st["K"], st["V"] = wl.make_kv_contiguous(cfg, slots, cap, seed + 1, device=DEV)
    st["eng"] = corun.Engine(cfg, W, slots, st["K"], st["V"],
                             opt=corun.options(max_prefill_len=longest, bi_prefill=case["kind"] == "prefill_batch"))
    return st


def run(st: dict):
    case, eng = st["case"], st["eng"]
    if case["kind"] == "sample":
        tok, lp = eng.sample(st["logits"], st["valid"], st["positions"], st["seeds"], st["temperature"])
        return {"tokens": tok, "logprobs": lp}
    if case["kind"] == "decode":
        eng.decode_step(st["tokens"], st["valid"], st["seq_lens"], st["logits"])
        return {"logits": st["logits"][:case["live"]], "k": st["K"], "v": st["V"]}
    if case["kind"] == "prefill":
        if case["start"]:
            eng.prefill_chunk(st["prompt"], case["start"], st["slot"], st["logits"])
        else:
            eng.prefill(st["prompt"], st["slot"], st["logits"])
    else:
        eng.prefill_batch(st["prompts"], st["slots"], st["logits"])
    return {"logits": st["logits"], "k": st["K"], "v": st["V"]}


# --------------------------------------------------------------------------
# What a pass cannot do without
# --------------------------------------------------------------------------

def work(case: dict) -> dict:
    """Weights, the cached keys and values that the rows attend to, the
    appended ones, and the logits, each once; multiply-adds of the live rows
    only."""
    c = _cfg(case)
    if case["kind"] == "sample":
        n = case["live"] * case["vocab"]
        return {"bytes": 4 * n + 16 * case["rows"], "flops": 4 * n}
    H, d, nq, nkv, V = c["hidden"], c["head_dim"], c["n_heads"], c["n_kv_heads"], c["vocab"]
    kv_tok = 2 * nkv * d * 2
    if case["kind"] == "decode":
        rows = out_rows = case["live"]
        mean = (case["hi"] - case["lo"]) / math.log(case["hi"] / case["lo"]) if case.get("paged") \
            else (case["lo"] + case["hi"]) / 2
        kv_read, pairs = rows * mean * kv_tok, rows * mean
    elif case["kind"] == "prefill":
        rows, out_rows, p0 = case["tokens"], 1, case["start"]
        kv_read, pairs = p0 * kv_tok, rows * p0 + rows * (rows + 1) / 2
    else:
        n, m = case["prompts"], (case["lo"] + case["hi"]) / 2
        rows, out_rows, kv_read, pairs = n * m, n, 0, n * m * (m + 1) / 2
    attn_w = H * wl.qkv_rows(c) + H * nq * d
    if c["n_experts"]:
        E, k, Fe = c["n_experts"], c["top_k"], c["expert_ffn"]
        touched = E * (1 - (1 - k / E) ** rows)      # experts that some row is routed to, on average
        mlp_w, mlp_f = E * H + touched * 3 * H * Fe, E * H + k * 3 * H * Fe
    else:
        mlp_w = mlp_f = 3 * H * c["ffn"]
    L = c["n_layers"]
    return {"bytes": L * (2 * (attn_w + mlp_w) + kv_read + rows * kv_tok) + 2 * V * H + rows * H * 2 + out_rows * V * 4,
            "flops": L * (2 * rows * (attn_w + mlp_f) + 4 * nq * d * pairs) + 2 * out_rows * V * H}


def tolerance(case: dict):
    """About four times what two correct plans of these kernels differ by:
    the same calls with another split of the projections' sums (split-K
    forced to three, no split-K, the other small-batch layer) gave at most
    0.0052 / 0.032 (2-norm / largest) on two layers and 0.0083 / 0.043 on
    four.  On the mixture of experts such a change also moves single rows to
    another expert where two router logits nearly tie (0.02 / 0.76 with one
    row of 81 moved)."""
    if case["kind"] == "sample":   # fp32 results of fp64 sums; the tokens are decided in fp64
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}
    if case["model"] == "moe":
        return {"rel": 0.03, "max": 0.99}
    return {"rel": 0.03, "max": 0.2} if case["layers"] > 2 else {"rel": 0.02, "max": 0.13}


# --------------------------------------------------------------------------
# The same results in 64 bits
# --------------------------------------------------------------------------

def _store(x, moe: bool):
    """What a stored activation keeps.  Dense models: 64 bits throughout.  A
    mixture of experts rounds to bf16 where the package stores bf16: its
    router compares such values, and in 64 bits would choose other experts."""
    return x.to(torch.float32).to(torch.bfloat16).double() if moe else x


def _rms(x, g, eps):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * g.double()


def _rope(x, pos, theta):
    """x [n, heads, d] rotated at positions pos [n], pairs (i, i + d / 2)."""
    d = x.shape[-1]
    f = theta ** (-2.0 * torch.arange(d // 2, device=x.device, dtype=torch.float64) / d)
    a = pos.double()[:, None] * f[None, :]
    cs, sn = a.cos()[:, None, :], a.sin()[:, None, :]
    x1, x2 = x[..., :d // 2], x[..., d // 2:]
    return torch.cat([x1 * cs - x2 * sn, x2 * cs + x1 * sn], -1)


def _layers(c: dict, W, tokens, pos, attend):
    """The residual after every layer for rows `tokens` at positions `pos`;
    attend(layer, q, k, v) appends k, v and returns the attention output."""
    d, nq, nkv, eps = c["head_dim"], c["n_heads"], c["n_kv_heads"], c["rms_eps"]
    moe = c["n_experts"] > 0
    n = tokens.numel()
    x = W.embed[tokens].double()
    for l in range(c["n_layers"]):
        h = _store(_rms(x, W.attn_norm[l], eps), moe)
        y = _store(h @ W.w_qkv[l].double().t(), moe).view(n, nq + 2 * nkv, d)
        q = _store(_rope(y[:, :nq], pos, c["rope_theta"]), moe)
        k = _store(_rope(y[:, nq:nq + nkv], pos, c["rope_theta"]), moe)
        o = _store(attend(l, q, k, y[:, nq + nkv:]), moe)
        x = x + o.reshape(n, nq * d) @ W.w_o[l].double().t()
        h = _store(_rms(x, W.mlp_norm[l], eps), moe)
        if not moe:
            for r in range(0, n, 4096):   # rows in blocks, for memory
                y = h[r:r + 4096] @ W.w_gate_up[l].double().t()
                a = torch.nn.functional.silu(y[:, :c["ffn"]]) * y[:, c["ffn"]:]
                x[r:r + 4096] += a @ W.w_down[l].double().t()
            continue
        Fe, top = c["expert_ffn"], c["top_k"]
        lg, sel = torch.topk(h @ W.w_router[l].double().t(), top, dim=-1)
        w = torch.softmax(lg, -1)
        add = torch.zeros_like(x)
        for e in range(c["n_experts"]):
            row, rank = (sel == e).nonzero(as_tuple=True)
            if row.numel():
                y = _store(h[row] @ W.w_exp_gate_up[l][e].double().t(), moe)
                a = _store(torch.nn.functional.silu(y[:, :Fe]) * y[:, Fe:], moe)
                add.index_add_(0, row, w[row, rank][:, None] * (a @ W.w_exp_down[l][e].double().t()))
        x = x + add
    return x


def _causal(q, k, v, p0: int):
    """q [n, nq, d] at positions p0 .. against k, v [p0 + n, nkv, d]."""
    n, nq, d = q.shape
    nkv = k.shape[1]
    G = nq // nkv
    out = torch.empty_like(q)
    for g in range(nkv):
        kg, vg = k[:, g].contiguous(), v[:, g].contiguous()
        for r in range(0, n, 1024):
            m = min(1024, n - r)
            T = p0 + r + m
            qs = q[r:r + m, g * G:(g + 1) * G].reshape(m * G, d)
            s = (qs @ kg[:T].t().contiguous()) / math.sqrt(d)
            at = torch.arange(p0 + r, p0 + r + m, device=q.device).repeat_interleave(G)
            s.masked_fill_(torch.arange(T, device=q.device)[None, :] > at[:, None], -math.inf)
            out[r:r + m, g * G:(g + 1) * G] = (torch.softmax(s, -1) @ vg[:T]).view(m, G, d)
            del s
    return out


def _exact_sample(st: dict):
    """argmax of l / T + g, g = -ln(-ln u), u from Philox4x32-10 (Salmon et
    al., SC 2011) keyed by the row's seed at counter (position, column, 0, 0);
    the log-probability of the chosen column."""
    n, V = st["logits"].shape
    mask = 0xFFFFFFFF
    tokens, lps = np.full(n, -1, np.int32), np.zeros(n)
    for r in range(n):
        if not st["valid"][r]:
            continue
        T = float(st["temperature"][r])
        x = st["logits"][r].double() / (T if T > 0 else 1.0)
        z = x
        if T > 0:
            sd = int(st["seeds"][r])
            k0, k1 = sd & mask, sd >> 32
            c1 = torch.arange(V, device=DEV)
            c0, c2, c3 = torch.full_like(c1, int(st["positions"][r])), torch.zeros_like(c1), torch.zeros_like(c1)
            for _ in range(10):
                a, b = c0 * 0xD2511F53, c2 * 0xCD9E8D57
                c0, c1, c2, c3 = ((b >> 32) & mask) ^ c1 ^ k0, b & mask, ((a >> 32) & mask) ^ c3 ^ k1, a & mask
                k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
            u = ((c0 >> 6).double() * 67108864.0 + (c1 >> 6).double() + 0.5) * 2.0 ** -52
            z = x - torch.log(-torch.log(u))
        tokens[r] = int(z.argmax())
        lps[r] = float(torch.log_softmax(x, 0)[int(tokens[r])])
    return {"tokens": tokens, "logprobs": lps}


def exact(case: dict, seed: int):
    st = prepare(case, seed)
    st.pop("eng").close()
    if case["kind"] == "sample":
        return _exact_sample(st)
    c, W = st["cfg"], st["W"]
    nq, nkv, d = c["n_heads"], c["n_kv_heads"], c["head_dim"]
    K, V = [t.double() for t in st.pop("K")], [t.double() for t in st.pop("V")]
    if case["kind"] == "decode":
        live = case["live"]
        tokens = torch.from_numpy(st["tokens"][:live]).to(DEV).long()
        lens = st["seq_lens"][:live]

        def attend(l, q, k, v):
            out = torch.empty_like(q)
            for b in range(live):
                n = int(lens[b])
                if case.get("paged"):
                    pg = torch.from_numpy(st["pt"][b, :n // PAGE + 1]).to(DEV).long()
                    K[l][pg[-1], :, n % PAGE], V[l][pg[-1], :, n % PAGE] = k[b], v[b]
                    kb, vb = (t[l][pg].transpose(0, 1).reshape(nkv, -1, d)[:, :n + 1] for t in (K, V))
                else:
                    K[l][b, :, n], V[l][b, :, n] = k[b], v[b]
                    kb, vb = K[l][b, :, :n + 1], V[l][b, :, :n + 1]
                s = (q[b].view(nkv, nq // nkv, d) @ kb.transpose(1, 2).contiguous()) / math.sqrt(d)
                out[b] = (torch.softmax(s, -1) @ vb.contiguous()).reshape(nq, d)
            return out

        x = _layers(c, W, tokens, torch.from_numpy(lens).to(DEV), attend)
    else:
        one = case["kind"] == "prefill"
        prompts = [st["prompt"]] if one else st["prompts"]
        slots = [st["slot"]] if one else st["slots"].tolist()
        p0 = case.get("start", 0)
        ends = []
        for p, slot in zip(prompts, slots):
            n = p.size

            def attend(l, q, k, v):
                K[l][slot, :, p0:p0 + n], V[l][slot, :, p0:p0 + n] = k.transpose(0, 1), v.transpose(0, 1)
                return _causal(q, K[l][slot, :, :p0 + n].transpose(0, 1), V[l][slot, :, :p0 + n].transpose(0, 1), p0)

            ends.append(_layers(c, W, torch.from_numpy(p).to(DEV).long(),
                                torch.arange(p0, p0 + n, device=DEV), attend)[-1:])
        x = torch.cat(ends)
    h = _store(_rms(x, W.final_norm, c["rms_eps"]), c["n_experts"] > 0)
    lm = torch.cat([h @ W.lm_head[r:r + 16384].double().t() for r in range(0, c["vocab"], 16384)], 1)
    return {"logits": lm[0] if case["kind"] == "prefill" else lm, "k": K, "v": V}
