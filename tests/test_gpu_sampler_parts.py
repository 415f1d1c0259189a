"""The sampler's row parts (4 ceil(V / 65536) of a multiple of 256 columns) and
the test that spares most columns their fp64 logarithms: vocabularies at the
parts' edges, masked (-inf) columns and parts, ties, flat rows, huge and tiny
temperatures and logits, against the oracle; the scratch-free form gives the
same bits."""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_14376_amd import corun
from paper_2608_14376_amd import workload as wl
from tests.gpu_helpers import DEV, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab", [16, 256, 272, 1024, 1040, 16368, 16384, 16400, 32768, 49168, 65536, 65552])
def test_parts_match_the_oracle(vocab):
    cfg = wl.config("tiny", n_layers=1, vocab=vocab)
    Wg = to_device(wl.make_weights(cfg, seed=95))
    rows = 14
    K, V = wl.make_kv_contiguous(cfg, rows, 16, seed=96, device=DEV)
    eng = corun.Engine(cfg, Wg, rows, K, V)
    rng = np.random.default_rng(vocab)
    l = rng.normal(0, 2.5, (rows, vocab)).astype(np.float32)
    ninf = np.float32(-np.inf)
    l[1] = 0.25                                       # flat: every column can win
    l[2, : vocab - 1] = ninf                          # only the last column is left
    l[3, vocab // 3:] = ninf                          # later parts masked whole
    l[4, : 2 * vocab // 3] = ninf                     # earlier ones
    l[5] = np.round(l[5])                             # ties
    l[6] *= 1e5
    l[7] *= 1e-6
    l[8] = np.finfo(np.float32).min                   # a mask of the type's lowest value
    l[8, vocab // 2] = 1.0
    l[9] = np.sort(l[9])                              # every column beats the ones before it
    T = np.array([0.6, 1.0, 0.7, 0.6, 1.3, 0.8, 1.0, 1.0, 0.6, 1.0, 1e-6, 1e4, 0.0, -1.0], np.float32)
    valid = np.ones(rows, np.uint8)
    pos = rng.integers(0, 1 << 20, rows).astype(np.int32)
    seeds = rng.integers(0, 1 << 63, rows, dtype=np.uint64)
    x = torch.from_numpy(l).to(DEV)
    tok, lp = eng.sample(x, valid, pos, seeds, T)
    for r in range(rows):
        ot, olp = oracle.sample(l[r], int(seeds[r]), int(pos[r]), float(T[r]))
        assert tok[r] == ot, (r, tok[r], ot)
        # fp32 result of fp64 sums
        assert abs(float(lp[r]) - olp) <= 1e-6 * max(1.0, abs(olp)), (r, lp[r], olp)
    tok2, lp2 = corun.sample_noalloc(x, valid, pos, seeds, T)
    assert np.array_equal(tok, tok2) and np.array_equal(lp.view(np.int32), lp2.view(np.int32))
    eng.close()


def test_nan_reaches_the_log_probability():
    """A NaN column never wins, but the row's log-probability is NaN wherever
    it stands: in a part of nothing else, of -inf besides, or of finite
    columns; -inf alone is only weightless.  Sampled and greedy rows."""
    vocab, part = 65520, 16384
    cfg = wl.config("tiny", n_layers=1, vocab=vocab)
    nan, ninf = np.float32(np.nan), np.float32(-np.inf)
    rng = np.random.default_rng(97)
    l = np.tile(rng.normal(0, 2.5, vocab).astype(np.float32), (10, 1))
    for r in (0, 5):
        l[r, part: 2 * part] = nan                    # a part of NaN
        l[r + 1, part: 2 * part] = ninf               # of -inf and one NaN
        l[r + 1, part + 777] = nan
        l[r + 2, 2 * part + 5] = nan                  # of finite columns and one NaN
        l[r + 3, 3 * part:] = nan                     # the short last part
        l[r + 4, part: 2 * part] = ninf               # no NaN
    rows = len(l)
    T = np.array([0.7] * 5 + [0.0] * 5, np.float32)
    valid, pos = np.ones(rows, np.uint8), np.arange(rows, dtype=np.int32)
    seeds = rng.integers(0, 1 << 63, rows, dtype=np.uint64)
    K, V = wl.make_kv_contiguous(cfg, rows, 16, seed=98, device=DEV)
    eng = corun.Engine(cfg, to_device(wl.make_weights(cfg, seed=99)), rows, K, V)
    x = torch.from_numpy(l).to(DEV)
    for tok, lp in (eng.sample(x, valid, pos, seeds, T), corun.sample_noalloc(x, valid, pos, seeds, T)):
        for r in range(rows):
            # without the NaN columns: the same winner
            ot, olp = oracle.sample(np.where(np.isnan(l[r]), ninf, l[r]), int(seeds[r]), int(pos[r]), float(T[r]))
            assert tok[r] == ot, (r, tok[r], ot)
            if np.isnan(l[r]).any():
                assert np.isnan(lp[r]), (r, lp[r])
            else:
                assert abs(float(lp[r]) - olp) <= 1e-6 * max(1.0, abs(olp)), (r, lp[r], olp)
    eng.close()


@pytest.mark.parametrize("T", [1e-12, 1e-13, 1e-14, 1e-15])
def test_tiny_temperatures_on_flat_rows(T):
    """Equal logits over a temperature so small that the noise is a few units
    of l / T's last place: every column's score counts, and ties go to the
    earlier column."""
    vocab, rows = 400, 512
    cfg = wl.config("tiny", n_layers=1, vocab=vocab)
    rng = np.random.default_rng(101)
    l = np.repeat(rng.uniform(1, 20, rows).astype(np.float32)[:, None], vocab, 1)
    valid, pos = np.ones(rows, np.uint8), rng.integers(0, 1 << 20, rows).astype(np.int32)
    seeds = rng.integers(0, 1 << 63, rows, dtype=np.uint64)
    K, V = wl.make_kv_contiguous(cfg, rows, 16, seed=102, device=DEV)
    eng = corun.Engine(cfg, to_device(wl.make_weights(cfg, seed=103)), rows, K, V)
    tok, lp = eng.sample(torch.from_numpy(l).to(DEV), valid, pos, seeds, np.full(rows, T, np.float32))
    want = [oracle.sample(l[r], int(seeds[r]), int(pos[r]), float(np.float32(T))) for r in range(rows)]
    assert [int(t) for t in tok] == [t for t, _ in want]
    assert np.allclose(lp, [p for _, p in want], rtol=1e-6, atol=0)
    eng.close()
