"""The forms of the decode projections at the row counts where they change: operand tiles of 8 (hi and lo in one tile), 16,
32 rows and, for the LM head, 48 and 64, the single kernel against the split one with its finishing pass (a layer whose W1/W3 and W2 lie just
beyond the line between them at three rows: 2052 feature tiles, 513 k-tiles), the prefill kernels' 32-token blocks beyond 32
rows, and the LM head's passes of 64 rows.  Gate: the suite's per-type tolerance; the hi + lo operands keep decode steps well below it."""
import numpy as np
import pytest
import torch

from oracle import stage_oracle as so
from tests.helpers import TOL, check, gpu_decode, gpu_prefill, make_gpu_stage, make_oracle
from workloads import StageConfig, generate

pytestmark = pytest.mark.gpu

WIDE = StageConfig("wide", "bf16", 4096, 32, 8, 16416, 1, 1, (0,), batch=1, seed=801)
NARROW = StageConfig("narrow", "f16", 512, 8, 2, 1472, 2, 2, (1,), batch=1, seed=802)      # W_O: 8 k-tiles, W2: 23
# the single kernel's blocks of two units: QKV 352 feature tiles, W_O and W2 288 (beyond 16 rows up to 108 k-tiles, longer ones are split:
# HALVED has 72 each), W1/W3 290 gate / up pairs; and W1/W3 at 772
PAIRS = StageConfig("pairs", "bf16", 4608, 36, 4, 4640, 1, 1, (0,), batch=1, seed=806)
HALVED = StageConfig("halved", "bf16", 4608, 36, 4, 4608, 1, 2, (1,), batch=1, seed=808)
# ... and few blocks whose contraction is too long for one kernel (GATED: W2, 386 k-tiles for 64 units)
GATED = StageConfig("gated", "f16", 1024, 8, 2, 12352, 2, 1, (0,), batch=1, seed=807)
_sides = {}


def _side(cfg):
    if cfg.name not in _sides:
        w = [generate.layer_weights(cfg, l) for l in range(cfg.n_layers)]
        _sides[cfg.name] = make_oracle(cfg, cfg.tp_ranks[0], w), make_gpu_stage(cfg, cfg.tp_ranks[0], w)
    return _sides[cfg.name]


@pytest.mark.parametrize("cfg,rows", [(WIDE, t) for t in (3, 8, 9, 17, 32, 33, 64, 65)] + [(NARROW, t) for t in (3, 9, 16, 31, 33, 64, 65, 97)] +
                         [(PAIRS, t) for t in (1, 2, 3, 8, 9, 16, 17, 32)] + [(GATED, t) for t in (1, 2, 3, 9, 17)] + [(HALVED, t) for t in (17, 32)],
                         ids=lambda v: getattr(v, "name", v))
def test_decode_step(cfg, rows):
    print(cfg.name, rows, flush=True)
    ora, st = _side(cfg)
    lens = [1 + (i * 7) % 5 for i in range(rows)]
    X = generate.hidden_rows(cfg, sum(lens))
    oc = ora.new_cache(rows)
    kv = st.kv_cache_create(rows, 16)
    ora.prefill(oc, X, lens)
    gpu_prefill(st, kv, cfg, X, lens)
    for i in range(rows):                       # the steps start from the very rows the GPU holds
        for l in range(cfg.n_layers):
            k, v = kv.read(l, i, 0, lens[i])
            oc.fill(l, i, k, v)
    for k in range(2):
        x = generate.hidden_rows(cfg, rows, stream_id=1 + k)
        p_ref, h_ref = ora.decode(oc, x)
        p, h = gpu_decode(st, kv, cfg, k, x)
        check(f"{rows} rows step {k} resid", h, h_ref, TOL[cfg.dtype])
        check(f"{rows} rows step {k} partial", p, p_ref, TOL[cfg.dtype])


@pytest.mark.parametrize("cfg,rows", [(NARROW, 35), (NARROW, 128), (NARROW, 129), (WIDE, 64), (WIDE, 65), (WIDE, 129)], ids=lambda v: getattr(v, "name", v))
def test_decode_rows_around_position_tiles(cfg, rows):
    """More than 32 sequences: the attention finishes the QKV projection (up to 128 rows and 512 (row, kv head) pairs, beyond
    that the projection does) and appends the new row, at contexts on both sides of the 32-position tiles and of the 8 tiles that its waves take in one go."""
    print(cfg.name, rows, flush=True)
    ora, st = _side(cfg)
    edge = (1, 31, 32, 33, 63, 64, 255, 256, 257, 290)
    lens = [edge[i % len(edge)] for i in range(rows)]
    oc = ora.new_cache(rows)
    kv = st.kv_cache_create(rows, 320)
    for l in range(cfg.n_layers):
        for i in range(rows):
            k, v = generate.synthetic_kv(cfg, l, i, lens[i])
            kv.fill(l, i, k, v)
            oc.fill(l, i, k, v)
    kv.set_lengths(lens)
    for k in range(2):
        x = generate.hidden_rows(cfg, rows, stream_id=1 + k)
        p_ref, h_ref = ora.decode(oc, x)
        p, hh = gpu_decode(st, kv, cfg, k, x)
        check(f"{rows} rows step {k} resid", hh, h_ref, TOL[cfg.dtype])
        check(f"{rows} rows step {k} partial", p, p_ref, TOL[cfg.dtype])


@pytest.mark.parametrize("hidden,vocab,rows", [(128, 1000, 40), (1024, 1000, 20), (4096, 1000, 20), (2048, 3208, 17), (2048, 3208, 32), (1024, 4104, 33), (1024, 4104, 48), (1024, 4104, 49), (1024, 4104, 64), (1024, 4104, 65)] +
                         # units of two tiles (from 1024 tiles on) and columns beyond the last: one kernel at 7, 9 and 17 rows, split at 17 of a short contraction and from 33 on
                         [(1536, 16411, 7), (1536, 16411, 9), (1536, 16411, 17), (1024, 16411, 17), (1024, 16411, 32), (1024, 16411, 48), (1024, 16411, 64)])
def test_head_rows(hidden, vocab, rows):
    import paper_2311_11514_amd as hx
    cfg = StageConfig("headrows", "bf16", hidden, 8, 8, 64, 1, 1, (0,), batch=1, seed=803, vocab=vocab)
    hw = generate.head_weights(cfg)
    hd = hx.Head(hidden, vocab, 1, 0, "bf16", cfg.rms_eps)
    hd.load(hw["g_final"].cuda(), hw["w_lm"].cuda())
    a, b = (generate.hidden_rows(cfg, rows, stream_id=s).to(torch.bfloat16) for s in (3, 4))
    tok, val = hd.greedy(a.cuda(), b.cuda())
    torch.cuda.synchronize()
    logits = so.rmsnorm(a.double().numpy() + b.double().numpy(), hw["g_final"].double().numpy(), cfg.rms_eps) @ hw["w_lm"].double().numpy()
    top = np.sort(logits, axis=1)
    # the operands carry 16 mantissa bits: a logit is off by about 2^-17 of the row's scale
    assert np.max(np.abs(val.cpu().numpy() - top[:, -1]) / np.abs(top[:, -1])) < 2e-4
    clear = top[:, -1] - top[:, -2] > 1e-3 * np.abs(top[:, -1])
    assert clear.mean() > 0.8 and np.array_equal(tok.cpu().numpy()[clear], np.argmax(logits, axis=1)[clear])


@pytest.mark.parametrize("rows,vocab", [(1, 4104), (5, 4104), (40, 4104), (2, 16411), (7, 16411), (17, 16411), (48, 16411)])
def test_head_ties_and_rows_that_are_not_finite(rows, vocab):
    """The lowest id wins an exact tie wherever the tied columns lie (with units of two tiles also in either tile of one unit); a row
    of NaN has no candidate: the shard's first id."""
    import paper_2311_11514_amd as hx
    hidden, end = 1024, vocab - 4
    cfg = StageConfig("headties", "bf16", hidden, 8, 8, 64, 1, 1, (0,), batch=1, seed=804, vocab=vocab)
    hw = generate.head_weights(cfg)
    w, a = hw["w_lm"].clone(), generate.hidden_rows(cfg, rows, stream_id=3).to(torch.bfloat16)
    best = torch.argmax((a.double() * hw["g_final"].double()) @ w.double(), dim=1)
    w[:, end] = w[:, 7]
    for i in range(rows):                                   # every row's best column once more, in a tile of its own ...
        w[:, (int(best[i]) + 1000) % 4000] = w[:, int(best[i])]
        if vocab > 16384:                                   # ... and in the other tile of its unit
            w[:, min(int(best[i]) ^ 16, vocab - 1)] = w[:, int(best[i])]
    first = torch.argmax((a.double() * hw["g_final"].double()) @ w.double(), dim=1)
    hd = hx.Head(hidden, vocab, 1, 0, "bf16", cfg.rms_eps)
    hd.load(hw["g_final"].cuda(), w.cuda())
    tok, val = hd.greedy(a.cuda())
    torch.cuda.synchronize()
    same = [torch.equal(w[:, int(t)], w[:, int(f)]) for t, f in zip(tok.cpu(), first)]
    assert all(int(t) == int(f) for t, f, s in zip(tok.cpu(), first, same) if s) and np.mean(same) > 0.8
    a[0] = float("nan")
    tok2, val2 = hd.greedy(a.cuda())
    torch.cuda.synchronize()
    assert int(tok2[0]) == 0 and float(val2[0]) == -float("inf")
    assert torch.equal(tok2[1:], tok[1:]) and torch.equal(val2[1:], val[1:])


@pytest.mark.parametrize("dtype,heads", [("bf16", 8), ("f16", 4)])
def test_decode_attention_cut_in_three(dtype, heads):
    """32 to 64 (sequence, kv head) pairs with one context long enough: every context is cut in three, the short ones into fewer
    pieces than that (one of them within a single tile)."""
    cfg = StageConfig("cut3", dtype, 512, heads, heads, 96, 2, 1, (0,), batch=1, seed=809)
    lens = [2100, 33, 1, 700, 2047, 64, 257, 96][:32 // heads]
    w = [generate.layer_weights(cfg, l) for l in range(2)]
    ora, st = make_oracle(cfg, 0, w), make_gpu_stage(cfg, 0, w)
    oc, kv = ora.new_cache(len(lens)), st.kv_cache_create(len(lens), 2200)
    for l in range(2):
        for i, n in enumerate(lens):
            k, v = generate.synthetic_kv(cfg, l, i, n)
            kv.fill(l, i, k, v)
            oc.fill(l, i, k, v)
    kv.set_lengths(lens)
    for k in range(2):
        x = generate.hidden_rows(cfg, len(lens), stream_id=1 + k)
        p_ref, h_ref = ora.decode(oc, x)
        p, h = gpu_decode(st, kv, cfg, k, x)
        check(f"step {k} resid", h, h_ref, TOL[dtype])
        check(f"step {k} partial", p, p_ref, TOL[dtype])
