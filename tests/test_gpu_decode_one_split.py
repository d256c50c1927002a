"""The split form of the decode projections where it has one split and finishes its own units: W1/W3 (1298 units, so that the last
block has half its waves) at one, two and four operand tiles and their edges; the LM head, whose units are one feature tile or two, up to 64
rows, with columns beyond the last; the lowest id wins an exact tie, a row of NaN has no candidate.  Beside them the single kernel of more
units (1802) or fewer operand tiles; every case says which form it is for.  Gate: the suite's per-type tolerance; the hi + lo operands
keep decode steps well below it."""
import numpy as np
import pytest
import torch

import paper_2311_11514_amd as hx
from oracle import stage_oracle as so
from tests.helpers import TOL, check, gpu_decode, gpu_prefill, make_gpu_stage, make_oracle
from workloads import StageConfig, generate

pytestmark = pytest.mark.gpu

_sides = {}


@pytest.mark.parametrize("ffn,splits", [(20768, 1), (28832, 0)])
@pytest.mark.parametrize("dtype,rows", [("bf16", t) for t in (3, 8, 9, 16, 17, 25, 32)] + [("f16", 5), ("f16", 12), ("f16", 30)])
def test_decode_step(dtype, rows, ffn, splits):
    print(dtype, rows, ffn, flush=True)
    cfg = StageConfig("one_%s_%d" % (dtype, ffn), dtype, 512, 8, 2, ffn, 1, 1, (0,), batch=1, seed=811)
    if cfg.name not in _sides:
        w = [generate.layer_weights(cfg, 0)]
        _sides[cfg.name] = make_oracle(cfg, 0, w), make_gpu_stage(cfg, 0, w)
    ora, st = _sides[cfg.name]
    assert st.decode_splits(2, rows) == splits
    lens = [1 + (i * 7) % 5 for i in range(rows)]
    X = generate.hidden_rows(cfg, sum(lens))
    oc = ora.new_cache(rows)
    kv = st.kv_cache_create(rows, 16)
    ora.prefill(oc, X, lens)
    gpu_prefill(st, kv, cfg, X, lens)
    for i in range(rows):                       # the steps start from the very rows the GPU holds
        k, v = kv.read(0, i, 0, lens[i])
        oc.fill(0, i, k, v)
    for k in range(2):
        x = generate.hidden_rows(cfg, rows, stream_id=1 + k)
        p_ref, h_ref = ora.decode(oc, x)
        p, h = gpu_decode(st, kv, cfg, k, x)
        check(f"{rows} rows step {k} resid", h, h_ref, TOL[dtype])
        check(f"{rows} rows step {k} partial", p, p_ref, TOL[dtype])


@pytest.mark.parametrize("hidden,vocab,rows,splits", [(1024, 60011, t, 1) for t in (9, 17, 32, 40, 64)] + [(1024, 59995, 16, 0)] +
                         [(1024, 59995, t, 1) for t in (25, 33, 64)] + [(2304, 59995, t, 1) for t in (3, 8, 9, 16)])
def test_head(hidden, vocab, rows, splits):
    print(hidden, vocab, rows, flush=True)
    cfg = StageConfig("headone", "bf16", hidden, 8, 8, 64, 1, 1, (0,), batch=1, seed=812, vocab=vocab)
    if (hidden, vocab) not in _sides:
        _sides[hidden, vocab] = generate.head_weights(cfg)
    hw = _sides[hidden, vocab]
    a, b = (generate.hidden_rows(cfg, rows, stream_id=s).to(torch.bfloat16) for s in (3, 4))
    g, w = hw["g_final"].double().numpy(), hw["w_lm"]
    w[:, vocab - 3] = w[:, 7]                   # exact ties, where they are the best: the lowest id
    a[1] = float("nan")
    hd = hx.Head(hidden, vocab, 1, 0, "bf16", cfg.rms_eps)
    assert hd.splits(rows) == splits
    hd.load(hw["g_final"].cuda(), w.cuda())
    tok, val = hd.greedy(a.cuda(), b.cuda())
    torch.cuda.synchronize()
    tok, val = tok.cpu().numpy(), val.cpu().numpy()
    x = a.double().numpy() + b.double().numpy()
    ok = np.arange(rows) != 1
    logits = so.rmsnorm(x[ok], g, cfg.rms_eps) @ w.double().numpy()
    top = np.sort(logits, axis=1)
    # the operands carry 16 mantissa bits: a logit is off by about 2^-17 of the row's scale
    assert np.max(np.abs(val[ok] - top[:, -1]) / np.abs(top[:, -1])) < 2e-4
    clear = top[:, -1] - top[:, -2] > 1e-3 * np.abs(top[:, -1])
    assert clear.mean() > 0.8 and np.array_equal(tok[ok][clear], np.argmax(logits, axis=1)[clear])
    assert tok[1] == 0 and (tok != vocab - 3).all()
