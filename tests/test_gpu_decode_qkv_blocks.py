"""The decode QKV projection of fewer than 128 units of 16 features: one kernel up to 128, 64 and 16 k-tiles at one, two and four operand
tiles, else a split contraction that the attention finishes.  Both sides of each line, with contexts that the attention splits and does not, over two
steps (the second reads the K / V rows that the first appended).  Gate: the suite's per-type tolerance; the hi + lo operands keep decode steps well
below it."""
import pytest

from tests.helpers import TOL, check, gpu_decode, gpu_prefill, make_gpu_stage, make_oracle
from workloads import StageConfig, generate

pytestmark = pytest.mark.gpu

_sides = {}


@pytest.mark.parametrize("dtype,hidden,heads,kv_heads,tp,rows", [
    ("bf16", 512, 8, 2, 1, 17), ("f16", 512, 8, 2, 1, 32), ("bf16", 640, 10, 5, 1, 17), ("bf16", 640, 10, 5, 1, 16),
    ("f16", 1024, 16, 4, 1, 3), ("bf16", 1024, 16, 4, 1, 12),
    ("bf16", 2048, 32, 8, 2, 9), ("f16", 2048, 32, 8, 2, 16), ("bf16", 2304, 36, 12, 4, 8), ("bf16", 2304, 36, 12, 4, 9),
    ("bf16", 4096, 32, 8, 4, 3), ("f16", 4096, 32, 8, 4, 8), ("bf16", 4608, 36, 12, 4, 3)])
def test_decode_step(dtype, hidden, heads, kv_heads, tp, rows):
    print(dtype, hidden, rows, flush=True)
    cfg = StageConfig("qkvb_%s_%d" % (dtype, hidden), dtype, hidden, heads, kv_heads, 64 * tp, 1, tp, (0,), batch=1, seed=821)
    if cfg.name not in _sides:
        w = [generate.layer_weights(cfg, 0)]
        _sides[cfg.name] = make_oracle(cfg, 0, w), make_gpu_stage(cfg, 0, w)
    ora, st = _sides[cfg.name]
    assert (st.decode_splits(0, rows) == 0) == (hidden // 32 <= (128 if rows <= 8 else 64 if rows <= 16 else 16))
    lens = [1 + (i * 7) % 5 for i in range(rows)]
    lens[1], lens[2] = 40, 300
    X = generate.hidden_rows(cfg, sum(lens))
    oc = ora.new_cache(rows)
    kv = st.kv_cache_create(rows, 304)
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
