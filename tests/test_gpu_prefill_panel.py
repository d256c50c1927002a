"""The 128 x 128 prefill projections (whole contraction, halves of it on two groups of waves) at the sizes where they can go wrong: one
k-tile (a stage that holds half of what it can), odd and even numbers of them, fewer and more than the four stages, matrices that end inside
a tile, one row more than a tile, a full last tile, ragged prompts, more tiles than one round of the chip; forced for every projection
of the stage, and chosen by size.  The gate is the suite's per type (rounding of 16-bit operands)."""
import pytest

import paper_2311_11514_amd as hx
from tests.helpers import TOL, check, gpu_prefill, make_gpu_stage, make_oracle
from workloads import StageConfig, generate

pytestmark = pytest.mark.gpu

# dtype, hidden, heads, kv heads, ffn, tp, rank, prompt lengths, forced
CASES = [
    ("bf16", 128, 2, 2, 64, 2, 1, [129], True),
    ("f16", 256, 4, 2, 160, 1, 0, [130, 1, 3], True),
    ("bf16", 256, 4, 1, 416, 1, 0, [256], True),
    ("bf16", 384, 3, 3, 992, 1, 0, [150, 3, 140], True),
    ("f16", 1024, 8, 2, 2880, 2, 1, [100, 171, 60], True),
    ("bf16", 256, 4, 4, 288, 1, 0, [100] * 88, True),
    ("f16", 1024, 16, 4, 1376, 1, 0, [140, 260], False),
    ("bf16", 1024, 8, 8, 1056, 1, 0, [90] * 45, False),
    ("bf16", 512, 8, 2, 1408, 1, 0, [3], False),
    ("f16", 1024, 8, 4, 2816, 1, 0, [40, 56], False),
]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}_H{c[1]}_F{c[4]}_T{sum(c[7])}" for c in CASES])
def test_prefill_through_128_tiles(case):
    dtype, H, hq, hkv, F, tp, rank, lens, forced = case
    print(case, flush=True)
    cfg = StageConfig("panel", dtype, H, hq, hkv, F, 2, tp, (rank,), batch=len(lens), seed=900 + H + F)
    w = [generate.layer_weights(cfg, l) for l in range(2)]
    X = generate.hidden_rows(cfg, sum(lens))
    ora = make_oracle(cfg, rank, w)
    oc = ora.new_cache(len(lens))
    p_ref, h_ref = ora.prefill(oc, X, lens)
    st = make_gpu_stage(cfg, rank, w)
    kv = st.kv_cache_create(len(lens), max(lens) + 4)
    hx.set_gemm_tile(128 if forced else 0)
    try:
        p, h = gpu_prefill(st, kv, cfg, X, lens)
    finally:
        hx.set_gemm_tile(0)
    check("prefill resid", h, h_ref, TOL[dtype])
    check("prefill partial", p, p_ref, TOL[dtype])
    d = cfg.head_dim
    for layer in range(2):
        kk, vv = kv.read(layer, len(lens) - 1, 0, lens[-1])
        check(f"K layer {layer}", kk.numpy().reshape(-1, d), oc.k[layer][-1].reshape(-1, d), TOL[dtype])
        check(f"V layer {layer}", vv.numpy().reshape(-1, d), oc.v[layer][-1].reshape(-1, d), TOL[dtype])
