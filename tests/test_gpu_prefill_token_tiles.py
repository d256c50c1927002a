"""Prefill projections in tiles of 256 features x 160, 192 or 224 tokens (two kinds of waves that own different numbers of tokens) at the
sizes where they can go wrong: contractions shorter than the four stages, matrices that end inside a feature block, token blocks of
one row, one row more than a tile, a last block that ends inside either kind of waves, split contractions with uneven and ragged
splits, more tiles than one round of the chip, the rows' sums of squares that pairs of waves add up; forced for every projection, and
chosen by size.  The gate is the suite's per type (rounding of 16-bit operands)."""
import numpy as np
import pytest
import torch

import paper_2311_11514_amd as hx
from tests.helpers import TOL, check, gpu_prefill, make_gpu_stage, make_oracle
from workloads import StageConfig, generate

pytestmark = pytest.mark.gpu

# dtype, hidden, heads, kv heads, ffn, tp, rank, prompt lengths, tile (0: chosen)
CASES = [
    ("bf16", 128, 2, 2, 64, 2, 1, [225], 224),                 # W2 of one k-tile
    ("f16", 256, 4, 2, 160, 1, 0, [190, 1, 3], 192),
    ("bf16", 384, 3, 3, 992, 1, 0, [150, 3, 140], 160),        # a feature block and a half
    ("bf16", 384, 3, 3, 992, 1, 0, [150, 3, 140], 224),
    ("f16", 1024, 8, 2, 2880, 2, 1, [100, 171, 60], 160),      # 45 k-tiles in two splits
    ("bf16", 1024, 8, 2, 2880, 2, 0, [449], 224),
    ("f16", 1024, 16, 4, 2816, 1, 0, [320, 97], 192),
    ("bf16", 256, 4, 4, 288, 1, 0, [100] * 88, 160),           # 275 token blocks
    ("f16", 1024, 16, 4, 14336, 1, 0, [140, 160], 0),          # W1/W3 in tiles of 160
]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}_H{c[1]}_F{c[4]}_T{sum(c[7])}_{c[8]}" for c in CASES])
def test_prefill_through_token_tiles(case):
    dtype, H, hq, hkv, F, tp, rank, lens, tile = case
    print(case, flush=True)
    cfg = StageConfig("tokens", dtype, H, hq, hkv, F, 2, tp, (rank,), batch=len(lens), seed=700 + H + F)
    w = [generate.layer_weights(cfg, l) for l in range(2)]
    X = generate.hidden_rows(cfg, sum(lens))
    ora = make_oracle(cfg, rank, w)
    oc = ora.new_cache(len(lens))
    p_ref, h_ref = ora.prefill(oc, X, lens)
    st = make_gpu_stage(cfg, rank, w)
    kv = st.kv_cache_create(len(lens), max(lens) + 4)
    hx.set_gemm_tile(tile)
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


@pytest.mark.parametrize("tile", [160, 192, 224])
def test_equal_prompts_have_equal_bits(tile):
    """wherever they sit in a tile, and whichever waves own their tokens"""
    cfg = StageConfig("tokens", "bf16", 1024, 8, 2, 2816, 2, 2, (1,), batch=4, seed=71)
    w = [generate.layer_weights(cfg, l) for l in range(2)]
    x = generate.hidden_rows(cfg, 90)
    st = make_gpu_stage(cfg, 1, w)
    kv = st.kv_cache_create(4, 96)
    hx.set_gemm_tile(tile)
    try:
        p, h = gpu_prefill(st, kv, cfg, torch.cat([x, x[:7], x, x]), [90, 7, 90, 90])
    finally:
        hx.set_gemm_tile(0)
    p, h = np.asarray(p), np.asarray(h)
    for a in (97, 187):
        assert (p[:90] == p[a:a + 90]).all() and (h[:90] == h[a:a + 90]).all()
