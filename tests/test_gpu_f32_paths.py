"""fp32 stage and head at the sizes where their kernels change form: one or two 16-row token tiles (16 / 17 / 32 rows), the
tiled products from 33 rows on (64-row tiles, split contraction), one or two columns per lane (from 4096 columns on),
FFN shards that are padded, 1 to 16 query heads per kv head, both head widths, prompts around the 16- and 128-row
attention tiles, more than 32 sequences.  fp32 sums of up to 4096 terms: n u = 2.4e-4 at the very worst, 1e-6 .. 1e-5 in
practice; the gate is the suite's 1e-4."""
import numpy as np
import pytest
import torch

from oracle import stage_oracle as so
from tests.helpers import TOL, check, gpu_decode, gpu_prefill, make_gpu_stage, make_oracle
from workloads import StageConfig, generate

pytestmark = pytest.mark.gpu

# hidden, heads, kv heads, ffn, tp, rank, prompt lengths
CASES = [
    (512, 8, 8, 1408, 2, 1, [1]),
    (512, 8, 2, 74, 2, 0, [5, 11]),
    (512, 4, 2, 333, 1, 0, [16, 1]),
    (512, 8, 1, 1408, 1, 0, [31, 1]),
    (512, 8, 4, 90, 1, 0, [33]),
    (1024, 8, 8, 2816, 2, 1, [64, 1]),
    (512, 8, 2, 1000, 1, 0, [129, 16, 17, 128, 15]),
    (256, 4, 2, 4100, 1, 0, [7]),
    (256, 2, 1, 4164, 1, 0, [20]),
    (4096, 32, 2, 40, 1, 0, [3]),
    (4096, 32, 2, 40, 1, 0, [1] * 20),
    (256, 4, 1, 96, 1, 0, [1, 2] * 20),
]


@pytest.mark.parametrize("case", CASES, ids=[f"H{c[0]}F{c[3]}T{sum(c[6])}" for c in CASES])
def test_f32_prefill_then_decode(case):
    H, hq, hkv, F, tp, rank, lens = case
    print(case, flush=True)
    cfg = StageConfig("f32case", "f32", H, hq, hkv, F, 2, tp, (rank,), batch=len(lens), seed=700 + H + F)
    w = [generate.layer_weights(cfg, l) for l in range(2)]
    X = generate.hidden_rows(cfg, sum(lens))
    ora = make_oracle(cfg, rank, w)
    oc = ora.new_cache(len(lens))
    st = make_gpu_stage(cfg, rank, w)
    kv = st.kv_cache_create(len(lens), max(lens) + 20)
    p_ref, h_ref = ora.prefill(oc, X, lens)
    p, h = gpu_prefill(st, kv, cfg, X, lens)
    check("prefill resid", h, h_ref, TOL["f32"])
    check("prefill partial", p, p_ref, TOL["f32"])
    for k in range(3):
        x = generate.hidden_rows(cfg, len(lens), stream_id=1 + k)
        p_ref, h_ref = ora.decode(oc, x)
        p, h = gpu_decode(st, kv, cfg, k, x)
        check(f"decode {k} resid", h, h_ref, TOL["f32"])
        check(f"decode {k} partial", p, p_ref, TOL["f32"])
    s, d = int(np.argmax(lens)), cfg.head_dim
    for layer in range(2):
        kk, vv = kv.read(layer, s, 0, lens[s] + 3)
        check(f"K layer {layer}", kk.numpy().reshape(-1, d), oc.k[layer][s].reshape(-1, d), TOL["f32"])
        check(f"V layer {layer}", vv.numpy().reshape(-1, d), oc.v[layer][s].reshape(-1, d), TOL["f32"])


# the tiled products' ways of dealing tiles out to the CUs: a launch of fewer than 256 tiles cut along the contraction, of whole
# tiles, of two full rounds and a few tiles whose k-steps go round (258 x 2 in W1/W3, the last one
# 52 columns wide), contractions of two and four k-steps; 17 token blocks, of which 15 columns of tiles make a round and one column of
# W_O (the residual) and nine of QKV are dealt out behind it
DEALT = [
    (1024, 8, 2, 1500, 1, 0, [200, 33]),
    (64, 1, 1, 4096, 1, 0, [40, 60]),
    (128, 2, 1, 130, 1, 0, [1000, 88]),
    (512, 4, 2, 16500, 1, 0, [100]),
    (1024, 8, 2, 16700, 1, 0, [80]),
    (2048, 16, 4, 96, 1, 0, [1033]),
]


@pytest.mark.parametrize("case", DEALT, ids=[f"H{c[0]}F{c[3]}T{sum(c[6])}" for c in DEALT])
def test_f32_tiles_dealt_out(case):
    test_f32_prefill_then_decode(case)


# equal prompts whose rows sit in different token blocks: tiles cut along the contraction, whole ones and both in one launch
# (88 columns x 9 token blocks in W1/W3; 24 and 16 columns x 17 in QKV and W_O), one-row prompts, decode steps of many sequences
@pytest.mark.parametrize("H,hq,hkv,F,rows,batch", [(512, 8, 2, 1408, 50, 3), (2048, 16, 4, 5632, 190, 3), (2048, 16, 4, 256, 350, 3), (1024, 8, 8, 2816, 1, 100)])
def test_f32_equal_sequences_have_equal_bits(H, hq, hkv, F, rows, batch):
    cfg = StageConfig("f32same", "f32", H, hq, hkv, F, 2, 1, (0,), batch=batch, seed=704)
    st = make_gpu_stage(cfg, 0, [generate.layer_weights(cfg, layer) for layer in range(2)])
    kv = st.kv_cache_create(batch, rows + 2)
    p, h = gpu_prefill(st, kv, cfg, generate.hidden_rows(cfg, rows).repeat(batch, 1), [rows] * batch)
    for out in (p, h, *gpu_decode(st, kv, cfg, 0, generate.hidden_rows(cfg, 1, stream_id=1).repeat(batch, 1))):
        out = np.asarray(out).reshape(batch, -1, H)
        assert (out == out[:1]).all()
    for layer in range(2):
        first = kv.read(layer, 0, 0, rows + 1)
        for s in range(1, batch):
            assert all(torch.equal(a, b) for a, b in zip(kv.read(layer, s, 0, rows + 1), first))


@pytest.mark.parametrize("rows", [24, 70])
def test_f32_non_finite_rows_stay_with_their_successors(rows):
    """A row that is not finite reaches the rows behind it through the cache, and none before it."""
    cfg = StageConfig("f32inf", "f32", 512, 8, 2, 96, 1, 1, (0,), batch=1, seed=701)
    w = [generate.layer_weights(cfg, 0)]
    st = make_gpu_stage(cfg, 0, w)
    kv = st.kv_cache_create(1, 128)
    X = generate.hidden_rows(cfg, rows)
    p0, h0 = gpu_prefill(st, kv, cfg, X, [rows])
    X[9, 5] = float("inf")
    p1, h1 = gpu_prefill(st, kv, cfg, X, [rows])
    check("rows before", h1[:9], h0[:9], TOL["f32"])
    check("rows before", p1[:9], p0[:9], TOL["f32"])
    assert np.isnan(np.asarray(h1[9:])).any(axis=1).all()


def test_f32_rows_at_any_float_address():
    """The caller's buffers need the alignment of a float, no more."""
    cfg = StageConfig("f32addr", "f32", 512, 8, 2, 96, 1, 1, (0,), batch=1, seed=702)
    st = make_gpu_stage(cfg, 0, [generate.layer_weights(cfg, 0)])
    kv = st.kv_cache_create(1, 128)
    for rows in (3, 50):
        X = generate.hidden_rows(cfg, rows).cuda()
        outs = []
        for off in (0, 1, 3):
            x, p, h = (torch.empty(rows * cfg.hidden + 4, device="cuda")[off:off + rows * cfg.hidden].view(rows, -1) for _ in range(3))
            x.copy_(X)
            st.prefill(kv, x, [rows], p, h)
            torch.cuda.synchronize()
            outs.append((p.clone(), h.clone()))
        assert all(torch.equal(a, b) for o in outs[1:] for a, b in zip(o, outs[0]))


@pytest.mark.parametrize("hidden,vocab,rows", [(516, 1003, 1), (512, 1000, 16), (1028, 4107, 17), (260, 4120, 40)])
def test_f32_head_shapes(hidden, vocab, rows):
    import paper_2311_11514_amd as hx
    cfg = StageConfig("f32head", "f32", hidden, 1, 1, 64, 1, 1, (0,), batch=1, seed=703, vocab=vocab)
    hw = generate.head_weights(cfg)
    hd = hx.Head(hidden, vocab, 1, 0, "f32", cfg.rms_eps)
    hd.load(hw["g_final"].cuda(), hw["w_lm"].cuda())
    a, b = generate.hidden_rows(cfg, rows, stream_id=3), generate.hidden_rows(cfg, rows, stream_id=4)
    for second in (None, b):
        x = a.double().numpy() + (0 if second is None else b.double().numpy())
        tok, val = hd.greedy(a.cuda(), None if second is None else b.cuda())
        torch.cuda.synchronize()
        ids, ref = so.head_shard_greedy(x, hw["g_final"].double().numpy(), hw["w_lm"].double().numpy(), cfg.rms_eps, 1, 0)
        assert np.max(np.abs(val.cpu().numpy() - ref) / np.abs(ref)) < TOL["f32"]
        logits = so.rmsnorm(x, hw["g_final"].double().numpy(), cfg.rms_eps) @ hw["w_lm"].double().numpy()
        top = np.sort(logits, axis=1)
        clear = top[:, -1] - top[:, -2] > 1e-4 * np.abs(top[:, -1])
        assert clear.mean() > 0.8 and np.array_equal(tok.cpu().numpy()[clear], ids[clear])
