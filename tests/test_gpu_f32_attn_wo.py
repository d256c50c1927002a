"""fp32 decode steps whose attention and W_O are one launch (few sequences with short contexts on a narrow stage), at contexts on both sides
of the 16-position tiles and of the line where the step goes back to two launches: none, one and several tiles per wave, waves without
a pair (three pairs), two waves to eight per pair, either head width, 1 to 16 query heads per kv head, ragged contexts.  The cached rows
and the other sequences' must come out right as well; a value that is not finite in the new row reaches its own element alone, as
with separate launches.  fp32 sums of up to 1024 terms: 1e-6 .. 1e-5 in practice; the gate is the suite's 1e-4."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2311_11514_amd.binding import lib
from tests.helpers import TOL, check, gpu_decode, make_gpu_stage, make_oracle
from workloads import StageConfig, generate

pytestmark = pytest.mark.gpu

# hidden, heads, kv heads, tp, rank, contexts
CASES = [
    (512, 8, 8, 2, 1, [0]), (512, 8, 8, 2, 0, [14]), (512, 8, 8, 2, 1, [45]),
    (1024, 16, 1, 1, 0, [252]), (256, 4, 1, 1, 0, [125, 1]), (256, 4, 1, 1, 0, [3, 31, 16]), (512, 8, 2, 1, 0, [46, 15]),
    (256, 2, 1, 1, 0, [125]), (1024, 8, 8, 8, 5, [30]),
]


@pytest.mark.parametrize("H,hq,hkv,tp,rank,lens", CASES, ids=[f"H{c[0]}h{c[1]}kv{c[2]}tp{c[3]}_{'_'.join(map(str, c[5]))}" for c in CASES])
def test_decode_across_the_line(H, hq, hkv, tp, rank, lens):
    print(H, hq, hkv, tp, lens, flush=True)
    cfg = StageConfig("awo", "f32", H, hq, hkv, 96, 2, tp, (rank,), batch=len(lens), seed=500 + H + hq)
    w = [generate.layer_weights(cfg, l) for l in range(2)]
    ora, st = make_oracle(cfg, rank, w), make_gpu_stage(cfg, rank, w)
    n, steps, d = len(lens), 6, cfg.head_dim
    oc, kv = ora.new_cache(n), st.kv_cache_create(n, max(lens) + steps)
    for l in range(2):
        for i in range(n):
            if lens[i]:
                k, v = generate.synthetic_kv(cfg, l, i, lens[i])
                kv.fill(l, i, k, v)
                oc.fill(l, i, k, v)
    kv.set_lengths(lens)
    for k in range(steps):
        x = generate.hidden_rows(cfg, n, stream_id=1 + k)
        p_ref, h_ref = ora.decode(oc, x)
        p, h = gpu_decode(st, kv, cfg, k, x)
        check(f"step {k} resid", h, h_ref, TOL["f32"])
        check(f"step {k} partial", p, p_ref, TOL["f32"])
    for l in range(2):
        for i in range(n):
            kk, vv = kv.read(l, i, 0, lens[i] + steps)
            check(f"K {l} {i}", kk.numpy().reshape(-1, d), oc.k[l][i].reshape(-1, d), TOL["f32"])
            check(f"V {l} {i}", vv.numpy().reshape(-1, d), oc.v[l][i].reshape(-1, d), TOL["f32"])


def test_new_row_that_is_not_finite():
    """One element of the new value row overflows: the head's output is infinite there and finite elsewhere, so that every column of W_O is infinite and
    none is NaN, though most of the tile's positions are masked."""
    cfg = StageConfig("awoinf", "f32", 128, 2, 2, 96, 1, 1, (0,), batch=2, seed=77)
    w = {k: v.clone() for k, v in generate.layer_weights(cfg, 0).items()}
    w["wv"][:, 5] = 3e38
    st = make_gpu_stage(cfg, 0, [w])
    kv = st.kv_cache_create(2, 16)
    for i, n in enumerate([4, 9]):
        kv.fill(0, i, *generate.synthetic_kv(cfg, 0, i, n))
    kv.set_lengths([4, 9])
    _, h = gpu_decode(st, kv, cfg, 0, generate.hidden_rows(cfg, 2, stream_id=1).abs() + 0.1)
    assert np.isinf(h).all()


def test_recorded_step_goes_by_the_capacity():
    """A replayed step meets contexts that the host has not seen: recorded for a cache whose rows all lie within the one launch's range it has one node
    less per layer than for a long cache, whatever the contexts at the recording.  Its replays agree with eager steps."""
    cfg = StageConfig("awograph", "f32", 256, 4, 1, 96, 2, 1, (0,), batch=1, seed=78)
    st = make_gpu_stage(cfg, 0, [generate.layer_weights(cfg, l) for l in range(2)])
    x = generate.hidden_rows(cfg, 1, stream_id=1).cuda()
    p, r, pe, re = (torch.empty_like(x) for _ in range(4))
    nodes = []
    for capacity in (200, 2000):
        kv, eager = st.kv_cache_create(1, capacity), st.kv_cache_create(1, capacity)
        for c in (kv, eager):
            for l in range(2):
                c.fill(l, 0, *generate.synthetic_kv(cfg, l, 0, 20))
            c.set_lengths([20])
        st.decode(eager, 0, x, pe, re)                  # (sizes the workspace)
        torch.cuda.synchronize()
        g, s = torch.cuda.CUDAGraph(keep_graph=True), torch.cuda.Stream()
        with torch.cuda.stream(s):
            g.capture_begin()
            st.decode(kv, 0, x, p, r, stream=s)
            g.capture_end()
        n = C.c_size_t()
        assert lib.hipGraphGetNodes(C.c_void_p(g.raw_cuda_graph()), None, C.byref(n)) == 0
        nodes.append(n.value)
        g.instantiate()
        for k in range(3):
            if k:
                st.decode(eager, k, x, pe, re)
            g.replay()
            torch.cuda.synchronize()
            assert torch.allclose(p, pe, rtol=1e-4, atol=1e-5) and torch.allclose(r, re, rtol=1e-4, atol=1e-5)
    print(nodes, flush=True)
    assert nodes[1] == nodes[0] + 2
