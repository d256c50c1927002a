"""W1/W3 of up to 128 rows in the skinny kernel that finishes its own tiles: the whole contraction in a block (four waves, or eight in two
groups), and two splits whose last block adds the other's sums; one to four token blocks, the last of them ragged; odd numbers of token
blocks, of which one group of waves has fewer; a matrix that ends inside a block of features.  Several calls on one stage: the
arrival counters are zero again, and which block was last does not show.  The gate is the suite's per type (rounding of
16-bit operands)."""
import pytest
import torch

from tests.helpers import TOL, check, gpu_prefill, make_gpu_stage, make_oracle
from workloads import StageConfig, generate

pytestmark = pytest.mark.gpu

# dtype, hidden, heads, kv heads, ffn, prompt lengths
CASES = [
    ("bf16", 1024, 8, 2, 16640, [100]),             # 260 feature blocks, one split, four waves
    ("f16", 1024, 16, 4, 16640, [30, 3]),
    ("bf16", 1024, 8, 8, 11008, [20]),              # 172 blocks, one split, eight waves
    ("bf16", 1024, 8, 2, 5536, [7, 12]),            # 87 blocks, the last one half, two splits, four waves
    ("f16", 4096, 32, 8, 6592, [60, 5, 10]),        # 103 blocks, two splits, eight waves
    ("bf16", 4096, 32, 8, 6592, [128]),
    ("bf16", 4096, 32, 8, 6624, [41]),              # 104 blocks, the last one half
]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}_H{c[1]}_F{c[4]}_T{sum(c[5])}" for c in CASES])
def test_w13_finishes_its_own_tiles(case):
    dtype, H, hq, hkv, F, lens = case
    print(case, flush=True)
    cfg = StageConfig("w13", dtype, H, hq, hkv, F, 1, 1, (0,), batch=len(lens), seed=600 + H + F)
    w = [generate.layer_weights(cfg, 0)]
    X = generate.hidden_rows(cfg, sum(lens))
    ora = make_oracle(cfg, 0, w)
    p_ref, h_ref = ora.prefill(ora.new_cache(len(lens)), X, lens)
    st = make_gpu_stage(cfg, 0, w)
    kv = st.kv_cache_create(len(lens), max(lens) + 4)
    p, h = gpu_prefill(st, kv, cfg, X, lens)
    check("prefill resid", h, h_ref, TOL[dtype])
    check("prefill partial", p, p_ref, TOL[dtype])
    for _ in range(6):
        p2, h2 = gpu_prefill(st, kv, cfg, X, lens)
        assert (p2 == p).all() and (h2 == h).all()


def test_overlapping_launches_leave_nothing_behind():
    """Two splits count their arrivals in counters that outlive the call.  The same FFN sub-layer many times on two streams at once (equal inputs, so that whatever
    the calls share holds the same values), which a caller must not do: calls after them are not affected."""
    cfg = StageConfig("w13over", "bf16", 1024, 8, 2, 5536, 1, 1, (0,), batch=1, seed=611)
    st = make_gpu_stage(cfg, 0, [generate.layer_weights(cfg, 0)])
    kv = st.kv_cache_create(1, 64)
    xs = [generate.hidden_rows(cfg, 19, stream_id=i).cuda() for i in range(2)]          # (128 x 128 tiles take more rows of this width)

    def alone(x):
        out = torch.empty_like(x)
        st.run_sublayer(kv, 0, 1, x, [19], 1, out)
        torch.cuda.synchronize()
        return out

    want = [alone(x) for x in xs]
    streams, outs = [torch.cuda.Stream(), torch.cuda.Stream()], [torch.empty_like(xs[1]) for _ in range(2)]
    for _ in range(100):
        for s, out in zip(streams, outs):
            st.run_sublayer(kv, 0, 1, xs[1], [19], 1, out, stream=s)
    torch.cuda.synchronize()
    for _ in range(3):
        for x, ref in zip(xs, want):
            assert torch.equal(alone(x), ref)
