"""The fp32 sums of a projection against 64 bits, on operands that are known exactly: run_sublayer's W2 with a gate of 32, where
silu(32) = 32 in fp32, and an up projection of rows of +-1 with integers of 7 or 10 bits, exact in any order.  n additions one behind the
other, each off by at most u = 2^-24 of the sum so far, which grows with the root of their number: u sqrt(n / 2) of the result where the
errors are independent.  A matrix instruction of 16-bit operands adds 32 products with about one such rounding; one of fp32
operands adds 2 products with two, to nearest (half of u, root mean square, with room).  The gates are these; a chain twice as long
misses them."""
import math

import pytest
import torch

import paper_2311_11514_amd as hx

pytestmark = pytest.mark.gpu

U = 2.0 ** -24
TYPE = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
# dtype, hidden, ffn, rows; 16 bits: the 128 x 128 tiles, a quarter of the contraction per chain (half of it below 48 k-tiles); fp32: chains of at most 256
# instructions, whole tiles, dealt-out ones and both in one launch
CASES = [
    ("bf16", 1024, 1504, 130),
    ("f16", 1024, 1536, 430),
    ("bf16", 2048, 2048, 330),
    ("f16", 1024, 2816, 600),
    ("bf16", 512, 7168, 200),
    ("f32", 512, 1408, 1000),
    ("f32", 2048, 5632, 572),
    ("f32", 2048, 5632, 1033),
]


@pytest.mark.parametrize("dtype,H,F,T", CASES, ids=[f"{c[0]}_H{c[1]}F{c[2]}T{c[3]}" for c in CASES])
def test_projection_sums(dtype, H, F, T):
    td = TYPE[dtype]
    g = torch.Generator().manual_seed(H + F + T)
    x = torch.randint(0, 2, (T, H), generator=g).double() * 2 - 1
    x[:, 0] = 1
    w1 = torch.zeros(H, F)
    w1[0] = 32
    top = 128 if dtype == "bf16" else 1024
    w3 = torch.randint(1 - top, top, (H, F), generator=g).double() / (16 * top)
    w2 = (torch.randn(F, H, generator=g) * 0.02).to(td)
    st = hx.Stage(H, H // 128, H // 128, F, 1, 1, 0, dtype, 1e-12)
    one, zero = torch.ones(H).to(td).cuda(), torch.zeros(H, H).to(td).cuda()
    st.load_layer(0, one, zero, zero, zero, zero, one, w1.to(td).cuda(), w3.to(td).cuda(), w2.cuda())
    kv = st.kv_cache_create(1, T)
    out = torch.empty(T, H, device="cuda")
    hx.set_gemm_tile(0 if dtype == "f32" else 128)
    try:
        st.run_sublayer(kv, 0, 1, x.float().cuda(), [T], 1, out)
        torch.cuda.synchronize()
    finally:
        hx.set_gemm_tile(0)
    exact = (32 * (x @ w3)).to(td).double() @ w2.double()
    err = float((out.cpu().double() - exact).norm() / exact.norm())
    gate = 0.5 * U * math.sqrt(2 * 256 / 2) if dtype == "f32" else U * math.sqrt(F / 32 / (2 if F < 48 * 32 else 4) / 2)
    print(f"{err:.3e} (gate {gate:.3e})", flush=True)
    assert err < gate


# dtype, hidden, heads, kv heads, rows: one, two and four operand tiles; QKV of 48, 96 and 192 units, all in one kernel
QKV_CASES = [("f16", 1024, 16, 4, 7), ("f16", 1024, 16, 4, 12), ("bf16", 1024, 16, 4, 16), ("f16", 512, 8, 2, 17), ("bf16", 512, 8, 2, 32), ("bf16", 2048, 32, 8, 9)]


@pytest.mark.parametrize("dtype,H,hq,hkv,T", QKV_CASES, ids=[f"{c[0]}_H{c[1]}T{c[4]}" for c in QKV_CASES])
def test_decode_qkv_sums_lo_products_apart(dtype, H, hq, hkv, T):
    """The hi products of k-tiles 0 and 8, one wave's first two, are +31 B + S and -31 B - S, exact in fp32; the lo product of tile 8 is less than half
    a unit of 31 B in the last place.  It is all that is left of V, and nothing is left of it where it is added to the hi products' sum."""
    td = TYPE[dtype]
    B, S, lo = (2.0 ** 15, 64.0, 2.0 ** -12) if dtype == "f16" else (2.0 ** 20, 64.0, 2.0 ** -9)
    wv = torch.zeros(H, hkv * 64)
    for tile, sign in ((0, 1), (8, -1)):
        wv[32 * tile:32 * tile + 31] = sign * B
        wv[32 * tile + 31] = sign * S
    x = torch.ones(T, H)
    x[:, 32 * 8 + 31] += lo * torch.tensor([1.0, -1.0]).repeat(16)[:T]
    st = hx.Stage(H, hq, hkv, 64, 1, 1, 0, dtype, 1e-5)
    assert st.decode_splits(0, T) == 0
    one, zero = torch.ones(H), torch.zeros
    st.load_layer(0, *[w.to(td).cuda() for w in (one, zero(H, H), zero(H, hkv * 64), wv, zero(H, H), one, zero(H, 64), zero(H, 64), zero(64, H))])
    kv = st.kv_cache_create(T, 32)
    st.run_sublayer(kv, 0, 0, x.cuda(), None, T, torch.empty(T, H, device="cuda"))
    torch.cuda.synchronize()
    x = x.double()
    exact = (x @ wv.double()) / torch.sqrt((x * x).mean(1, keepdim=True) + 1e-5)
    got = torch.stack([kv.read(0, i, 0, 1)[1].reshape(-1).double() for i in range(T)])
    err = float(((got - exact) / exact).abs().max())
    print(f"{err:.3e}", flush=True)
    assert err < (2.0 ** -10 if dtype == "f16" else 2.0 ** -7)
