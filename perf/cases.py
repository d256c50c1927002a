"""The work a user of this library has it do, as cases that can be timed and checked.

A case is one GPU's share of a pipeline stage (or the LM head behind the last stage) and a batch; `run` takes it through
the public entry points: `Stage.prefill`, `Stage.decode` / `decode_static`, `embed_rows`, `Head.greedy`.

  kind "prefill"   one prefill call over packed ragged prompts
  kind "decode"    the cache goes back to the end of its context (a continuation is generated anew), then `steps` decode calls
  kind "generate"  token-in / token-out: embedding, prefill, then `steps` times embedding, decode and greedy head
  kind "head"      final norm, LM head and arg-max over the rows of a decode step

`lo` .. `hi` are the sequences' prompt (prefill, generate) or context (decode) lengths, spread evenly over that range in a
fixed order, so that a case's work does not depend on the seed.  Everything else is drawn from the seed, with the
distributions of workloads/generate.py: weights N(0, 0.02^2), gains 1 + 0.02 N(0, 1), rows and synthetic K / V N(0, 1).
"""
from __future__ import annotations

import math

import torch

import paper_2311_11514_amd as hx

TORCH_TYPE = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
EPS, THETA = 1e-5, 10000.0

# the layer of the 70B configurations
L70 = dict(hidden=8192, heads=64, kv_heads=8, ffn=28672)
# layers kept per stage of that width and degree: enough that the weights of one pass do not stay in the memory-side cache
L70_LAYERS = {1: 1, 2: 2, 4: 3, 8: 4}


def _case(kind, dtype, layers, tp, rank, batch, lo, hi, steps=0, vocab=0, static=False, **dims):
    return dict(kind=kind, dtype=dtype, layers=layers, tp=tp, rank=rank, batch=batch, lo=lo, hi=hi, steps=steps, vocab=vocab,
                static=static, **dims)


def _l70(kind, dtype, tp, rank, batch, lo, hi, steps=0, static=False):
    return _case(kind, dtype, L70_LAYERS[tp], tp, rank, batch, lo, hi, steps, 0, static, **L70)


def _head(dtype, tp, rank, rows, hidden, vocab):
    return dict(kind="head", dtype=dtype, tp=tp, rank=rank, batch=rows, hidden=hidden, vocab=vocab)


def listed():
    return [
        # the tiny full-precision stage of workloads/configs.py, token in to token out: the smallest calls, launches count
        dict(_case("generate", "f32", 2, 2, 0, 1, 32, 32, 8, 1000, hidden=512, heads=8, kv_heads=8, ffn=1408), name="tiny_f32_generate"),
        # a reduced-width stage in full precision, as it is run to check a 16-bit deployment: three ragged prompts
        dict(_case("prefill", "f32", 2, 1, 0, 3, 45, 301, hidden=2048, heads=16, kv_heads=4, ffn=5632), name="f32_prefill"),
        # a small 16-bit model with 64-wide heads serving seven ragged requests end to end
        dict(_case("generate", "f16", 4, 1, 0, 7, 11, 330, 8, 32000, hidden=2048, heads=32, kv_heads=8, ffn=5632), name="f16_small_generate"),
        # interactive decoding, one sequence, TP2 shard at context 1024
        dict(_l70("decode", "bf16", 2, 0, 1, 1024, 1024, 8), name="decode_tp2_b1"),
        # batched decoding on the narrowest shard, 16 sequences at context 2048
        dict(_l70("decode", "bf16", 8, 3, 16, 2048, 2048, 8), name="decode_tp8_b16"),
        # the headline's decode step: full-width layer, 32 ragged contexts
        dict(_l70("decode", "bf16", 1, 0, 32, 240, 4027, 4), name="decode_tp1_b32"),
        # a throughput server: more sequences than the latency kernels take, fp16, ragged contexts
        dict(_l70("decode", "f16", 4, 2, 90, 150, 1250, 8), name="decode_tp4_b90_f16"),
        # time to first token of one short prompt
        dict(_l70("prefill", "bf16", 4, 1, 1, 117, 117), name="prefill_tp4_117"),
        # time to first token of one ordinary prompt, fp16
        dict(_l70("prefill", "f16", 2, 1, 1, 430, 430), name="prefill_tp2_430_f16"),
        # the prefill configuration: four prompts of 512 rows on a TP4 shard
        dict(_l70("prefill", "bf16", 4, 1, 4, 512, 512), name="prefill_tp4_4x512"),
        # the headline's prefill: ragged prompts up to 4096 rows through a full-width layer
        dict(_l70("prefill", "bf16", 1, 0, 6, 128, 4096), name="prefill_tp1_ragged"),
        # next tokens of a decode batch: the 70B LM head, 48 rows
        dict(_head("bf16", 1, 0, 48, 8192, 32000), name="head_b48"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "prefill", "prefill", "prefill", "generate", "head"])
    half = rng.choice(["bf16", "bf16", "f16"])
    if kind == "head":
        tp = rng.choice([1, 1, 2, 4])
        hidden = rng.choice([2048, 4096, 8192])
        return _head(half, tp, rng.randrange(tp), _log_int(rng, 1, 128), hidden, rng.choice([32000, 32000, 50304]))
    if kind == "generate" or rng.random() < 0.2:
        # small models: either head width, any query group, both 16-bit types and full precision
        dtype = rng.choice(["f32", half, half])
        hidden = rng.choice([512, 1024, 2048] if dtype == "f32" else [1024, 2048, 4096])
        d = rng.choice([64, 128])
        heads = hidden // d
        group = rng.choice([g for g in (1, 2, 4, 8) if g <= heads])
        tp = rng.choice([t for t in (1, 2) if (heads // group) % t == 0])
        batch = _log_int(rng, 1, 12)
        hi = _log_int(rng, 8, 400)
        lo = max(1, int(hi * rng.uniform(0.1, 1.0)))
        return _case(kind, dtype, rng.choice([2, 3, 4]), tp, rng.randrange(tp), batch, lo, hi, 0 if kind == "prefill" else 8,
                     rng.choice([1000, 32000]) if kind == "generate" else 0, hidden=hidden, heads=heads, kv_heads=heads // group,
                     ffn=hidden * 11 // 4 // 64 * 64)
    tp = rng.choice([1, 2, 4, 8])
    rank = rng.randrange(tp)
    if kind == "decode":
        batch = _log_int(rng, 1, 128)
        hi = _log_int(rng, 64, 4096)
        hi = min(hi, 70000 // batch)            # context rows of the whole batch
        lo = max(1, int(hi * rng.uniform(0.05, 1.0)))
        return _l70("decode", half, tp, rank, batch, lo, hi, 4 if tp == 1 else 8, batch <= 32 and rng.random() < 0.25)
    rows = _log_int(rng, 16, 12000)
    batch = min(_log_int(rng, 1, 32), max(1, rows // 16))
    mean = rows / batch
    spread = rng.uniform(0.0, 0.95)
    lo, hi = max(1, int(mean * (1 - spread))), max(1, min(4096, int(mean * (1 + spread))))
    return _l70("prefill", half, tp, rank, batch, min(lo, hi), hi)


def _lens(case):
    n, lo, hi = case["batch"], case["lo"], case["hi"]
    return [lo + int(round((hi - lo) * (((i + 1) * 0.6180339887498949) % 1.0))) for i in range(n)]


# ---- inputs -------------------------------------------------------------------------------------------------------
def _normal(seed, what, *shape, dtype=torch.float32):
    """N(0, 1) draws of the stream `what` (a few small integers) of this seed."""
    s = seed
    for w in what:
        s = s * 1000003 + w + 1
    g = torch.Generator(device="cuda")
    g.manual_seed(s % (1 << 62))
    return torch.randn(*shape, generator=g, device="cuda", dtype=dtype)


def _layer(case, seed, layer):
    """One layer's global tensors in the stage's type, in the order of Stage.load_layer."""
    H, F, d, td = case["hidden"], case["ffn"], case["hidden"] // case["heads"], TORCH_TYPE[case["dtype"]]
    shapes = [(H,), (H, case["heads"] * d), (H, case["kv_heads"] * d), (H, case["kv_heads"] * d), (case["heads"] * d, H),
              (H,), (H, F), (H, F), (F, H)]
    out = []
    for i, s in enumerate(shapes):
        z = _normal(seed, (0, layer, i), *s, dtype=td)
        out.append(z.mul_(0.02) if len(s) == 2 else z.mul_(0.02).add_(1.0))
    return out


def _synthetic_kv(case, seed, layer):
    """K, V of every sequence's context, packed: [sum of lens, local kv heads, d], values of the stage's type."""
    n, hkv, d, td = sum(_lens(case)), case["kv_heads"] // case["tp"], case["hidden"] // case["heads"], TORCH_TYPE[case["dtype"]]
    return [_normal(seed, (1, layer, i), n, hkv, d, dtype=td).float() for i in range(2)]


def _rows(case, seed, what, n):
    return _normal(seed, (2, what), n, case["hidden"], dtype=TORCH_TYPE[case["dtype"]])


def _tokens(case, seed, what, n):
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 1000003 + 77 + what) % (1 << 62))
    return torch.randint(0, case["vocab"], (n,), generator=g, device="cuda", dtype=torch.int32)


def _ends(case, seed):
    """Embedding table (generate only), final gain and LM head."""
    td, H, V = TORCH_TYPE[case["dtype"]], case["hidden"], case["vocab"]
    table = _normal(seed, (3, 0), V, H, dtype=td) if case["kind"] == "generate" else None
    return table, _normal(seed, (3, 1), H, dtype=td).mul_(0.02).add_(1.0), _normal(seed, (3, 2), H, V, dtype=td).mul_(0.02)


def prepare(case, seed):
    kind, B, td = case["kind"], case["batch"], TORCH_TYPE[case["dtype"]]
    s = {"case": case}
    if kind in ("head", "generate"):
        table, g_final, w_lm = _ends(case, seed)
        s["table"] = table
        s["head"] = hx.Head(case["hidden"], case["vocab"], case["tp"], case["rank"], case["dtype"])
        s["head"].load(g_final, w_lm)
        del w_lm
    if kind == "head":
        s["a"], s["b"] = _rows(case, seed, 0, B), _rows(case, seed, 1, B)
        return s
    lens = _lens(case)
    st = hx.Stage(case["hidden"], case["heads"], case["kv_heads"], case["ffn"], case["layers"], case["tp"], case["rank"], case["dtype"])
    for l in range(case["layers"]):
        st.load_layer(l, *_layer(case, seed, l))
    kv = st.kv_cache_create(B, max(lens) + case["steps"])
    s.update(stage=st, kv=kv, lens=lens)
    empty = lambda *shape: torch.empty(*shape, case["hidden"], dtype=td, device="cuda")  # noqa: E731
    if kind != "decode":
        n = sum(lens)
        s["x"] = _tokens(case, seed, 0, n) if kind == "generate" else _rows(case, seed, 0, n)
        s["partial"], s["resid"] = empty(n), empty(n)
    else:
        for l in range(case["layers"]):
            k, v = (t.cpu() for t in _synthetic_kv(case, seed, l))
            at = 0
            for i, n in enumerate(lens):
                kv.fill(l, i, k[at:at + n], v[at:at + n])
                at += n
        kv.set_lengths(lens)
    if case["steps"]:
        s["steps_x"] = [_tokens(case, seed, 1 + t, B) if kind == "generate" else _rows(case, seed, 1 + t, B) for t in range(case["steps"])]
        s["steps_partial"], s["steps_resid"] = empty(case["steps"], B), empty(case["steps"], B)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "head":
        return s["head"].greedy(s["a"], s["b"])
    st, kv = s["stage"], s["kv"]
    out = {}
    if kind == "decode":
        kv.set_lengths(s["lens"])
    else:
        x = hx.embed_rows(s["table"], s["x"]) if kind == "generate" else s["x"]
        st.prefill(kv, x, s["lens"], s["partial"], s["resid"])
        out.update(partial=s["partial"], resid=s["resid"])
    step = st.decode_static if case["static"] else st.decode
    greedy = []
    for t in range(case["steps"]):
        x = hx.embed_rows(s["table"], s["steps_x"][t]) if kind == "generate" else s["steps_x"][t]
        p, r = s["steps_partial"][t], s["steps_resid"][t]
        step(kv, t, x, p, r)
        if kind == "generate":
            greedy.append(s["head"].greedy(r, p))
    if case["steps"]:
        out.update(steps_partial=s["steps_partial"], steps_resid=s["steps_resid"])
    if greedy:
        out["logits"] = [g[1] for g in greedy]
        if case["dtype"] == "f32":      # in 16 bits a near-tie goes to either side with the rounding of the layers before it
            out["tokens"] = [g[0] for g in greedy]
    return out


# ---- what a pass cannot do without ----------------------------------------------------------------------------------
def _es(case):
    return 4 if case["dtype"] == "f32" else 2


def work(case):
    H, es, B = case["hidden"], _es(case), case["batch"]
    head_elems = H * (case["vocab"] // case["tp"])
    if case["kind"] == "head":
        return {"bytes": es * (head_elems + H + 2 * B * H) + 8 * B, "flops": 2 * B * head_elems}
    d, t, L = H // case["heads"], case["tp"], case["layers"]
    hq, hkv = case["heads"] // t, case["kv_heads"] // t
    w = L * (H * (hq + 2 * hkv) * d + hq * d * H + 3 * H * (case["ffn"] // t))
    lens, nbytes, flops = _lens(case), 0, 0
    kv_row = 2 * hkv * d * es * L
    if case["kind"] != "decode":
        n = sum(lens)
        nbytes += es * (w + 3 * n * H) + n * kv_row
        flops += 2 * n * w + sum(2 * x * (x + 1) * d * hq * L for x in lens)
    for k in range(case["steps"]):
        nbytes += es * (w + 3 * B * H) + sum(x + k + 1 for x in lens) * kv_row
        flops += 2 * B * w + sum(4 * (x + k + 1) * d * hq * L for x in lens)
        if case["kind"] == "generate":
            nbytes += es * head_elems
            flops += 2 * B * head_elems
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Differences between two correct implementations, taken as sqrt(2) times their measured distance to 64 bits (two
    sets of independent roundings).  fp32: sums in another order, 1e-6 .. 3e-6.  The head and decode steps of up to 32
    rows carry their activations in two 16-bit parts: what is left is the sums' order (head, 5e-7), or the rounding of the
    outputs and of the cached rows (decode, 2.3e-3 bf16).  Everything else rounds each layer's operands to 16 bits, and every
    layer passes that on: 9e-3 (bf16) / 1.2e-3 (fp16) times the square root of the layers."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "differ": 0.01}
    bf16 = case["dtype"] == "bf16"
    if case["kind"] == "head":
        return {"rel": 1e-5, "differ": 0.01}
    if case["kind"] == "decode" and case["batch"] <= 32:
        return {"rel": 4e-3 if bf16 else 6e-4}
    return {"rel": min(0.03, (1.3e-2 if bf16 else 1.7e-3) * math.sqrt(case["layers"]))}


# ---- 64-bit reference -----------------------------------------------------------------------------------------------
def _norm(x, g):
    return x / torch.sqrt(x.square().mean(1, keepdim=True) + EPS) * g


def _rope(x, pos):
    """x [n, heads, d] rotated at positions pos [n], pairing element i with i + d / 2."""
    half = x.shape[2] // 2
    inv = THETA ** (-2.0 * torch.arange(half, device=x.device, dtype=torch.float64) / x.shape[2])
    ang = (pos.double()[:, None] * inv)[:, None, :]
    c, s = torch.cos(ang), torch.sin(ang)
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], 2)


class _Exact:
    def __init__(self, case, seed):
        self.case, t, r = case, case["tp"], case["rank"]
        self.d = case["hidden"] // case["heads"]
        q, k, f = (case[n] // t for n in ("heads", "kv_heads", "ffn"))
        self.hq, self.hkv = q, k
        q, k = q * self.d, k * self.d
        cut = [None, (1, q), (1, k), (1, k), (0, q), None, (1, f), (1, f), (0, f)]
        self.layers = []
        for l in range(case["layers"]):
            ws = _layer(case, seed, l)
            self.layers.append([w.double() if c is None else w.narrow(c[0], r * c[1], c[1]).double() for w, c in zip(ws, cut)])
        self.cache = [[None] * case["batch"] for _ in self.layers]

    def attend(self, q, k, v, past):
        """q [n, hq, d] behind `past` cached rows, k / v [past + n, hkv, d]."""
        n, G = q.shape[0], self.hq // self.hkv
        out = torch.empty_like(q)
        mask = torch.arange(k.shape[0], device=q.device)[None, :] > past + torch.arange(n, device=q.device)[:, None]
        for c in range(self.hkv):
            kt, vc = k[:, c].t().contiguous(), v[:, c].contiguous()
            for h in range(c * G, (c + 1) * G):
                s = (q[:, h].contiguous() @ kt / math.sqrt(self.d)).masked_fill_(mask, -math.inf)
                out[:, h] = torch.softmax(s, 1) @ vc
        return out

    def forward(self, x, news):
        """Rows x [sum(news), H], news[i] of sequence i; returns (partial, resid)."""
        h, T = x.double(), x.shape[0]
        for l, (ga, wq, wk, wv, wo, gf, w1, w3, w2) in enumerate(self.layers):
            past = [0 if c is None else c[0].shape[0] for c in self.cache[l]]
            pos = torch.cat([torch.arange(p, p + n, device=h.device) for p, n in zip(past, news)])
            n = _norm(h, ga)
            q, k = (_rope((n @ w).view(T, -1, self.d), pos) for w in (wq, wk))
            v = (n @ wv).view(T, -1, self.d)
            o, at = torch.empty_like(q), 0
            for i, m in enumerate(news):
                c, rows = self.cache[l][i], slice(at, at + m)
                kv = [k[rows], v[rows]] if c is None else [torch.cat([c[0], k[rows]]), torch.cat([c[1], v[rows]])]
                self.cache[l][i] = kv
                o[rows] = self.attend(q[rows], kv[0], kv[1], past[i])
                at += m
            h = h + o.reshape(T, -1) @ wo
            n = _norm(h, gf)
            p = (torch.nn.functional.silu(n @ w1) * (n @ w3)) @ w2
            if l + 1 < len(self.layers):
                h = h + p
        return p, h


def exact(case, seed):
    kind, B = case["kind"], case["batch"]
    if kind in ("head", "generate"):
        table, g, w = _ends(case, seed)
        vl = case["vocab"] // case["tp"]
        g, w = g.double(), w.narrow(1, case["rank"] * vl, vl).double()
        top = lambda a, b: (_norm(a + b, g) @ w).max(1).values  # noqa: E731
    if kind == "head":
        return [None, top(_rows(case, seed, 0, B).double(), _rows(case, seed, 1, B).double())]
    lens, e, out = _lens(case), _Exact(case, seed), {}
    if kind == "decode":
        for l in range(case["layers"]):
            k, v = (t.double().split(lens) for t in _synthetic_kv(case, seed, l))
            e.cache[l] = [[a, b] for a, b in zip(k, v)]
    else:
        n = sum(lens)
        out["partial"], out["resid"] = e.forward(table[_tokens(case, seed, 0, n).long()] if kind == "generate" else _rows(case, seed, 0, n), lens)
    ps, rs, logits = [], [], []
    for t in range(case["steps"]):
        p, r = e.forward(table[_tokens(case, seed, 1 + t, B).long()] if kind == "generate" else _rows(case, seed, 1 + t, B), [1] * B)
        ps.append(p)
        rs.append(r)
        if kind == "generate":
            logits.append(top(r, p))
    if case["steps"]:
        out["steps_partial"], out["steps_resid"] = torch.stack(ps), torch.stack(rs)
    if logits:
        out["logits"] = logits
    return out
