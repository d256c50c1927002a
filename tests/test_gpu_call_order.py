"""The order of calls on streams: every one of a row of calls sees its own row maps and lengths (they share a small ring of
staging buffers, and a prefill leaves the cache's lengths on the device in stream order), and a prefill comes behind whatever
is on the device, on streams that the stage has never seen as well."""
import numpy as np
import pytest
import torch

from tests.helpers import make_gpu_stage
from workloads import StageConfig, generate

pytestmark = pytest.mark.gpu

LENS = [[5, 40], [130], [1, 1, 1], [17, 3, 64, 2], [200, 1], [2], [33, 33], [7, 7, 7, 7]]


def _setup(dtype):
    cfg = StageConfig("order", dtype, 512, 8, 2, 1408, 2, 1, (0,), batch=4, seed=821)
    st = make_gpu_stage(cfg, 0, [generate.layer_weights(cfg, l) for l in range(2)])
    td = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    xs = [generate.hidden_rows(cfg, sum(n), stream_id=i).to("cuda", td) for i, n in enumerate(LENS)]
    ds = [generate.hidden_rows(cfg, len(n), stream_id=50 + i).to("cuda", td) for i, n in enumerate(LENS)]
    return cfg, st, xs, ds


def _one(st, kv, x, d, lens, stream=None):
    outs = [torch.empty_like(t) for t in (x, x, d, d)]
    st.prefill(kv, x, lens, outs[0], outs[1], stream=stream)
    st.decode(kv, 0, d, outs[2], outs[3], stream=stream)
    return outs


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_calls_in_a_row_equal_calls_one_by_one(dtype):
    _, st, xs, ds = _setup(dtype)
    kv = st.kv_cache_create(4, 256)
    alone = []
    for x, d, n in zip(xs, ds, LENS):
        alone.append(_one(st, kv, x, d, n))
        torch.cuda.synchronize()
    row = [_one(st, kv, x, d, n) for _ in range(2) for x, d, n in zip(xs, ds, LENS)]
    torch.cuda.synchronize()
    for i, got in enumerate(row):
        assert all(torch.equal(a, b) for a, b in zip(got, alone[i % len(LENS)])), i
    assert kv.get_lengths(4) == [8, 8, 8, 8]
    # another stream for every other call: the stage's buffers are shared, the calls still do not meet
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    mixed = [_one(st, kv, x, d, n, streams[i % 2]) for i, (x, d, n) in enumerate(zip(xs, ds, LENS))]
    torch.cuda.synchronize()
    for i, got in enumerate(mixed):
        assert all(torch.equal(a, b) for a, b in zip(got, alone[i])), i


def test_lengths_beyond_a_smaller_batch_are_cleared():
    """A batch of four, then a prefill of one: a row of the fourth sequence starts at position 0 again."""
    cfg, st, xs, _ = _setup("bf16")
    kv = st.kv_cache_create(4, 256)
    h = generate.hidden_rows(cfg, 4, stream_id=90).to("cuda", torch.float32)
    p = [torch.empty_like(xs[3]), torch.empty_like(xs[3])]
    part = [torch.empty_like(h), torch.empty_like(h)]
    for k, big_first in enumerate((True, False)):
        if big_first:
            st.prefill(kv, xs[3], LENS[3], *p)
        else:
            kv = st.kv_cache_create(4, 256)
        st.prefill(kv, xs[5], LENS[5], p[0][:2], p[1][:2])
        st.run_sublayer(kv, 0, 0, h, None, 4, part[k])
        torch.cuda.synchronize()
        assert kv.get_lengths(4) == [2, 0, 0, 0]
    assert torch.equal(part[0], part[1])


def test_prefill_refuses_to_be_recorded():
    """Row maps are built by the host for the call: a recorded prefill would replay another call's maps."""
    import paper_2311_11514_amd as hx
    _, st, xs, _ = _setup("bf16")
    kv = st.kv_cache_create(4, 256)
    p, r = torch.empty_like(xs[0]), torch.empty_like(xs[0])
    st.prefill(kv, xs[0], LENS[0], p, r)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        g.capture_begin()
        with pytest.raises(hx.HexgenError):
            st.prefill(kv, xs[0], LENS[0], p, r)
        g.capture_end()
    torch.cuda.synchronize()
    assert kv.get_lengths(2) == LENS[0]


def _recorded_step(st, kv, n):
    """A decode_static step of n sequences, recorded on a stream of its own (the recording itself runs nothing)."""
    x = torch.randn(n, 512, device="cuda").to(torch.bfloat16)
    p, r = torch.empty_like(x), torch.empty_like(x)
    st.decode_static(kv, 0, x, p, r)                    # once eagerly: looks the scratch array up
    torch.cuda.synchronize()
    g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.stream(s):
        g.capture_begin()
        st.decode_static(kv, 1, x, p, r, stream=s)
        g.capture_end()
    torch.cuda.synchronize()
    return g, s, (x, p, r)


def _late(stream):
    """Keeps `stream` busy for some milliseconds, so that what follows on it runs late."""
    with torch.cuda.stream(stream):
        torch.cuda._sleep(20_000_000)


@pytest.mark.parametrize("again_on_recording_stream", [True, False])
def test_prefill_comes_behind_a_replayed_step(again_on_recording_stream):
    _, st, xs, ds = _setup("bf16")
    kv = st.kv_cache_create(4, 256)
    want = _one(st, kv, xs[6], ds[6], LENS[6])
    torch.cuda.synchronize()
    st.prefill(kv, xs[3], LENS[3], torch.empty_like(xs[3]), torch.empty_like(xs[3]))
    g, rec, keep = _recorded_step(st, kv, 4)
    other = torch.cuda.Stream()
    mine = rec if again_on_recording_stream else None
    if mine is None:                                    # the stage's last eager call is on the stream of the prefill below
        st.decode(kv, 2, *keep)
    torch.cuda.synchronize()
    _late(other)
    with torch.cuda.stream(other):
        g.replay()
    got = _one(st, kv, xs[6], ds[6], LENS[6], mine)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(got, want))


def test_lengths_that_a_replay_advanced_are_cleared():
    """The recorded step of four sequences, replayed behind a prefill of one: the host does not know of the other three."""
    cfg, st, xs, _ = _setup("bf16")
    h = generate.hidden_rows(cfg, 4, stream_id=90).to("cuda", torch.float32)
    p = [torch.empty_like(xs[5]), torch.empty_like(xs[5])]
    part = [torch.empty_like(h), torch.empty_like(h)]
    fresh = st.kv_cache_create(4, 256)
    st.prefill(fresh, xs[5], LENS[5], *p)
    st.run_sublayer(fresh, 0, 0, h, None, 4, part[0])
    kv = st.kv_cache_create(4, 256)
    st.prefill(kv, xs[3], LENS[3], torch.empty_like(xs[3]), torch.empty_like(xs[3]))
    g, _, keep = _recorded_step(st, kv, 4)
    st.prefill(kv, xs[5], LENS[5], *p)
    g.replay()
    st.prefill(kv, xs[5], LENS[5], *p)
    st.run_sublayer(kv, 0, 0, h, None, 4, part[1])
    torch.cuda.synchronize()
    assert kv.get_lengths(4) == [2, 0, 0, 0]
    assert torch.equal(part[0], part[1])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_prefill_comes_behind_the_producer_of_its_rows(dtype):
    _, st, xs, ds = _setup(dtype)
    kv = st.kv_cache_create(4, 256)
    want = _one(st, kv, xs[0], ds[0], LENS[0])
    torch.cuda.synchronize()
    x, other = torch.zeros_like(xs[0]), torch.cuda.Stream()
    torch.cuda.synchronize()
    _late(other)
    with torch.cuda.stream(other):
        x.copy_(xs[0])
    got = _one(st, kv, x, ds[0], LENS[0])
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(got, want))
