"""The launch that brings a batch's descriptor to the device: its status is its own, the staging
buffer is not overwritten before it has been read, and it can be captured."""
import ctypes

import numpy as np
import pytest

from paper_2603_14371_amd import binding as B
from paper_2603_14371_amd import synth
from paper_2603_14371_amd.synth import ACTION, DECODE, _TraceBuilder, _workload

pytestmark = pytest.mark.gpu


def _runtime():
    """The HIP runtime that this process has loaded."""
    with open("/proc/self/maps") as f:
        return ctypes.CDLL(next(l.split()[-1] for l in f if "libamdhip64" in l))


def _world(n_streams, **kw):
    from paper_2603_14371_amd.harness import GpuWorld
    b = _TraceBuilder()
    sids = [b.stream(-1, DECODE) for _ in range(n_streams)]
    w = _workload("upload", 5160, 1, 512, b.trace)
    gw = GpuWorld(w, synth.DataSource(w["seed"]), max_append_tokens=8192, max_q_tokens=16, **kw)
    gw.run(w["trace"])
    return gw, sids


def test_an_error_left_by_another_call_does_not_fail_the_build():
    import torch
    gw, sids = _world(1)
    hip = _runtime()
    torch.cuda.synchronize()
    hip.hipGetLastError()
    assert hip.hipSetDevice(999) != 0          # refused on the host; stays the thread's last error
    try:
        batch = B.oxy_batch_build(gw.pool, [(sids[0], 3)], 0, gw._stream())
    finally:
        left = hip.hipGetLastError()
    assert left != 0                           # and it is still there for whoever asks
    assert B.oxy_stream_info(gw.pool, sids[0])[2] == 3
    B.oxy_batch_destroy(batch)
    gw.close()


def test_staging_is_not_overwritten_before_it_has_been_read():
    """Append-only batches of alternating streams, built and destroyed without a wait while a long
    product keeps the stream busy: every row must land in its own batch's slot."""
    import torch
    gw, sids = _world(2, max_live_batches=1)
    n, rounds = 40, 12
    k = torch.randint(0, 1 << 15, (rounds, n, 256), dtype=torch.int16, device="cuda")
    v = torch.randint(0, 1 << 15, (rounds, n, 256), dtype=torch.int16, device="cuda")
    a = torch.randn((4096, 4096), device="cuda", dtype=torch.bfloat16)
    torch.cuda.synchronize()
    for r in range(rounds):
        a = (a @ a).clamp_(-1, 1)
        batch = B.oxy_batch_build(gw.pool, [(sids[r % 2], n)], B.BATCH_APPEND_ONLY, gw._stream())
        B.oxy_stream_append(gw.pool, batch, 0, k[r].data_ptr(), v[r].data_ptr(), gw._stream())
        B.oxy_batch_destroy(batch)
    for s in (0, 1):
        gk, gv = gw.gather(0, gw.stream_slots(sids[s]))
        assert np.array_equal(gk, k[s::2].cpu().numpy().view(np.uint16).reshape(-1, 256))
        assert np.array_equal(gv, v[s::2].cpu().numpy().view(np.uint16).reshape(-1, 256))
    gw.close()


def test_a_captured_step_replays_like_the_eager_one():
    """Build and one layer captured together and replayed between eager steps of the same pool."""
    import torch
    from paper_2603_14371_amd.harness import GpuWorld
    b = _TraceBuilder()
    pid = b.prefix(100)
    act, dec = b.stream(pid, ACTION), b.stream(pid, DECODE)
    w = _workload("captured", 5161, 1, 64, b.trace)
    gw = GpuWorld(w, synth.DataSource(w["seed"]), max_q_tokens=16, max_append_tokens=16, poison=True)
    gw.run(w["trace"])
    items = [(act, 12), (dec, 1)]
    kv = torch.randn((2, 13, 256), device="cuda").to(torch.bfloat16)
    q = torch.randn((13, 8, 256), device="cuda").to(torch.bfloat16)
    out = torch.empty((13, 8, 256), dtype=torch.bfloat16, device="cuda")

    def step(stream):
        B.oxy_stream_rewind(gw.pool, dec, 0)
        batch = B.oxy_batch_build(gw.pool, items, 0, stream)
        B.oxy_append_attention(gw.pool, batch, 0, kv[0].data_ptr(), kv[1].data_ptr(), q.data_ptr(),
                               out.data_ptr(), 0, w["scale"], stream)
        B.oxy_batch_destroy(batch)

    step(gw._stream())
    torch.cuda.synchronize()
    eager = out.clone()
    assert torch.isfinite(eager).all()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        step(side.cuda_stream)
    for _ in range(4):
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager)
        out.zero_()
        step(gw._stream())
        torch.cuda.synchronize()
        assert torch.equal(out, eager)
    del graph
    gw.close()
