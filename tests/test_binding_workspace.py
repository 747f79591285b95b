"""The binding's scratch: one buffer per thread, device and stream, none kept under graph
capture.  The keeping rules run on the CPU (stream handles and the capture state are faked);
the GPU test replays a captured layer after larger eager calls."""
import threading

import pytest
import torch

from paper_2608_04401_amd import binding as B
from paper_2608_04401_amd import synth

CPU = torch.device("cpu")


def _fresh(monkeypatch, stream=0):
    monkeypatch.setattr(B, "_ws", threading.local(), raising=False)
    monkeypatch.setattr(B, "_stream", lambda: stream)
    monkeypatch.setattr(torch._C, "_cuda_isCurrentStreamCapturing", lambda: False)


def test_one_buffer_per_stream(monkeypatch):
    _fresh(monkeypatch, stream=1)
    a = B.workspace(100, CPU)
    assert B.workspace(50, CPU) is a and a.numel() >= 100
    monkeypatch.setattr(B, "_stream", lambda: 2)
    b = B.workspace(100, CPU)  # calls on stream 2 may run beside those of stream 1
    assert b.data_ptr() != a.data_ptr()
    larger = B.workspace(200, CPU)
    assert larger.numel() >= 200 and B.workspace(100, CPU) is larger
    monkeypatch.setattr(B, "_stream", lambda: 1)
    assert B.workspace(100, CPU) is a


def test_one_buffer_per_thread(monkeypatch):
    _fresh(monkeypatch)
    a = B.workspace(100, CPU)
    got = []
    t = threading.Thread(target=lambda: got.append(B.workspace(100, CPU)))
    t.start()
    t.join()
    # two threads enqueueing on one stream interleave their launches
    assert got[0].data_ptr() != a.data_ptr()
    assert B.workspace(100, CPU) is a


def test_nothing_kept_under_capture(monkeypatch):
    _fresh(monkeypatch)
    a = B.workspace(100, CPU)
    monkeypatch.setattr(torch._C, "_cuda_isCurrentStreamCapturing", lambda: True)
    b, c = B.workspace(100, CPU), B.workspace(100, CPU)
    assert len({t.data_ptr() for t in (a, b, c)}) == 3
    monkeypatch.setattr(torch._C, "_cuda_isCurrentStreamCapturing", lambda: False)
    assert B.workspace(100, CPU) is a


def test_streams_kept_are_bounded(monkeypatch):
    _fresh(monkeypatch)
    for stream in range(3 * B._WS_STREAMS):
        monkeypatch.setattr(B, "_stream", lambda: stream)
        B.workspace(64, CPU)
    assert len(B._ws.pool) == B._WS_STREAMS


@pytest.mark.gpu
def test_replay_after_larger_eager_calls():
    """A small captured layer replayed after a larger layer has run and other memory has been
    taken and overwritten: the graph's scratch is still its own, so the eager result."""
    N, d, m = 16, 256, 128
    Wr = synth.device_normal_bf16((N, d), 1, 0.02)
    Wgu = synth.device_normal_bf16((N, 2 * m, d), 2, 0.02)
    Wd = synth.device_normal_bf16((N, d, m), 3, 0.02)
    x = synth.device_normal_bf16((300, d), 4, 1.0)
    big = synth.device_normal_bf16((5000, d), 5, 1.0)
    want = B.elb_moe_forward(x, Wr, Wgu, Wd, K=4).view(torch.int16).clone()
    out = torch.empty_like(x)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        B.elb_moe_forward(x, Wr, Wgu, Wd, K=4, out=out)
    for _ in range(3):
        B.elb_moe_forward(big, Wr, Wgu, Wd, K=4)  # needs a larger buffer than the graph's
        taken = [torch.full((1 << 20,), 7, dtype=torch.int32, device="cuda") for _ in range(8)]
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), want)
        assert all(bool((t == 7).all()) for t in taken)


@pytest.mark.gpu
def test_two_streams_at_once():
    """Layer calls on two streams, enqueued in turn without waiting: each gives the result of
    its own input."""
    N, d, m = 16, 512, 256
    Wr = synth.device_normal_bf16((N, d), 1, 0.02)
    Wgu = synth.device_normal_bf16((N, 2 * m, d), 2, 0.02)
    Wd = synth.device_normal_bf16((N, d, m), 3, 0.02)
    xs = [synth.device_normal_bf16((1000, d), 10 + i, 1.0) for i in range(2)]
    want = [B.elb_moe_forward(x, Wr, Wgu, Wd, K=4).view(torch.int16) for x in xs]
    streams = [torch.cuda.Stream() for _ in xs]
    torch.cuda.synchronize()
    ys = [[], []]
    for _ in range(10):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                ys[i].append(B.elb_moe_forward(xs[i], Wr, Wgu, Wd, K=4))
    torch.cuda.synchronize()
    for i in range(2):
        assert all(torch.equal(y.view(torch.int16), want[i]) for y in ys[i])
