"""The scratch buffers of calls that are given no workspace: one per host thread, device and
stream, a bounded number of them, and none shared with a graph."""
import threading

import numpy as np
import pytest
import torch

kq = pytest.importorskip("paper_2003_05148_amd")


class Buffer:
    def __init__(self, device=None):
        self.buf = None

    def get(self, nbytes):
        return self


def test_scratch_is_per_stream_and_thread_and_bounded(monkeypatch):
    """(no GPU: the streams are numbers, the buffers plain objects)"""
    now = [7]
    monkeypatch.setattr(kq, "_stream", lambda device: now[0])
    monkeypatch.setattr(kq, "Workspace", Buffer)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: False)
    dev = torch.device("cuda", 0)

    def at(stream):
        now[0] = stream
        return kq._ws(dev, 100)

    def body():
        one, two = at(7), at(8)
        assert one is not two
        assert at(7) is one and at(8) is two
        other = []
        t = threading.Thread(target=lambda: other.append(kq._ws(dev, 100)))   # (the stream is still 8)
        t.start()
        t.join()
        assert other[0] is not two
        for s in range(100):
            at(s)
        assert len(kq._scratch.__dict__) <= kq._MAX_SCRATCH

    failed = []

    def run():  # in a thread of its own: this one's buffers stay as they are
        try:
            body()
        except BaseException as e:
            failed.append(e)

    t = threading.Thread(target=run)
    t.start()
    t.join()
    assert not failed, failed


@pytest.mark.gpu
def test_calls_on_two_streams_do_not_share_scratch():
    """Fits and scalar quantizations of different sizes queued on two streams, with outputs of
    their own, give the results of the same calls one after another."""
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(3)

    def made(n, k):
        X = torch.from_numpy(rng.standard_normal((n, 9)).astype(np.float32)).to(dev)
        return X, X[:k].clone()

    jobs = []
    for n, k, m in ((60000, 700, 1000003), (40001, 256, 900001)):
        X, C = made(n, k)
        v = torch.from_numpy(rng.standard_normal(m).astype(np.float32)).to(dev)
        jobs.append((X, C, v))

    def work(job):
        X, C, v = job
        return [*kq.kq_fit_layer(X, C, 6), *kq.kq_quantize_scalars(v, 6, 12)]

    want = [[t.clone() for t in work(j)] for j in jobs]
    streams = [torch.cuda.Stream(dev), torch.cuda.Stream(dev)]
    torch.cuda.synchronize()
    for _ in range(10):
        got = []
        for s, j in zip(streams, jobs):
            with torch.cuda.stream(s):
                got.append(work(j))
        torch.cuda.synchronize()
        for g, w in zip(got, want):
            for a, b in zip(g, w):
                assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.gpu
def test_a_captured_call_has_scratch_of_its_own():
    """A call captured without a workspace, then eager calls that grow this thread's scratch:
    every replay still gives the eager result."""
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(4)
    X = torch.from_numpy(rng.standard_normal((30000, 9)).astype(np.float32)).to(dev)
    C = X[:300].clone()
    big = torch.from_numpy(rng.standard_normal((200000, 9)).astype(np.float32)).to(dev)
    want = [t.clone() for t in kq.kq_fit_layer(X, C, 4)]
    out = [torch.empty_like(t) for t in want]
    s = torch.cuda.Stream(dev)
    s.wait_stream(torch.cuda.current_stream(dev))
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        kq.kq_fit_layer(X, C, 4, *out)
    for _ in range(4):
        for t in out:
            t.zero_()
        g.replay()
        kq.kq_fit_layer(big, big[:900].clone(), 2)
        torch.cuda.synchronize()
        for a, b in zip(out, want):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
