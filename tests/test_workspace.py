"""The binding's own scratch buffers: one per thread and stream, a bounded number of them, none kept from a capture."""
import threading

import pytest
import torch

from paper_2505_10526_amd import binding


@pytest.fixture
def host(monkeypatch):
    """The buffers on the CPU, with the current stream and the capture state as the test sets them."""
    state = {"stream": 1, "capturing": False}
    monkeypatch.setattr(binding, "_stream_handle", lambda: state["stream"])
    monkeypatch.setattr(binding, "_capturing", lambda: state["capturing"])
    monkeypatch.setattr(binding, "_scratch", binding._Scratch())
    monkeypatch.setattr(binding, "_recorded", [])
    return state


def at(nbytes=1 << 20):
    return binding.workspace(nbytes, "cpu")


def test_streams_and_threads_have_buffers_of_their_own(host):
    first = at()
    assert at(100) is first                                  # the next call on the stream waits for this one anyway
    host["stream"] = 2
    other = at()
    assert other.data_ptr() != first.data_ptr()
    host["stream"] = 1
    assert at() is first
    got = []
    t = threading.Thread(target=lambda: got.append(at()))
    t.start()
    t.join()
    assert got[0].data_ptr() not in (first.data_ptr(), other.data_ptr())
    bigger = at(3 << 20)
    assert bigger.numel() >= 3 << 20 and at() is bigger


def test_the_number_of_buffers_is_bounded(host):
    for s in range(50):
        host["stream"] = s
        at()
    assert len(binding._scratch.buffers) == binding._Scratch.LIMIT
    host["stream"] = 49
    last = at()
    for s in (48, 47, 49):
        host["stream"] = s
        at()
    assert at() is last


def test_capture_keeps_nothing_and_loses_nothing(host):
    host["capturing"] = True
    a, b = at(), at()
    assert a is not b and not binding._scratch.buffers       # the graph's memory, one a call
    host["capturing"] = False
    warm = at()
    host["capturing"] = True
    assert at() is warm and at() is warm
    host["capturing"] = False
    assert at(5 << 20) is not warm
    assert len(binding._recorded) == 1 and binding._recorded[0] is warm      # a replay may still use it


@pytest.mark.gpu
def test_stream_handle_is_the_current_streams():
    assert binding._stream_handle() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(torch.cuda.Stream()) as _:
        assert binding._stream_handle() == torch.cuda.current_stream().cuda_stream != torch.cuda.default_stream().cuda_stream


@pytest.mark.gpu
def test_two_streams_at_once():
    """Split products on two streams, no workspace given: each result is the one it has alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    M, N, K = 60, 3584, 18944
    assert binding.load().massv_linear_workspace(M, N, K, binding.BF16) > 4 * M * N      # partial sums between two launches
    x = [torch.randn(M, K, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2)]
    w = binding.weight_pack(torch.randn(N, K, generator=g, device="cuda").mul_(0.02).to(torch.bfloat16))
    alone = [binding.linear(t, w) for t in x]
    streams = [torch.cuda.Stream() for _ in range(2)]
    out = [[torch.empty_like(alone[0]) for _ in range(20)] for _ in range(2)]
    torch.cuda.synchronize()
    for i in range(20):
        for j, s in enumerate(streams):
            with torch.cuda.stream(s):
                binding.linear(x[j], w, out=out[j][i])
    torch.cuda.synchronize()
    for j in range(2):
        assert all(torch.equal(o, alone[j]) for o in out[j])


@pytest.mark.gpu
def test_a_recorded_call_replays_beside_eager_ones():
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    M, N, K = 60, 3584, 18944
    x = torch.randn(M, K, generator=g, device="cuda").to(torch.bfloat16)
    w = binding.weight_pack(torch.randn(N, K, generator=g, device="cuda").mul_(0.02).to(torch.bfloat16))
    want, out = binding.linear(x, w), torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        binding.linear(x, w, out=out)
    for i in range(4):
        out.zero_()
        binding.linear(x[: 20 + i], w)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
