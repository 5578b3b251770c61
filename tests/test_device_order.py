"""How links move between a lattice on a stream of its own and device arrays of torch's: in the
order of torch's current stream, whatever else it, the lattice's stream and other threads do."""

import threading

import numpy as np
import pytest
import torch

import gauge_inputs as gi
from paper_1412_3655_amd import gf

DIMS = (6, 4, 4, 6)


class _Stream:
    def __init__(self, handle):
        self.cuda_stream = handle


class _Tensor:
    is_cuda = True
    dtype = torch.float64
    device = torch.device("cuda", 1)
    held = None

    def is_contiguous(self):
        return True

    def numel(self):
        return 16 * 72

    def data_ptr(self):
        return 256

    def record_stream(self, stream):
        self.held = stream.cuda_stream


@pytest.mark.parametrize("handle", [0, 0x2000])
@pytest.mark.parametrize("call", [gf.gf_set_links, gf.gf_get_links])
def test_stream_of_the_tensors_device(monkeypatch, call, handle):
    """The library gets torch's current stream on the tensor's device, which need not be the
    current device, and torch holds the memory for it."""
    streams = {torch.device("cuda", 1): _Stream(handle)}
    calls = []
    monkeypatch.setattr(gf, "gf_lattice_info", lambda lat: (16, 0))
    monkeypatch.setattr(gf, "gf_lattice_group", lambda lat: 3)
    monkeypatch.setattr(gf, "_is_device_tensor", lambda t: isinstance(t, _Tensor))
    monkeypatch.setattr(gf, "_call", lambda *a: calls.append(a))
    monkeypatch.setattr(torch.cuda, "current_stream", lambda dev: streams[dev])
    t = _Tensor()
    call(7, t)
    assert calls == [(call.__name__ + "_device_on", 7, 256, handle or None)]
    assert t.held == handle


def test_arguments_without_device():
    for name in ("gf_set_links_device_on", "gf_get_links_device_on"):
        assert getattr(gf.lib(), name)(None, None, None) == gf.GF_E_ARG


def _links(k):
    return torch.from_numpy(gi.gen_links(DIMS, 0.8, k)).cuda()


@pytest.mark.gpu
def test_beside_another_threads_capture():
    """Links from and to device arrays, on a stream of torch's other than the default one, while
    another thread captures: the calls work and so does the capture."""
    u = gi.gen_links(DIMS, 0.8, 33)
    src = torch.from_numpy(u).cuda()
    out = torch.empty_like(src)
    x = torch.ones(64, device="cuda")
    graph, begun, ended = torch.cuda.CUDAGraph(), threading.Event(), threading.Event()
    captured, failed = [], []

    def capture():
        try:
            with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
                captured.append(x * 2)
                begun.set()
                ended.wait(60)
        except Exception as e:  # noqa: BLE001
            failed.append(e)
            begun.set()

    with gf.Lattice(DIMS, stream=torch.cuda.Stream()) as lat, torch.cuda.stream(torch.cuda.Stream()):
        lat.set_links(src)
        lat.get_links(out)
        torch.cuda.synchronize()
        out.fill_(0.0)
        other = threading.Thread(target=capture)
        other.start()
        try:
            assert begun.wait(60)
            lat.set_links(src)
            lat.get_links(out)
        finally:
            ended.set()
            other.join()
        assert not failed
        torch.cuda.synchronize()
    graph.replay()
    torch.cuda.synchronize()
    assert float(captured[0].sum()) == 128.0
    assert np.array_equal(out.cpu().numpy()[:, :, :2], u[:, :, :2])


@pytest.mark.gpu
def test_captured_with_torchs_work():
    """Links taken by a graph that torch captures, from a lattice on a stream of its own: every
    replay takes the present links, with eager calls in between."""
    links = [_links(k) for k in (34, 35, 36)]
    out, twice, eager = (torch.empty_like(links[0]) for _ in range(3))
    with gf.Lattice(DIMS, stream=torch.cuda.Stream()) as lat:
        lat.set_links(links[0])
        lat.get_links(out)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
            lat.get_links(out)
            torch.mul(out, 2.0, out=twice)
        for u in (*links, links[0]):
            lat.set_links(u)
            lat.sweep(1, 1.7)
            lat.get_links(eager)
            torch.cuda.synchronize()
            out.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, eager) and torch.equal(twice, 2.0 * eager)


@pytest.mark.gpu
@pytest.mark.parametrize("side", [False, True])
def test_source_overwritten_at_once(side):
    """The lattice's stream has 10 ms of waiting before the links can be taken, and torch
    overwrites them as soon as the call is back."""
    src = _links(37)
    u = src.cpu().numpy()
    own = torch.cuda.Stream()
    with gf.Lattice(DIMS, stream=own) as lat, torch.cuda.stream(torch.cuda.Stream() if side else None):
        torch.cuda.synchronize()
        with torch.cuda.stream(own):
            torch.cuda._sleep(20_000_000)
        lat.set_links(src)
        src.fill_(float("nan"))
        got = lat.get_links()
    assert np.array_equal(got[:, :, :2], u[:, :, :2])


@pytest.mark.gpu
def test_sweeps_wait_for_the_links_that_are_taken():
    """Torch's stream has 10 ms of waiting before it takes the links, and the lattice's stream is
    given sweeps as soon as the call is back."""
    src = _links(38)
    out = torch.empty_like(src)
    with gf.Lattice(DIMS, stream=torch.cuda.Stream()) as lat:
        lat.set_links(src)
        torch.cuda.synchronize()
        torch.cuda._sleep(20_000_000)
        lat.get_links(out)
        lat.sweep(3, 1.7)
        swept = lat.get_links()
    assert np.array_equal(out.cpu().numpy()[:, :, :2], src.cpu().numpy()[:, :, :2])
    assert not np.array_equal(swept, out.cpu().numpy())


@pytest.mark.gpu
def test_threads_take_links_of_one_lattice():
    """Two threads with streams of their own, each of which overwrites its array before each call."""
    src = _links(39)
    want = src.cpu().numpy()[:, :, :2]
    failed = []

    def take(lat):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                out = torch.empty_like(src)
                for _ in range(20):
                    torch.cuda._sleep(200_000)
                    out.fill_(float("nan"))
                    lat.get_links(out)
                    if not np.array_equal(out.cpu().numpy()[:, :, :2], want):
                        failed.append("other links")
        except Exception as e:  # noqa: BLE001
            failed.append(e)

    with gf.Lattice(DIMS, stream=torch.cuda.Stream()) as lat:
        lat.set_links(src)
        torch.cuda.synchronize()
        threads = [threading.Thread(target=take, args=(lat,)) for _ in range(2)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
    assert not failed
