"""How the binding orders a lattice's stream against torch's for device arrays, with stand-ins for
torch's streams and events and for the library, and on the GPU."""

import threading
import time

import numpy as np
import pytest
import torch

import gauge_inputs as gi
from paper_1412_3655_amd import gf

LATTICE = 0x1000  # the lattice's handle and its stream's


class _Stream:
    def __init__(self, handle, idle=True):
        self.cuda_stream = handle
        self.idle = idle

    def query(self):
        if self.idle is None:
            raise RuntimeError("operation not permitted when stream is capturing")
        return self.idle

    def wait_event(self, event):
        LOG.append((self.cuda_stream, "waits for", event.of))


class _Event:
    of = None

    def record(self, stream):
        self.of = stream.cuda_stream
        time.sleep(0.02)  # another thread runs


class _Tensor:
    is_cuda = True
    dtype = torch.float64
    device = torch.device("cuda", 1)

    def is_contiguous(self):
        return True

    def numel(self):
        return 16 * 72

    def data_ptr(self):
        return 256

    def record_stream(self, stream):
        LOG.append((stream.cuda_stream, "uses the tensor"))


LOG = []
LOCAL = threading.local()


@pytest.fixture
def binding(monkeypatch):
    """Sets the stream that is torch's current one for the calling thread."""
    LOG.clear()
    monkeypatch.setattr(gf, "_LATTICES", {LATTICE: gf._Record(LATTICE)})
    monkeypatch.setattr(gf, "gf_lattice_info", lambda lat: (16, 0))
    monkeypatch.setattr(gf, "gf_lattice_group", lambda lat: 3)
    monkeypatch.setattr(gf, "_is_device_tensor", lambda t: isinstance(t, _Tensor))
    monkeypatch.setattr(gf, "_call", lambda name, *a: LOG.append((LATTICE, name)))
    monkeypatch.setattr(torch.cuda, "current_stream", lambda dev=None: LOCAL.stream)
    monkeypatch.setattr(torch.cuda, "default_stream", lambda dev=None: _Stream(0))
    monkeypatch.setattr(torch.cuda, "ExternalStream", lambda h, device=None: _Stream(h))
    monkeypatch.setattr(torch.cuda, "Event", _Event)
    # what torch answers for the device that is current, another one than the tensor's
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: False)

    def current(stream):
        LOCAL.stream = stream

    return current


@pytest.mark.parametrize("call", [gf.gf_set_links, gf.gf_get_links])
def test_capturing_stream_is_not_asked(binding, call):
    """A stream that the tensor's device captures, while another device is current."""
    binding(_Stream(0x2000, idle=None))
    call(LATTICE, _Tensor())
    assert LOG.index((LATTICE, "waits for", 0x2000)) < LOG.index((LATTICE, call.__name__ + "_device"))


def test_idle_default_stream_is_not_waited_for(binding):
    for idle in (True, False):
        binding(_Stream(0, idle))
        LOG.clear()
        gf.gf_set_links(LATTICE, _Tensor())
        assert ((LATTICE, "waits for", 0) in LOG) == (not idle)


@pytest.mark.parametrize("call", [gf.gf_set_links, gf.gf_get_links])
def test_threads_share_a_lattice(binding, call):
    """Each thread's call comes behind what that thread's current stream was given, though the
    threads take turns between any two steps."""
    go = threading.Barrier(2)
    failed = []

    def thread(handle):
        try:
            binding(_Stream(handle))
            go.wait()
            call(LATTICE, _Tensor())
        except Exception as e:  # noqa: BLE001
            failed.append(e)

    threads = [threading.Thread(target=thread, args=(h,)) for h in (0x2000, 0x3000)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed
    before = [entry for entry in LOG if entry[:2] == (LATTICE, "waits for")]
    assert sorted(of for _, _, of in before) == [0x2000, 0x3000]
    if call is gf.gf_get_links:  # and each current stream behind the lattice's
        assert {entry for entry in LOG if entry[0] != LATTICE} == {(h, "waits for", LATTICE) for h in (0x2000, 0x3000)}


@pytest.mark.gpu
def test_beside_another_threads_capture():
    """Links from and to device arrays, on a stream of torch's other than the default one, while
    another thread captures: the calls work and so does the capture."""
    dims = (6, 4, 4, 6)
    u = gi.gen_links(dims, 0.8, 33)
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

    with gf.Lattice(dims, stream=torch.cuda.Stream()) as lat, torch.cuda.stream(torch.cuda.Stream()):
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
    replay takes the present links, and eager calls in between use the same events."""
    dims = (6, 4, 4, 6)
    links = [torch.from_numpy(gi.gen_links(dims, 0.8, k)).cuda() for k in (34, 35, 36)]
    out, twice, eager = (torch.empty_like(links[0]) for _ in range(3))
    with gf.Lattice(dims, stream=torch.cuda.Stream()) as lat:
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
