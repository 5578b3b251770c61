"""Canonical links in and out of the device layout at the edges of its 64-site tiles.

Volumes below one tile, with a part-filled last tile, and one that the pool
moves through its staging buffer in two chunks of which the first is no multiple
of a tile; device arrays at the alignment of a double.
"""

import numpy as np
import pytest
import torch

import gauge_inputs as gi
from paper_1412_3655_amd import gf

pytestmark = pytest.mark.gpu

DIMS = [(2, 2, 2, 2), (6, 2, 2, 4), (2, 4, 2, 6), (10, 6, 4, 6)]


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("prec,storage", [(gf.GF_FP64, 12), (gf.GF_FP64, 8), (gf.GF_FP32, 12), (gf.GF_FP32, 8),
                                          (gf.GF_MIXED, 12), (gf.GF_MIXED, 8)])
def test_round_trip(dims, prec, storage):
    u = gi.gen_links(dims, 0.8, 11)
    flat = torch.empty(u.size + 1, dtype=torch.float64, device="cuda")
    dev = flat[1:].view(u.shape)  # 8 bytes past a 16-byte boundary
    dev.copy_(torch.from_numpy(u))
    back = torch.zeros(u.size + 1, dtype=torch.float64, device="cuda")
    out = back[1:].view(u.shape)
    with gf.Lattice(dims, prec, storage=storage) as lat:
        lat.set_links(dev)
        lat.get_links(out)
        host = lat.get_links()
        if prec == gf.GF_MIXED:
            lat.promote_fp64()  # g = 1: the float64 links as they came
            d = lat.get_links()
            assert np.abs(d - u).max() <= 1e-14
    got = out.cpu().numpy()
    assert np.array_equal(got, host)
    assert float(back[0]) == 0.0
    # row 2 is rebuilt; 8 reals: a few roundings of the codec, float32 ones of 2^-24
    tol = 1e-13 if prec == gf.GF_FP64 else 2e-6
    assert np.abs(got - u).max() <= tol
    if storage == 12 and prec == gf.GF_FP64:
        assert np.array_equal(got[:, :, :2], u[:, :, :2])
    if storage == 12 and prec != gf.GF_FP64:
        assert np.array_equal(got[:, :, :2], u[:, :, :2].astype(np.float32).astype(np.float64))


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("prec", [gf.GF_FP64, gf.GF_FP32])
def test_round_trip_su2(dims, prec):
    u = gi.gen_links_su2(dims, 0.8, 12)
    with gf.Lattice(dims, prec, group=2) as lat:
        lat.set_links(u)
        got = lat.get_links()
    assert np.abs(got - u).max() <= (1e-15 if prec == gf.GF_FP64 else 2.0**-23)


@pytest.mark.parametrize("reals", [12, 8])
def test_pool_moves_a_lattice_in_chunks(reals):
    dims = (16, 16, 16, 16)  # 65536 sites through a buffer of 58254
    u = gi.gen_links(dims, 0.8, 13)
    with gf.Pool(1 << 30, 2, gf.GF_MIXED, reals32=reals) as pool:
        assert pool.admit(1, dims, u, max_sweeps=0)
        pool.step()
        assert [d["job_id"] for d in pool.poll()] == [1]
        got = pool.fetch_links(1)
    assert np.abs(got - u).max() <= 1e-14


@pytest.mark.parametrize("busy", [False, True])
def test_device_arrays_are_ordered_after_torch(busy):
    """A lattice on its own stream takes links that torch's current stream has yet to produce
    (busy: behind 10 ms of waiting) and fills an array that torch has yet to write, twice over."""
    dims = (6, 4, 4, 6)
    links = [gi.gen_links(dims, 0.8, k) for k in (31, 32)]
    out = torch.empty(links[0].shape, dtype=torch.float64, device="cuda")
    with gf.Lattice(dims, stream=torch.cuda.Stream()) as lat:
        for u in links:
            src = torch.from_numpy(u).cuda()
            torch.cuda.synchronize()
            if busy:
                torch.cuda._sleep(20_000_000)
            tmp = src * 1.0
            lat.set_links(tmp)
            del tmp
            if busy:
                torch.cuda._sleep(20_000_000)
                out.fill_(float("nan"))
            lat.get_links(out)
            got = (out * 1.0).cpu().numpy()
            assert np.array_equal(got[:, :, :2], u[:, :, :2])
