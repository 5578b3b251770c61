"""theta, F and the plaquette where their launches have uneven shapes.

Blocks are dealt to the 8 XCDs in contiguous runs and one block adds the
partial sums 8 x 256 pairs at a time: extents whose block counts are below 8,
no multiple of 8, and just past one such round, against the oracle.
"""

import numpy as np
import pytest

import gauge_inputs as gi
import oracle
from paper_1412_3655_amd import gf

pytestmark = pytest.mark.gpu


# blocks of 256 sites per colour: 1, 1 (ragged), 17, 41, and 1188 (2376 pairs: one round of 2048 and a rest)
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 6, 2, 10), (12, 10, 8, 10), (14, 10, 10, 16), (24, 24, 24, 44)])
def test_landau_and_plaquette(dims):
    u = gi.gen_links(dims, 0.7, 3)
    th, F = oracle.measure(u, dims)
    P = oracle.plaquette(u, dims)
    with gf.Lattice(dims) as lat:
        lat.set_links(u)
        got_th, got_F = lat.measure()
        got_P = lat.plaquette()
    # float64 sums of V terms of order 1 in different orders: relative 2^-53 sqrt(V), times 8 for margin
    tol = 8 * 2.0**-53 * np.sqrt(gi.volume(dims)) + 1e-15
    assert abs(got_th - th) <= 8 * tol * th
    assert abs(got_F - F) <= tol and abs(got_P - P) <= tol


# a thread or two per site, in columns of tiles: halves below 32768 sites, whole below 65536, then halves of
# 12 reals: one column, two of 24 and 16 tiles whose timeslices are no whole number of tiles (float64), and
# three tiles left over; 8 reals whole
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("reals", [12, 8])
@pytest.mark.parametrize("dims", [(16, 16, 16, 8), (18, 16, 16, 8), (16, 16, 16, 18), (26, 22, 18, 10)])
def test_plaquette_tiles(dims, prec, reals):
    u = gi.gen_links(dims, 0.7, 6)
    with gf.Lattice(dims, gf.GF_FP32 if prec == "f32" else gf.GF_FP64, storage=reals) as lat:
        lat.set_links(u)
        want = oracle.plaquette(lat.get_links(), dims)
        got = lat.plaquette()
    # as above; float32 storage may round row 2 on the way out: a trace / 3 of four links, each within 2^-23
    tol = 8 * 2.0**-53 * np.sqrt(gi.volume(dims)) + 1e-15 if prec == "f64" else 4 * 2.0**-23
    # the 8-real decode, relative 1e-15 per entry on average, much less over the lattice
    assert abs(got - want) <= tol + (1e-13 if reals == 8 else 0.0)


@pytest.mark.parametrize("dims", [(4, 6, 2, 10), (14, 10, 10, 6), (24, 24, 24, 2)])
def test_coulomb_slices(dims):
    u = gi.gen_links(dims, 0.7, 4)
    with gf.Lattice(dims, gauge=gf.GF_COULOMB) as lat:
        lat.set_links(u)
        th, F = lat.measure_timeslices()
    want_th, want_F = oracle.coulomb_measure(u, dims)[:2]
    tol = 8 * 2.0**-53 * np.sqrt(gi.volume(dims)) + 1e-15
    assert np.abs(np.max(th) - np.max(want_th)) <= 8 * tol * np.max(want_th)
    assert np.abs(np.mean(F) - np.mean(want_F)) <= tol


@pytest.mark.parametrize("dims", [(4, 6, 2, 10), (14, 10, 10, 16)])
def test_su2(dims):
    u = gi.gen_links_su2(dims, 0.7, 5)
    th, F = oracle.su2lat_measure(u, dims)
    P = oracle.su2lat_plaquette(u, dims)
    with gf.Lattice(dims, group=2) as lat:
        lat.set_links(u)
        got_th, got_F = lat.measure()
        got_P = lat.plaquette()
    tol = 8 * 2.0**-53 * np.sqrt(gi.volume(dims)) + 1e-15
    assert abs(got_th - th) <= 8 * tol * th
    assert abs(got_F - F) <= tol and abs(got_P - P) <= tol


@pytest.mark.parametrize("group", [3, 2])
@pytest.mark.parametrize("dims", [(4, 6, 2, 10), (14, 10, 10, 6), (24, 24, 24, 2), (2, 2, 2, 38)])
def test_every_slice(dims, group):
    """Timeslice by timeslice: a block's tile and timeslice come out of one number."""
    u = (gi.gen_links if group == 3 else gi.gen_links_su2)(dims, 0.7, 4)
    with gf.Lattice(dims, gauge=gf.GF_COULOMB, group=group) as lat:
        lat.set_links(u)
        th, F = lat.measure_timeslices()
    want_th, want_F = (oracle.coulomb_measure if group == 3 else oracle.su2lat_coulomb_measure)(u, dims)[:2]
    tol = 8 * 2.0**-53 * np.sqrt(gi.volume(dims) / dims[3]) + 1e-15
    assert np.all(np.abs(np.asarray(th) - want_th) <= 8 * tol * np.asarray(want_th))
    assert np.all(np.abs(np.asarray(F) - want_F) <= tol)
