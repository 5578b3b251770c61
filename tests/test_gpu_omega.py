"""Sweeps whose omega, rule or precision changes from call to call on one lattice: the power of the
exact float64 rule is kept with the lattice and has to be that of the sweep."""

import numpy as np
import pytest

import gauge_inputs as gi
from paper_1412_3655_amd import gf

pytestmark = pytest.mark.gpu

DIMS = (4, 4, 4, 6)
EXACT, BINOMIAL = gf.GF_OR_EXACT, gf.GF_OR_BINOMIAL1


@pytest.mark.parametrize("group", [3, 2])
def test_rule_and_omega_change(group):
    u = (gi.gen_links if group == 3 else gi.gen_links_su2)(DIMS, 0.7, 41)
    with gf.Lattice(DIMS, group=group) as lat:
        lat.set_links(u)
        for omega, mode in ((1.7, BINOMIAL), (1.7, EXACT), (1.3, EXACT), (1.9, BINOMIAL), (1.9, EXACT), (1.0, EXACT)):
            with gf.Lattice(DIMS, group=group) as fresh:
                fresh.set_links(lat.get_links())
                fresh.sweep(1, omega, mode)
                want = fresh.get_links()
            lat.sweep(1, omega, mode)
            assert np.array_equal(lat.get_links(), want), (omega, mode)


@pytest.mark.parametrize("storage", [12, 8])
def test_precision_changes(storage):
    with gf.Lattice(DIMS, gf.GF_MIXED, storage=storage) as lat, gf.Lattice(DIMS) as ref:
        lat.set_links(gi.gen_links(DIMS, 0.7, 42))
        lat.sweep(3, 1.7)  # float32
        lat.promote_fp64()
        ref.set_links(lat.get_links())
        for lattice in (lat, ref):
            lattice.sweep(3, 1.7)
        assert np.array_equal(lat.get_links(), ref.get_links())
