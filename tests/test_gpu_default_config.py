"""The configuration of a lattice that nobody tuned: on both sides of every line of its rule the
links are those of an explicitly set configuration, bit for bit."""

import numpy as np
import pytest

import gauge_inputs as gi
from paper_1412_3655_amd import gf

pytestmark = pytest.mark.gpu

# sites per colour 5120 | 5760, 12096 | 13824 (the lanes change), 40960 | 46080 (heat bath); the last
# one's float64 links in 12 reals are beyond 48 MiB, the others' links below
DIMS = [(8, 8, 10, 16), (8, 8, 10, 18), (12, 12, 12, 14), (12, 12, 12, 16), (16, 16, 16, 20), (16, 16, 18, 20),
        (20, 20, 20, 20)]


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("prec,storage,group", [(gf.GF_FP64, 12, 3), (gf.GF_FP64, 8, 3), (gf.GF_FP32, 12, 3),
                                                (gf.GF_MIXED, 8, 3), (gf.GF_FP64, 12, 2)])
def test_default_gives_the_same_links(dims, prec, storage, group):
    u = (gi.gen_links if group == 3 else gi.gen_links_su2)(dims, 0.7, 21)
    got = []
    for explicit in (False, True):
        with gf.Lattice(dims, prec, group=group, storage=storage) as lat:
            if explicit:
                tps = 4 if group == 3 else 1
                lat.set_sweep_config(tps, 128)
                lat.set_anneal_config(tps, 128)
            lat.set_links(u)
            lat.anneal(1, 1.0, 1.0, 3)
            lat.sweep(2, 1.7)
            got.append(lat.get_links())
    assert np.array_equal(got[0], got[1])
