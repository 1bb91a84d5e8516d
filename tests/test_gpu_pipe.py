"""Whole-lattice (cyclic) sweep kernel with draw waves ahead of phase waves, and the halo tiles' spare lanes and second
units, against the CPU oracle: exact equality."""
import numpy as np
import pytest

import oracle
from paper_1309_4349_amd import kk, workloads as wl

pytestmark = pytest.mark.gpu


def _check(L, layout, w, n, tile=None, t0=0):
    print(f"case {L} {layout} omega={w} n={n} tile={tile}", flush=True)
    seed = wl.job_seed(62, L)
    ref = oracle.init(L, 0.45, seed)
    with kk.Sim(L, 0.45, w, seed, layout=layout) as s:
        if tile is not None:
            s.set_tile(*tile)
        if t0:
            s.set_lattice(ref, t0)
        acc = oracle.sweeps(ref, w, seed, t0, n)
        s.sweep(n)
        assert np.array_equal(s.get_lattice(), ref)
        assert s.stats()[2] == acc


# every width of the kernel (2 .. 9 words per row: each split of the waves and units), the launch boundary of 256
# sweeps, the sweep counter across 2^32, and both signs of omega
@pytest.mark.parametrize("L,layout,w,n", [(64, "int8", 0.5, 257), (96, "bitpacked", 0.9, 5), (128, "int8", -0.6, 5),
                                          (160, "bitpacked", 0.0, 5), (192, "int8", 1.2, 5), (224, "bitpacked", 0.4, 5),
                                          (256, "int8", 0.88, 4), (288, "bitpacked", -1.1, 4)])
def test_whole_lattice_matches_oracle(L, layout, w, n):
    whole = (0, 0, 2)  # the whole lattice in one workgroup
    _check(L, layout, w, n, whole)
    _check(L, layout, w, 3, whole, t0=2**32 - 2)
    _check(L, layout, w, 4)


# halo tiles whose last wave is mostly spare lanes, with two units per thread of which most threads hold one, and off
# the 32-site grid with ragged last tiles
@pytest.mark.parametrize("L,layout,tile", [(512, "bitpacked", (16, 128, 2)), (320, "int8", (2, 16, 1)),
                                           (404, "int8", (2, 16, 1)), (388, "int8", (8, 64, 2)), (36, "int8", (1, 16, 1)),
                                           (416, "bitpacked", (4, 30, 1))])
def test_halo_tiles_match_oracle(L, layout, tile):
    _check(L, layout, 0.8, 3, tile)
    _check(L, layout, -0.5, 2, tile)


# two sweeps in one launch: side by side with one and with two units per thread, in turn, windows taller and wider than
# the lattice, one sweep left over, and the counter's 2^32 between the two
@pytest.mark.parametrize("L,layout,tile", [(416, "bitpacked", (2, 20, 1)), (404, "int8", (8, 64, 1)),
                                           (512, "bitpacked", (16, 128, 2)), (576, "int8", (8, 256, 2)),
                                           (404, "int8", (16, 96, 2)), (36, "int8", (1, 12, 1)), (36, "int8", (2, 36, 1)),
                                           (320, "int8", (4, 160, 2)), (4, "int8", None), (2724, "int8", None)])
def test_two_sweeps_per_launch_match_oracle(L, layout, tile):
    _check(L, layout, 0.8, 5 if L < 1000 else 2, tile)
    _check(L, layout, -0.5, 2, tile, t0=2**32 - 1)
