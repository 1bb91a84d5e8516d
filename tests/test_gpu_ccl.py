"""Cluster histograms from 64 x 64 tiles, and the summed observables, against the CPU oracle: exact equality at whole,
ragged and single tiles, with clusters that cross every edge, wrap around, spiral, and are as many as a tile can hold."""
import numpy as np
import pytest

import oracle
from paper_1309_4349_amd import kk

pytestmark = pytest.mark.gpu


def _patterns(H, L):
    y, x = np.mgrid[0:H, 0:L]
    rng = np.random.default_rng(H * 8192 + L)
    yield "checkerboard", (x + y) % 2
    yield "columns", (x % 4 == 3) * 1
    yield "rows", (y % 4 == 3) * 1
    yield "diagonals", ((x + y) % 5 == 0) * 1
    yield "antidiagonals", ((x - y) % 3 == 0) * 1
    yield "comb", ((x % 2 == 0) | (y == H // 2)) * 1
    yield "snake", ((y % 2 == 0) | (x == np.where(y % 4 == 1, L - 1, 0))) * 1
    yield "frame", ((x % 64 < 2) | (y % 64 > 61)) * 1
    for p in (0.1, 0.41, 0.5, 0.593, 0.9):
        yield f"random {p}", rng.random((H, L)) < p


@pytest.mark.parametrize("L,layout", [(36, "int8"), (64, "bitpacked"), (68, "int8"), (128, "int8"), (192, "bitpacked"),
                                      (132, "int8"), (388, "int8"), (416, "bitpacked")])
def test_square_tiles_match_oracle(L, layout):
    with kk.Sim(L, 0.5, 0.5, 7, layout=layout) as s:
        for name, lat in _patterns(L, L):
            lat = np.ascontiguousarray(lat, dtype=np.uint8)
            print(f"case {L} {layout} {name}", flush=True)
            s.set_lattice(lat)
            for species in (1, 0):
                assert s.cluster_hist(species) == oracle.cluster_hist(lat, species)
            assert s.energy()[0] == oracle.energy(lat)


@pytest.mark.parametrize("L,H", [(12, 12), (60, 64), (68, 60), (76, 132), (132, 196), (20, 132), (260, 128)])
def test_ring_tiles_match_oracle(L, H):
    with kk.Sim(L, 0.5, 0.5, 7, geometry="triangular", rows=H) as s:
        for name, lat in _patterns(H, L):
            lat = np.ascontiguousarray(lat, dtype=np.uint8)
            print(f"case ring {L} x {H} {name}", flush=True)
            s.set_lattice(lat)
            for species in (1, 0):
                assert s.cluster_hist(species) == oracle.tri_cluster_hist(lat, species)
            assert s.energy()[0] == oracle.tri_energy(lat)


@pytest.mark.parametrize("L,H", [(145, 147), (66, 63)])
def test_odd_ring_tiles_match_oracle(L, H):
    with kk.Sim(L, 0.5, 0.5, 7, geometry="triangular", rows=H, scheme="mpkk") as s:
        for name, lat in _patterns(H, L):
            lat = np.ascontiguousarray(lat, dtype=np.uint8)
            print(f"case odd ring {L} x {H} {name}", flush=True)
            s.set_lattice(lat)
            assert s.cluster_hist(1) == oracle.tri_cluster_hist(lat, 1)
            assert s.energy()[0] == oracle.tri_energy(lat)
