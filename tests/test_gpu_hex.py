"""Bit-plane kernels of the triangular lattice against the CPU oracle, at the edges of their tiles: exact equality."""
import numpy as np
import pytest

import oracle
from paper_1309_4349_amd import kk, workloads as wl

pytestmark = pytest.mark.gpu


def _check(L, H, scheme, tile, x, w, n, t0=0):
    print(f"case hex {scheme} {L}x{H} tile={tile} omega={w}", flush=True)
    seed = wl.job_seed(61, L * 1000 + H)
    run = oracle.tri_sweeps if scheme == "classes" else oracle.mpkk_steps
    ref = oracle.init_rect(L, H, x, seed)
    s = kk.Sim(L, x, w, seed, geometry="triangular", rows=H, scheme=scheme)
    if tile is not None:
        s.tri_set_tile(*tile)
    if t0:
        s.set_lattice(ref, t0)
    acc = run(ref, w, seed, t0, n)
    s.sweep(n)
    assert np.array_equal(s.get_lattice(), ref)
    assert s.stats()[2] == acc
    s.close()


# the smallest tile on the smallest ring; a width of 32 bit groups and one more site; a tile wider than the bit words
# and one taller than the LDS (both cut into parts); widths off the multiple of 4; one column of 4 sites left over; the
# sign of omega, omega = 0 and thresholds of 0
@pytest.mark.parametrize("L,H,tile,x,w", [
    (84, 84, (16, 16), 0.5, 0.8), (612, 180, (440, 40), 0.5, 0.6), (612, 180, (441, 40), 0.5, 0.6),
    (1020, 84, (900, 16), 0.4, 0.9), (396, 400, (57, 300), 0.5, 0.5), (244, 124, (121, 37), 0.3, -0.7),
    (148, 100, (72, 20), 0.5, 0.0), (132, 132, (17, 63), 0.5, 9.0), (100, 88, (32, 22), 0.6, -6.0),
])
def test_hex_class_tiles_match_oracle(L, H, tile, x, w):
    _check(L, H, "classes", tile, x, w, 3)
    _check(L, H, "classes", tile, x, w, 2, t0=2**32 - 1)


# as above for the literal MPKK (31 groups of 14 columns at most), on rings with an even and an odd number of domains:
# past the ring's end the even and odd domains trade classes
@pytest.mark.parametrize("L,H,tile,x,w", [
    (59, 63, (16, 16), 0.5, 0.8), (61, 63, (17, 21), 0.5, 0.5), (437, 119, (392, 40), 0.5, 0.6),
    (437, 119, (393, 40), 0.4, 0.9), (801, 63, (700, 17), 0.5, 0.6), (157, 448, (57, 400), 0.5, 0.5),
    (94, 77, (29, 33), 0.3, -0.7), (66, 70, (24, 28), 0.5, 0.0), (59, 70, (16, 27), 0.5, 9.0),
])
def test_hex_mpkk_tiles_match_oracle(L, H, tile, x, w):
    _check(L, H, "mpkk", tile, x, w, 3)
    _check(L, H, "mpkk", tile, x, w, 2, t0=2**32 - 1)
