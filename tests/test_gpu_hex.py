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
