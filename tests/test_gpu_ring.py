"""Whole rings of the triangular lattice on bit planes, and a byte per site where a ring has no equal segments, against
the CPU oracle: exact equality."""
import numpy as np
import pytest

import oracle
from paper_1309_4349_amd import kk, workloads as wl

pytestmark = pytest.mark.gpu


def _check(L, H, x, w, n, t0=0):
    print(f"case ring {L}x{H} omega={w} n={n} t0={t0}", flush=True)
    seed = wl.job_seed(63, L * 1000 + H)
    ref = oracle.init_rect(L, H, x, seed)
    with kk.Sim(L, x, w, seed, geometry="triangular", rows=H) as s:
        s.tri_set_tile(L, H)
        if t0:
            s.set_lattice(ref, t0)
        acc = oracle.tri_sweeps(ref, w, seed, t0, n)
        s.sweep(n)
        assert np.array_equal(s.get_lattice(), ref)
        assert s.stats()[2] == acc


# 3 segments of 3 words per class (the least), of 5; 25 and 19 segments; 1, 2, 3 and 4 waves per class, the most words;
# none (148 = 4 * 37); past 64 class orders and past one launch's sweeps; the sign of omega, omega = 0, thresholds of 0
@pytest.mark.parametrize("L,H,x,w,n", [
    (12, 12, 0.5, 0.5, 200), (20, 12, 0.4, -0.8, 70), (100, 100, 0.5, 0.4, 1030), (76, 76, 0.5, 0.0, 20),
    (100, 96, 0.6, -6.0, 20), (132, 132, 0.5, 0.9, 70), (244, 160, 0.3, -0.7, 9), (260, 280, 0.5, 9.0, 5),
    (388, 200, 0.5, 0.6, 5), (148, 148, 0.5, 0.8, 5), (36, 4, 0.5, 0.8, 9), (4, 24, 0.5, 0.4, 70), (12, 300, 0.5, 0.6, 9),
])
def test_whole_rings_match_oracle(L, H, x, w, n):
    _check(L, H, x, w, n)
    _check(L, H, x, w, 3, t0=2**32 - 2)
    _check(L, H, x, w, 1)


def test_batch_of_rings_of_both_kinds_matches_oracle():
    sides = [12, 52, 60, 76, 100, 132, 148, 204]
    jobs = [wl.Job(sides[i % 8], 0.45, 0.5 if i % 3 else -0.5, wl.job_seed(64, i), (0, 1, 7, 66)[i % 4])
            for i in range(72)]
    b = kk.TriBatch(jobs)
    assert b.info()["resident"] == len(jobs)
    b.run()
    for i, j in enumerate(jobs):
        ref = oracle.init_rect(j.L, j.L, j.composition, j.seed)
        acc = oracle.tri_sweeps(ref, j.omega, j.seed, 0, j.sweeps)
        s = b.sim(i)
        assert np.array_equal(s.get_lattice(), ref), (i, j.L, j.sweeps)
        assert s.stats()[2] == acc
    b.close()
