"""GPU: whole rings of a batch of fewer than 64 replicas, in one launch, against the CPU oracle: rings on bit planes and a
byte per site, uneven runs, replicas without a sweep, and handles whose tile changes between two runs."""
import numpy as np
import pytest

import oracle
from paper_1309_4349_amd import kk, workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sides,sweeps", [([140], [3]), ([12, 100, 140, 36, 156, 132, 76, 52], [5, 66, 0, 1, 4, 2, 1030, 9])])
def test_few_whole_rings_match_oracle(sides, sweeps):
    jobs = [wl.Job(L, 0.45, -0.5 if i % 3 == 2 else 0.6, wl.job_seed(66, i), n) for i, (L, n) in enumerate(zip(sides, sweeps))]
    print(f"case few rings {sides}", flush=True)
    b = kk.TriBatch(jobs)
    assert b.info() == {"resident": 0, "batched": 0, "plain": len(jobs), "tile_jobs": 0}
    acc = [0] * len(jobs)
    refs = [oracle.init_rect(j.L, j.L, j.composition, j.seed) for j in jobs]
    for rnd in range(3):
        b.run()
        for i, j in enumerate(jobs):
            acc[i] += oracle.tri_sweeps(refs[i], j.omega, j.seed, rnd * j.sweeps, j.sweeps)
            s = b.sim(i)
            assert np.array_equal(s.get_lattice(), refs[i]), (rnd, i)
            assert s.stats() == ((rnd + 1) * j.sweeps, (rnd + 1) * j.sweeps * j.L * j.L, acc[i])
        if rnd == 0:
            b.sim(0).tri_set_tile(0)  # a launch per class
        elif rnd == 1:
            b.sim(0).tri_set_tile(sides[0], sides[0])
            if len(jobs) > 1:
                b.sim(2).tri_set_tile(16, 16)
    b.close()
