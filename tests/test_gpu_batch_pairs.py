"""Batch tiles with two sweeps per launch, side by side and in turn, and with one, against the CPU oracle: replicas whose
runs end after the first or the second sweep of a launch, past a chunk of class orders, and two runs in a row."""
import numpy as np
import pytest

import oracle
from paper_1309_4349_amd import kk, workloads as wl

pytestmark = pytest.mark.gpu


def _job(i, L, sweeps, layout="int8"):
    return wl.Job(L=L, composition=0.4, omega=0.7 if i % 2 else -0.4, seed=wl.job_seed(65, i), sweeps=sweeps, layout=layout)


# few workgroups (side by side); a tile too tall for it (in turn); int8 lattices in more than 256 workgroups (in turn);
# bit-packed ones in more than 1024 (one sweep); replicas without a sweep
@pytest.mark.parametrize("jobs,tile", [
    ([_job(i, L, n) for i, (L, n) in enumerate([(400, 3), (36, 258), (404, 2), (100, 1), (300, 0)])], None),
    ([_job(i, 400, n, "int8") for i, n in enumerate((1, 2, 5))], (8, 128, 2)),
    ([_job(i, L, n, "bitpacked") for i, (L, n) in enumerate([(416, 5), (512, 4), (320, 1)])], (16, 20, 1)),
    ([_job(i, 300 + 4 * (i % 5), i % 4) for i in range(40)], (8, 50, 2)),
    ([_job(i, 320, i % 3, "bitpacked") for i in range(40)], (8, 16, 2)),
])
def test_batch_two_sweeps_match_oracle(jobs, tile):
    print(f"case batch pairs {len(jobs)} replicas tile={tile}", flush=True)
    b = kk.Batch(jobs)
    if tile is not None:
        b.set_tile(*tile)
    refs = [oracle.init(j.L, j.composition, j.seed) for j in jobs]
    for rnd in range(2):
        b.run()
        for i, j in enumerate(jobs):
            acc = oracle.sweeps(refs[i], j.omega, j.seed, rnd * j.sweeps, j.sweeps)
            s = b.sim(i)
            assert np.array_equal(s.get_lattice(), refs[i]), (rnd, i, j.L, j.sweeps)
            assert s.stats()[0] == (rnd + 1) * j.sweeps
    b.close()
