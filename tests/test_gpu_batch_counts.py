"""GPU: attempts and accepted exchanges of every replica of a batch, against the CPU oracle, where a launch makes two sweeps
side by side, two in turn, or one: replicas whose run ends with the first sweep of a launch, replicas without a sweep."""
import numpy as np
import pytest

import oracle
from paper_1309_4349_amd import kk, workloads as wl

pytestmark = pytest.mark.gpu


def _jobs(sides, sweeps, layout):
    return [wl.Job(L=L, composition=0.4, omega=0.7 if i % 2 else -0.4, seed=wl.job_seed(67, i), sweeps=n, layout=layout)
            for i, (L, n) in enumerate(zip(sides, sweeps))]


# side by side: few workgroups; in turn: a tile too tall for it, and int8 in more than 256 workgroups; one: bit-packed in
# more than 1024; 96 and 256 are resident
@pytest.mark.parametrize("sides,sweeps,layout,tile", [
    ((400, 36, 96, 404, 100, 300), (3, 258, 5, 2, 1, 0), "int8", None),
    ((400, 400, 400), (1, 2, 5), "int8", (8, 128, 2)),
    (tuple(300 + 4 * (i % 5) for i in range(40)), tuple(i % 4 for i in range(40)), "int8", (8, 50, 2)),
    ((256,) + (320,) * 40, (3,) + tuple(i % 3 for i in range(40)), "bitpacked", (8, 16, 2)),
])
def test_batch_counts_match_oracle(sides, sweeps, layout, tile):
    jobs = _jobs(sides, sweeps, layout)
    print(f"case batch counts {len(jobs)} replicas tile={tile}", flush=True)
    b = kk.Batch(jobs)
    if tile is not None:
        b.set_tile(*tile)
    refs = [oracle.init(j.L, j.composition, j.seed) for j in jobs]
    acc = [0] * len(jobs)
    for rnd in range(2):
        b.run()
        for i, j in enumerate(jobs):
            acc[i] += oracle.sweeps(refs[i], j.omega, j.seed, rnd * j.sweeps, j.sweeps)
            s = b.sim(i)
            assert s.stats() == ((rnd + 1) * j.sweeps, (rnd + 1) * j.sweeps * j.L * j.L, acc[i]), (rnd, i)
            assert np.array_equal(s.get_lattice(), refs[i]), (rnd, i)
    b.close()
