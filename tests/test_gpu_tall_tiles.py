"""The tallest tiles that kk_set_tile accepts, one word wide, against the CPU oracle."""
import numpy as np
import pytest

import oracle
from paper_1309_4349_amd import kk, workloads as wl

pytestmark = pytest.mark.gpu


# 990 rows: the tie lists of 16 waves still fit beside the tile; 992 and 996: they do not, and 12 waves run it
@pytest.mark.parametrize("L,layout,rows", [(1024, "bitpacked", 990), (1024, "bitpacked", 992), (1036, "int8", 996)])
def test_one_word_tiles_match_oracle(L, layout, rows):
    print(f"case tile 1 x {rows} on {L}^2 {layout}", flush=True)
    seed = wl.job_seed(71, rows)
    ref = oracle.init(L, 0.4, seed)
    acc = oracle.sweeps(ref, 0.6, seed, 0, 3)
    with kk.Sim(L, 0.4, 0.6, seed, layout=layout) as s:
        s.set_tile(1, rows, 2)
        s.sweep(1)
        s.sweep(2)
        assert np.array_equal(s.get_lattice(), ref)
        assert s.stats() == (3, 3 * L * L, acc)
