"""Initial placement by counted keys and one ordered bin, against the CPU oracle: exact equality."""
import numpy as np
import pytest

import oracle
from paper_1309_4349_amd import kk

pytestmark = pytest.mark.gpu


# fewer sites than a workgroup's threads, whole and ragged rounds of them, more than one round per workgroup; one site,
# all but one, and counts that end a bin early or late
@pytest.mark.parametrize("L,layout", [(4, "int8"), (32, "bitpacked"), (36, "int8"), (416, "bitpacked"), (1036, "int8"),
                                      (2048, "bitpacked")])
def test_placement_matches_oracle(L, layout):
    N = L * L
    for k, n1 in enumerate((1, 2, N // 3, N // 2, N // 2 + 1, N - 1)):
        print(f"case place {L} {layout} n1={n1}", flush=True)
        with kk.Sim(L, n1 / N, 0.5, 100 + k, layout=layout) as s:
            assert np.array_equal(s.get_lattice(), oracle.init(L, n1 / N, 100 + k))


@pytest.mark.parametrize("L,H,scheme", [(12, 8, "classes"), (100, 96, "classes"), (145, 147, "mpkk")])
def test_ring_placement_matches_oracle(L, H, scheme):
    for k, x in enumerate((0.001, 0.37, 0.5, 0.999)):
        print(f"case place ring {L}x{H} x={x}", flush=True)
        with kk.Sim(L, x, 0.5, 200 + k, geometry="triangular", rows=H, scheme=scheme) as s:
            assert np.array_equal(s.get_lattice(), oracle.init_rect(L, H, x, 200 + k))
