"""The fused GMRES smoothing of 2D levels against the oracle's (modified
Gram-Schmidt, numpy least squares), one smoothing from zero and, on two levels,
smoothings from a guess: at the edges of the one-workgroup form (1024 and 1089
nodes: two and five nodes per thread; 2500 and 2601: the last it takes and the
first over many workgroups), with one iteration, five, six (the first beyond
the register forms) and twenty, a zero column among others, and odd sizes.
Both orthogonalise to rounding, so the results agree to 1e-10 as the cycles
do."""

import numpy as np
import pytest

from oracle import multigrid, solver as osolver
import workloads as W
from gpu_util import to_dev, to_host, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,levels,its", [(2, 1, 1), (9, 1, 5), (31, 1, 5), (32, 1, 5), (49, 1, 5), (49, 1, 6), (50, 1, 5),
                                          (50, 1, 1), (12, 1, 20), (75, 1, 7), (98, 2, 5), (140, 2, 3)])
def test_smoothing_matches_oracle(n, levels, its):
    from paper_2506_18694_amd import Solver
    k = max(2.0, n / 6.4)
    pr = osolver.Problem(2, n, k, 2.0, levels=levels, cycles=1, cycle="w", smooth_its=its)
    b = W.random_complex((3, (n + 1) ** 2), 11)
    b[1] = 0
    s = Solver(2, n, levels, k, 0.0, 2.0, cycle="w", smooth_its=its, restart=1)
    x = to_host(s.vcycle(to_dev(b)))
    assert np.all(x[1] == 0)
    ref = np.stack([multigrid.wcycle(pr.hierarchy, bi, np.zeros_like(bi), 0, its) for bi in b[[0, 2]]])
    assert rel_l2(x[[0, 2]], ref) < 1e-10
    s.close()
