"""The LDS-resident cycle of the small 2D levels and the coarse solve against
the oracle, at the edges of their ranges: the largest finest small level (36
cells in FP32, 32 in FP64: three nodes on some threads), the smallest, a
coarsest mesh of 100 nodes (the last the kernel takes), of 121 and of 400 (the
many-workgroup solve), and hierarchies down to one cell.  Tolerances: one cycle
is a few hundred roundings per value, 1e-12 in FP64; in FP32 6e-8 each, 2e-4 as
for the other FP32 cycles."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32", 2e-4)])
@pytest.mark.parametrize("n,levels", [(72, 4), (64, 4), (64, 7), (40, 4), (40, 3), (8, 3), (16, 5), (76, 3)])
def test_cycle_matches_oracle(n, levels, precision, tol):
    from oracle import solver as osolver
    from paper_2506_18694_amd import Solver
    import workloads as W
    from gpu_util import rel_l2, to_dev, to_host
    k = n / 6.4
    b = W.random_complex((3, (n + 1) ** 2), 7)
    if precision == "fp32":
        b = b.astype(np.complex64)
    s = Solver(2, n, levels, k, precision=precision, restart=1)
    x = to_host(s.vcycle(to_dev(b, "complex128" if precision == "fp64" else "complex64")))
    pr = osolver.Problem(2, n, k, k, levels=levels)
    ref = np.stack([pr.vcycle(bi) for bi in b.astype(np.complex128)])
    assert rel_l2(x, ref) < tol
    s.close()
