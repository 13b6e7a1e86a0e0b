"""The GMRES smoothing over many workgroups on large 2D meshes.  Its inner
products are left as one partial sum per workgroup, which the next launch's
workgroups add up: at most 768 a column, so that adding them stays small beside
the vectors however large the mesh.  Sizes sit around a wavefront's and a
workgroup's worth of partial sums (64, 65, 256, 257), the last mesh with one
chunk of nodes a workgroup (627^2 nodes) and the first with two and three;
five iterations and seven (beyond the register forms).  Against the oracle's
smoothing 1e-10, as for the smaller meshes.  A smoothing of sixteen times the
nodes has to take less than sixteen times as long."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _time(f, reps):
    f()
    torch.cuda.synchronize()
    best = float("inf")
    for _ in range(5):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            f()
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1) / reps)
    return best


@pytest.mark.parametrize("n,its,nrhs", [(180, 5, 2), (181, 5, 2), (361, 5, 2), (362, 7, 1), (512, 5, 2), (626, 5, 1),
                                        (627, 5, 2), (627, 7, 1), (885, 5, 1), (886, 6, 1)])
def test_smoothing_matches_oracle(n, its, nrhs):
    from oracle import multigrid
    from oracle.operators import combine
    from oracle import fem
    from paper_2506_18694_amd import Solver
    import workloads as W
    from gpu_util import rel_l2, to_dev, to_host
    k, dh = n / 6.4, 2.0
    K, M, MG = fem.assemble(2, n)
    L = combine(K, M, MG, (1.0, dh * dh - k * k - 2j * dh * k * k, dh - 1j * k * k))
    lev = multigrid.Level(n, L.tocsr())
    b = W.random_complex((nrhs, (n + 1) ** 2), 13)
    s = Solver(2, n, 1, k, 0.0, dh, cycle="w", smooth_its=its, restart=1)
    x = to_host(s.vcycle(to_dev(b)))
    s.close()
    ref = np.stack([multigrid.gmres_jacobi(lev, np.zeros_like(bi), bi, its) for bi in b])
    assert rel_l2(x, ref) < 1e-10


def test_smoothing_time_is_linear_in_the_nodes():
    from paper_2506_18694_amd import Solver
    ms = {}
    for n, reps in ((512, 40), (2048, 10)):
        s = Solver(2, n, 1, 20.0, 0.0, 2.0, cycle="w", restart=1)
        b = torch.randn(1, (n + 1) ** 2, dtype=torch.complex128, device="cuda")
        ms[n] = _time(lambda: s.vcycle(b), reps)
        s.close()
    assert ms[2048] < 16 * ms[512]
