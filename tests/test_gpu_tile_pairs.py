"""The two-level launches of the small 2D levels against the same passes one
level per launch.  The number of columns in a launch decides whether a pair of
levels shares its launches, up to 256 workgroups on the way down and 1024 on
the way up; every node gets the same roundings either way, so a column alone,
among a few (only the way up is paired) and among many (no pair) has to come
out bit for bit the same, and one cycle has to agree with the oracle's.  Sizes
sit around the owned columns of a region (12 down, 28 up), with both parities
of the number of streaming levels."""

import pytest

torch = pytest.importorskip("torch")

import workloads as W
from gpu_util import rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,levels,faces", [(64, 3, 0), (48, 3, 0), (56, 3, 5), (96, 4, 10), (112, 4, 0),
                                            (172, 3, 0), (192, 5, 15)])
def test_levels_do_not_depend_on_sharing_a_launch(n, levels, faces, precision):
    from paper_2506_18694_amd import Solver
    g = torch.Generator(device="cuda").manual_seed(n)
    down = (n // 2 // 6 + 1) ** 2
    many = 1024 // (((n // 28) + 1) * (n // 12 + 1)) * 5 + 5
    v = torch.randn(many, (n + 1) ** 2, dtype=torch.complex128, device="cuda", generator=g)
    for f, at in enumerate(((slice(None), 0), (slice(None), n), (0, slice(None)), (n, slice(None)))):
        if faces >> f & 1:
            v.view(many, n + 1, n + 1)[(slice(None),) + at] = 0
    b = v if precision == "fp64" else v.to(torch.complex64)
    s = Solver(2, n, levels, n / 6.4, precision=precision, mg_cycles=2, hss_steps=2, restart=1,
               dirichlet_faces=faces)
    xs, zs = s.vcycle(b), s.precondition(v)
    for cols in (1, 2, 256 // down + 1):
        assert torch.equal(s.vcycle(b[:cols].contiguous()), xs[:cols])
        assert torch.equal(s.precondition(v[:cols].contiguous()), zs[:cols])
    s.close()


@pytest.mark.parametrize("n,levels", [(48, 3), (112, 4), (192, 5)])
def test_paired_cycle_matches_the_oracle(n, levels):
    from oracle import multigrid, solver as osolver
    from paper_2506_18694_amd import Solver
    k = n / 6.4
    pr = osolver.Problem(2, n, k, k, levels=levels, cycles=1)
    b = W.random_complex((1, pr.L.shape[0]), 5)
    s = Solver(2, n, levels, k, 0.0, k, restart=1)
    x = to_host(s.vcycle(to_dev(b)))
    ref = multigrid.vcycle(pr.hierarchy, b[0])
    # rounding only; the coarse solves differ by their condition number times it
    assert rel_l2(x[0], ref) < 1e-10
    s.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,levels,faces", [(64, 3, 0), (100, 3, 6), (144, 3, 0), (208, 5, 9)])
def test_finest_level_shares_the_launch_of_an_odd_one(n, levels, faces, precision):
    """One (or three) streaming levels below the finest: the odd level's
    post-smoothing runs in the finest level's four-sweep and update passes, up
    to 400 and 1024 workgroups."""
    from paper_2506_18694_amd import Solver
    g = torch.Generator(device="cuda").manual_seed(n)
    many = 1024 // (((n // 28) + 1) * (n // 12 + 1)) + 2
    v = torch.randn(many, (n + 1) ** 2, dtype=torch.complex128, device="cuda", generator=g)
    for f, at in enumerate(((slice(None), 0), (slice(None), n), (0, slice(None)), (n, slice(None)))):
        if faces >> f & 1:
            v.view(many, n + 1, n + 1)[(slice(None),) + at] = 0
    s = Solver(2, n, levels, n / 6.4, precision=precision, mg_cycles=3, hss_steps=3, restart=1,
               dirichlet_faces=faces)
    zs = s.precondition(v)
    for cols in (1, 3, 400 // (n // 20 + 1) ** 2 + 1):
        assert torch.equal(s.precondition(v[:cols].contiguous()), zs[:cols])
    s.close()
