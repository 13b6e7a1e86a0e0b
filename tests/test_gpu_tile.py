"""The LDS-tile passes of the small 2D launches against the register-streaming
ones.  The number of columns in a launch decides which of them run; both give
every node the same roundings, so a column alone (16-row tiles), among a few
(32-row tiles) and among many (streaming kernels) has to come out bit for bit
the same.  Sizes sit at and around the tile edges (20, 24, 26 and 28 owned
columns) and include the smallest streaming mesh."""

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,levels,faces", [(16, 2, 0), (36, 3, 15), (56, 3, 0), (88, 4, 3), (92, 3, 9),
                                            (104, 3, 0), (208, 4, 0)])
def test_column_does_not_depend_on_the_launch_size(n, levels, faces, precision):
    from paper_2506_18694_amd import Solver
    many = 4 * (3200 // n) ** 2 // 16 + 9
    g = torch.Generator(device="cuda").manual_seed(n)
    v = torch.randn(many, (n + 1) ** 2, dtype=torch.complex128, device="cuda", generator=g)
    s = Solver(2, n, levels, n / 6.4, precision=precision, mg_cycles=3, hss_steps=3, restart=1,
               dirichlet_faces=faces)
    if faces:
        mask = torch.ones(n + 1, n + 1, device="cuda")
        for f, at in enumerate(((slice(None), 0), (slice(None), n), (0, slice(None)), (n, slice(None)))):
            if faces >> f & 1:
                mask[at] = 0
        v = v * mask.reshape(-1)
    b = v if precision == "fp64" else v.to(torch.complex64)
    zs, xs = s.precondition(v), s.vcycle(b)
    for cols in (1, 7):
        assert torch.equal(s.precondition(v[:cols].contiguous()), zs[:cols])
        assert torch.equal(s.vcycle(b[:cols].contiguous()), xs[:cols])
    s.close()
