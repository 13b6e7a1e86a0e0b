"""A column's 3D result does not depend on how many columns share its launches,
bit for bit: the number of columns chooses between the forms of the block
passes and, from 7 MB a vector on, between blocks and marching passes, which
give every node the same roundings.  Sizes sit at the edges of the regions (10
and 12 owned columns of 16, 12 owned rows and 28 owned columns of the marching
passes) on both sides of 96 cells, where the marching passes take over for any
number, with Dirichlet faces; three cycles a step run every pass.  One column
among many is also held against the one-node-per-thread kernels (an independent
path): a few hundred roundings per value, 1e-12 in FP64, 2e-4 in FP32."""

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32", 2e-4)])
@pytest.mark.parametrize("n,levels,faces", [(12, 2, 0), (12, 3, 21), (24, 3, 0), (28, 3, 24), (36, 3, 0), (48, 4, 63),
                                            (56, 4, 0), (80, 5, 0), (88, 4, 3), (96, 6, 0), (112, 5, 42)])
def test_column_does_not_depend_on_the_launch_size(n, levels, faces, precision, tol):
    from paper_2506_18694_amd import Solver
    bytes_col = (n + 1) ** 3 * (16 if precision == "fp64" else 8)
    many = max(3, 7000000 // bytes_col + 1)
    kw = dict(precision=precision, mg_cycles=3, hss_steps=2, restart=1, dirichlet_faces=faces)
    g = torch.Generator(device="cuda").manual_seed(n)
    v = torch.randn(many, (n + 1) ** 3, dtype=torch.complex128, device="cuda", generator=g)
    mask = torch.ones(n + 1, n + 1, n + 1, device="cuda")
    for f in range(6):
        if faces >> f & 1:
            mask.select(2 - f // 2, n if f & 1 else 0).fill_(0)
    v = (v * mask.reshape(-1)).contiguous()
    b = v if precision == "fp64" else v.to(torch.complex64)
    s = Solver(3, n, levels, n / 6.4, **kw)
    zs, xs = s.precondition(v), s.vcycle(b)
    for cols in sorted({1, 2, many // 3 + 1, many - 1}):
        assert torch.equal(s.precondition(v[:cols].contiguous()), zs[:cols])
        assert torch.equal(s.vcycle(b[:cols].contiguous()), xs[:cols])
    s.close()
    r = Solver(3, n, levels, n / 6.4, streaming=False, **kw)
    for z, y in ((zs, r.precondition(v[-1:].contiguous())), (xs, r.vcycle(b[-1:].contiguous()))):
        assert torch.linalg.vector_norm(z[-1] - y[0]) < tol * torch.linalg.vector_norm(y[0])
    r.close()
