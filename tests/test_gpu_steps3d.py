"""The single steps of a 3D level (operator, residual, Jacobi sweep, zero-guess
sweep, restricted residual) through the marching passes, against the
one-node-per-thread kernels (an independent path): at the edges of a region's
owned columns (30 and 14 of 32 and 16), on meshes of two cells and more, with
one to three columns and Dirichlet faces, and on both sides of 4M nodes, where
the FP32 residual changes its regions.  A step is a few tens of roundings per
value: 1e-13 in FP64, 2e-5 in FP32."""

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-13), ("fp32", 2e-5)])
@pytest.mark.parametrize("n,levels,nrhs,faces", [(2, 2, 3, 0), (4, 2, 1, 0), (12, 2, 2, 5), (16, 3, 1, 0), (28, 3, 3, 0),
                                                 (32, 4, 1, 48), (56, 4, 1, 0), (64, 5, 2, 0), (88, 4, 3, 10),
                                                 (128, 6, 1, 0), (160, 6, 1, 0)])
def test_steps_match_node_kernels(n, levels, nrhs, faces, precision, tol):
    from paper_2506_18694_amd import Solver
    kw = dict(precision=precision, mg_cycles=2, hss_steps=1, restart=1, dirichlet_faces=faces)
    g = torch.Generator(device="cuda").manual_seed(n)
    dt = torch.complex128 if precision == "fp64" else torch.complex64
    mask = torch.ones(n + 1, n + 1, n + 1, device="cuda")
    for f in range(6):
        if faces >> f & 1:
            mask.select(2 - f // 2, n if f & 1 else 0).fill_(0)
    x, b = ((torch.randn(nrhs, (n + 1) ** 3, dtype=dt, device="cuda", generator=g) * mask.reshape(-1)).to(dt)
            for _ in range(2))
    a, r = Solver(3, n, levels, n / 6.4, **kw), Solver(3, n, levels, n / 6.4, streaming=False, **kw)
    for step in (lambda s: s.apply("L", x), lambda s: s.apply("B0", x), lambda s: s.hss_residual(b, x),
                 lambda s: s.jacobi(b, x), lambda s: s.jacobi(b), lambda s: s.restrict_residual(x, b)):
        u, v = step(a), step(r)
        assert torch.linalg.vector_norm(u - v) < tol * torch.linalg.vector_norm(v)
    a.close()
    r.close()
