"""Rates of the 3D passes against yardsticks measured beside them (the best of
several timings each): an operator pass and the zero-guess sweep against a copy
of the vector, which moves the same bytes, a residual against an addition of its
vectors, and many columns of a small mesh against fewer of a larger one with as
many nodes."""

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _ms(f, reps):
    f()
    torch.cuda.synchronize()
    best = float("inf")
    for _ in range(6):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            f()
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1) / reps)
    return best


def _step(n, levels, nrhs, precision):
    from paper_2506_18694_amd import Solver
    dt = torch.complex128 if precision == "fp64" else torch.complex64
    g = torch.Generator(device="cuda").manual_seed(n)
    x, b, y = (torch.randn(nrhs, (n + 1) ** 3, dtype=dt, device="cuda", generator=g) for _ in range(3))
    s = Solver(3, n, levels, n / 6.4, precision=precision, mg_cycles=2, hss_steps=1, restart=1)
    return s, x, b, y


def test_operator_runs_near_the_copy_rate():
    s, x, b, y = _step(256, 6, 1, "fp64")
    assert _ms(lambda: s.apply("L", x), 20) < 1.2 * _ms(lambda: y.copy_(x), 20)
    s.close()


def test_residual_of_many_columns_runs_near_the_rate_of_an_addition():
    # 16 columns of 128^3: 275 MB a vector, beyond every cache
    s, x, b, y = _step(128, 6, 16, "fp32")
    assert _ms(lambda: s.hss_residual(b, x), 20) < 1.7 * _ms(lambda: torch.add(b, x, out=y), 20)
    s.close()


def test_zero_guess_sweep_runs_near_the_copy_rate():
    s, x, b, y = _step(128, 6, 16, "fp32")
    assert _ms(lambda: s.jacobi(b), 20) < 1.2 * _ms(lambda: y.copy_(x), 20)
    s.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_columns_of_a_small_mesh_cost_what_their_nodes_do(precision):
    from paper_2506_18694_amd import Solver
    ms = {}
    for n, levels, nrhs in ((80, 5, 16), (128, 6, 4)):  # 8.5M and 8.6M nodes
        s = Solver(3, n, levels, n / 6.4, precision=precision, mg_cycles=3, hss_steps=4, restart=1)
        v = torch.randn(nrhs, (n + 1) ** 3, dtype=torch.complex128, device="cuda")
        ms[n] = _ms(lambda: s.precondition(v), 3)
        s.close()
    assert ms[80] < 1.25 * ms[128]
