"""Poisson solves on grids of at most 64^2 by the exact products in one workgroup
(tolerance mode with mg_max_cycles >= 16; V-cycles where fewer are allowed)
against the solution by sine sums in extended precision.

Tolerance: a solve ends at ||r|| <= mg_rtol ||f|| or at the rounding floor
||r|| <= F = 0.35 eps (8/h^2 ||u|| + ||f||), with r as the solver forms it; its
rounding is at most another 3 F (eps per term of ||L_h|| ||u|| + ||f||).  Hence
||u - u*|| <= (mg_rtol ||f|| + 4 F) / lambda_min, lambda_min = (8/h^2) sin^2(pi/2N).
"""
import numpy as np
import pytest

import wandqs_inputs as wi

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _exact(f, h):
    n = f.shape[-1] - 1
    k = np.arange(1, n, dtype=np.longdouble)
    pi = 2 * np.arcsin(np.longdouble(1))
    S = np.sin(pi * np.outer(k, k) / n)
    s2 = np.sin(pi * k / (2 * n)) ** 2
    lam = -(4 / np.longdouble(h) ** 2) * (s2[:, None] + s2[None, :])
    u = np.zeros(f.shape, dtype=np.longdouble)
    u[1:-1, 1:-1] = (np.longdouble(2) / n) ** 2 * (S @ ((S @ f[1:-1, 1:-1].astype(np.longdouble) @ S) / lam) @ S)
    return u


@pytest.mark.parametrize("N", [8, 16, 32, 64])
@pytest.mark.parametrize("nrhs,precision,cycles", [(1, "fp64", 16), (2, "fp64", 50), (2, "mixed", 50),
                                                   (2, "fp64", 15)])
def test_small_poisson_matches_sine_sums(torch_cuda, N, nrhs, precision, cycles):
    from paper_2012_00881_amd import Simulation
    print(f"[case] small Poisson N={N} nrhs={nrhs} {precision} {cycles}", flush=True)
    rng = np.random.default_rng(N + nrhs)
    h = 12.0 / N
    cfg = wi.scaled(wi.config("C1"), n_cells=N, half_width=6.0, precision=precision, mg_max_cycles=cycles)
    sim = Simulation(cfg)
    for rep in range(3):  # later batches are sized by the solve before
        f = np.zeros((nrhs, N + 1, N + 1))
        f[:, 1:-1, 1:-1] = rng.standard_normal((nrhs, N - 1, N - 1))
        f[0] *= 10.0 ** (rep - 1)
        u0 = np.zeros_like(f)
        if rep:
            u0[:, 1:-1, 1:-1] = rng.standard_normal((nrhs, N - 1, N - 1))
        st, u, cyc, _ = sim.mg_solve(f, u0=u0)
        assert st == 0
        u = u.cpu().numpy()
        for r in range(nrhs):
            n = np.linalg.norm
            floor = 0.35 * EPS * (8.0 / h ** 2 * n(u[r]) + n(f[r]))
            bound = (cfg["mg_rtol"] * n(f[r]) + 4 * floor) / (8.0 / h ** 2 * np.sin(np.pi / (2 * N)) ** 2)
            err = float(np.sqrt(((u[r] - _exact(f[r], h)) ** 2).sum()))
            print(f"cycles {cyc} error / bound {err / bound:.2e}", flush=True)
            assert err <= bound
            for edge in (u[r][0], u[r][-1], u[r][:, 0], u[r][:, -1]):
                assert np.all(edge == 0.0)
        if cycles >= 16:
            assert cyc <= 4
    sim.close()
