"""Poisson solves in the tolerance mode on grids of 128^2 .. 2048^2: the exact
sine-transform iteration on the finest level against the V-cycles, which a
caller that allows fewer than 16 cycles keeps.

Tolerance: both end at the rounding floor, ||r|| <= 0.35 eps (8/h^2 ||u|| +
||f||) with ||f|| <= 8/h^2 ||u||, so the solutions differ by at most
2 * 0.35 * 2 * eps * 8/h^2 / lambda_min of ||u||, lambda_min >= (8/h^2) / N^2
(sin x >= 2x/pi): 1.4 eps N^2.
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


def _solve(N, f, u0, max_cycles, precision="fp64"):
    from paper_2012_00881_amd import Simulation
    sim = Simulation(wi.scaled(wi.config("C1"), n_cells=N, mg_max_cycles=max_cycles,
                               precision=precision))
    st, u, cyc, rel = sim.mg_solve(f, u0=u0)
    sim.close()
    return st, u.cpu().numpy(), cyc, rel


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("N,nrhs", [(128, 1), (128, 2), (256, 2), (512, 1), (1024, 2), (2048, 1)])
def test_direct_matches_vcycles(torch_cuda, N, nrhs, precision):
    print(f"[case] Poisson direct N={N} nrhs={nrhs} {precision}", flush=True)
    rng = np.random.default_rng(N + nrhs)
    f = np.zeros((nrhs, N + 1, N + 1))
    f[:, 1:-1, 1:-1] = rng.standard_normal((nrhs, N - 1, N - 1))
    u0 = np.zeros_like(f)
    u0[:, 1:-1, 1:-1] = 0.1 * rng.standard_normal((nrhs, N - 1, N - 1))
    sd, ud, cd, rd = _solve(N, f, u0, 16, precision)
    sv, uv, cv, _ = _solve(N, f, u0, 15, precision)
    assert sd == 0 and sv == 0
    print(f"cycles {cd} against {cv}, rel {rd}", flush=True)
    assert cd < cv  # the route: iterations of the exact solve, not V-cycles
    for r in range(nrhs):
        d = np.linalg.norm(ud[r] - uv[r]) / np.linalg.norm(uv[r])
        assert d <= 1.4 * EPS * N * N, d
        for edge in (ud[r][0], ud[r][-1], ud[r][:, 0], ud[r][:, -1]):
            assert np.all(edge == 0.0)


def test_direct_zero_rhs_and_nan(torch_cuda):
    """f = 0 from a nonzero guess ends at u ~ 0 (the tolerance is then relative
    to the first residual); a NaN ends in WANDQS_E_NOCONV, as V-cycles do."""
    N = 128
    u0 = np.zeros((1, N + 1, N + 1))
    u0[:, 1:-1, 1:-1] = np.random.default_rng(1).standard_normal((1, N - 1, N - 1))
    st, u, _, _ = _solve(N, np.zeros_like(u0), u0, 50)
    assert st == 0
    # one exact solve leaves the transform's rounding, at most a few 1e-14 of u0
    assert np.abs(u).max() <= 1e-13 * np.abs(u0).max()
    f = np.zeros_like(u0)
    f[0, 5, 7] = np.nan
    st, _, _, _ = _solve(N, f, None, 50)
    assert st == -4
