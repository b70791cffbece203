"""Solves on grids of at most 64^2, which run whole in one workgroup (several
V-cycles a launch): against the oracle at every size, sweep count, form and
operator, and k cycles in one launch against k launches of one.

Tolerance against the oracle: both solutions sit at the rounding floor,
||r|| <= 0.35 eps (8/h^2 ||u|| + ||f||), which bounds their difference by
1.4 eps N^2 of ||u|| (lambda_min >= (8/h^2) / N^2): 1.3e-12 at N = 64.
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


def _inputs(N, seed, nrhs=2):
    rng = np.random.default_rng(seed)
    f = np.zeros((nrhs, N + 1, N + 1))
    f[:, 1:-1, 1:-1] = rng.standard_normal((nrhs, N - 1, N - 1))
    u0 = np.zeros_like(f)
    u0[:, 1:-1, 1:-1] = 0.1 * rng.standard_normal((nrhs, N - 1, N - 1))
    return f, u0, rng.uniform(0.0, 30.0, (N + 1, N + 1))


@pytest.mark.parametrize("N", [8, 16, 32, 64])
@pytest.mark.parametrize("helm", [False, True])
@pytest.mark.parametrize("nu,precision", [((2, 2), "fp64"), ((1, 3), "fp64"), ((3, 1), "mixed")])
def test_small_solve_matches_oracle(torch_cuda, oracle_mod, N, helm, nu, precision):
    from paper_2012_00881_amd import Simulation
    L = 6.0
    print(f"[case] small grid N={N} helm={helm} nu={nu} {precision}", flush=True)
    f, u0, k2 = _inputs(N, 300 + N)
    k2 = k2 if helm else None
    cfg = wi.scaled(wi.config("C1"), n_cells=N, half_width=L, nu_pre=nu[0], nu_post=nu[1],
                    precision=precision)
    sim = Simulation(cfg)
    st, u, cyc, _ = sim.mg_solve(f, u0=u0, k2=k2)
    sim.close()
    assert st == 0
    u = u.cpu().numpy()
    for r in range(2):
        so, ref, co, _ = oracle_mod.mg_solve(N, 2 * L / N, f[r], u0=u0[r], k2=k2)
        assert so == 0
        d = np.linalg.norm(u[r] - ref) / np.linalg.norm(ref)
        print(f"cycles {cyc} oracle {co} difference {d:.2e}", flush=True)
        assert d <= 1.4 * EPS * N * N
        for edge in (u[r][0], u[r][-1], u[r][:, 0], u[r][:, -1]):
            assert np.all(edge == 0.0)


@pytest.mark.parametrize("N", [8, 16, 32, 64])
@pytest.mark.parametrize("helm", [False, True])
def test_cycles_in_one_launch_equal_single_cycles(torch_cuda, N, helm):
    from paper_2012_00881_amd import Simulation
    print(f"[case] small grid cycles N={N} helm={helm}", flush=True)
    f, u0, k2 = _inputs(N, 400 + N)
    k2 = k2 if helm else None
    base = wi.scaled(wi.config("C1"), n_cells=N, mg_rtol=0.0)
    sim = Simulation(wi.scaled(base, mg_max_cycles=3))
    _, u3, _, _ = sim.mg_solve(f, u0=u0, k2=k2)
    sim.close()
    sim = Simulation(wi.scaled(base, mg_max_cycles=1))
    u = u0
    for _ in range(3):
        _, u, _, _ = sim.mg_solve(f, u0=u, k2=k2)
    sim.close()
    assert np.array_equal(u.cpu().numpy(), u3.cpu().numpy())
    assert float(u3.abs().max()) > 0.0
