"""Helmholtz V-cycles in a thin plasma, where k2 is close to 0 everywhere and the
cycle has to be as good as the Poisson one: a wide smooth source, k2 = n0 = 0.02
in a disc and 0 elsewhere, half width 6 (h^2 k2 <= 0.05 on the 8-cell level).

A V(2,2) cycle of the textbook contracts by 0.04 .. 0.07 here (the range that the
CPU solver's pin asserts for the Poisson problem): eight cycles from a zero guess
leave ||r|| <= 0.07^8 ||f|| = 5.8e-10 ||f||, and 11 of them reach 1e-12.
"""
import numpy as np
import pytest

import wandqs_inputs as wi

pytestmark = pytest.mark.gpu

L, N0, RATE = 6.0, 0.02, 0.07


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _inputs(N, nrhs):
    g = np.linspace(-L, L, N + 1)
    X, Y = g[None, :], g[:, None]
    f = np.stack([np.exp(-((X - 1.0 - r) ** 2 + Y ** 2)) for r in range(nrhs)])
    f[:, [0, -1]] = 0.0
    f[:, :, [0, -1]] = 0.0
    return f, N0 * ((X ** 2 + Y ** 2) < 4.0)


def _residual(u, f, k2, h):
    c = u[1:-1, 1:-1]
    lap = (u[1:-1, :-2] + u[1:-1, 2:] + u[:-2, 1:-1] + u[2:, 1:-1] - 4.0 * c) / h ** 2
    return np.linalg.norm(f[1:-1, 1:-1] - (lap - k2[1:-1, 1:-1] * c)) / np.linalg.norm(f)


def _cfg(N, **kw):
    return wi.scaled(wi.config("C1"), n_cells=N, half_width=L, n0=N0, nu_pre=2, nu_post=2, **kw)


@pytest.mark.parametrize("N", [8, 16, 32, 64, 128, 256, 512])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_fixed_cycles_contract_like_the_textbook(torch_cuda, N, precision):
    from paper_2012_00881_amd import Simulation
    from paper_2012_00881_amd.wandqs import mg_solve_noalloc
    f, k2 = _inputs(N, 2)
    cfg = _cfg(N, mg_rtol=0.0, mg_max_cycles=8, precision=precision)
    print(f"[case] thin plasma N={N} {precision}", flush=True)
    sim = Simulation(cfg)
    st, u, _, _ = sim.mg_solve(f, k2=k2)
    sim.close()
    assert st == 0
    out = [u.cpu().numpy()]
    if N <= 256:
        st, v = mg_solve_noalloc(cfg, f, k2=k2)
        torch_cuda.cuda.synchronize()
        assert st == 0
        out.append(v.cpu().numpy())
    worst = max(_residual(w[r], f[r], k2, 2 * L / N) for w in out for r in range(2))
    print(f"residual {worst:.2e}", flush=True)
    assert worst <= RATE ** 8


@pytest.mark.parametrize("N", [64, 128, 256, 512])
def test_tolerance_solves_need_no_more_cycles(torch_cuda, N):
    from paper_2012_00881_amd import Simulation
    f, k2 = _inputs(N, 1)
    sim = Simulation(_cfg(N, mg_rtol=1e-12, mg_max_cycles=11))
    print(f"[case] thin plasma tolerance N={N}", flush=True)
    st, u, cyc, _ = sim.mg_solve(f, k2=k2)
    sim.close()
    print(f"cycles {cyc}", flush=True)
    assert st == 0, cyc
