"""Slices after a non-uniform solve on the same context, which keeps its line
factors in the arrays of the earlier slices' fields.

A solve that meets the stop rule without a cycle leaves the fields as they were,
so the slices behind it are the same bits as without it, whatever its factors hold
(M = 4 / h^2 makes the first pivot of every line 0 and the factors undefined).
After a solve with cycles the slices start from another guess and agree to the
rounding floor of the field solves (1e-10, as the parity tests).
"""
import numpy as np
import pytest

import wandqs_inputs as wi

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _slices(N, solve, n=6, **kw):
    from paper_2012_00881_amd import Simulation
    cfg = wi.scaled(wi.config("C1"), n_cells=N, half_width=8.0, dxi0=0.02, **kw)
    st = wi.synthetic_state(cfg, seed=N, p_max=0.2, xi=1.0)
    p = np.stack([st["x"], st["y"], st["px"], st["py"]])
    sim = Simulation(cfg)
    sim.set_state(particles=p, xi=1.0, dxi=0.02)
    if solve:
        solve(sim)
    out = []
    for _ in range(n):
        F, _ = sim.step(fields=True)
        out.append(F.cpu())
    out.append(sim.get_state()["particles"].cpu())
    sim.close()
    return out


@pytest.mark.parametrize("N", [64, 128, 256, 512])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_slices_after_a_solve_without_cycles(torch_cuda, N, precision):
    print(f"[case] slices after an undefined factorisation N={N} {precision}", flush=True)
    X = np.linspace(-8.0, 8.0, N + 1)
    M = np.full((N + 1, N + 1), 4.0 / (16.0 / N) ** 2)

    def solve(sim):
        st, _, cyc, _ = sim.nu_mg_solve(X, X, np.zeros((N + 1, N + 1)), M=M)
        assert st == 0 and cyc == 0

    for a, b in zip(_slices(N, None, precision=precision), _slices(N, solve, precision=precision)):
        assert torch_cuda.equal(a, b)


@pytest.mark.parametrize("N", [64, 256])
def test_slices_after_a_solve(torch_cuda, N):
    print(f"[case] slices after a non-uniform solve N={N}", flush=True)
    X = wi.nonuniform_axis(N, 8.0, "regions")
    J = np.random.default_rng(N).standard_normal((N + 1, N + 1))

    def solve(sim):
        st, _, cyc, _ = sim.nu_mg_solve(X, X, J)
        assert st == 0 and cyc >= 1

    for a, b in zip(_slices(N, None), _slices(N, solve)):
        assert float((a - b).norm()) <= 1e-10 * float(a.norm())


@pytest.mark.parametrize("N", [64, 256])
@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_a_state_set_after_an_undefined_solve(torch_cuda, N, bad):
    print(f"[case] state after a solve with {bad} N={N}", flush=True)
    X = wi.nonuniform_axis(N, 8.0, "regions")
    J = np.ones((N + 1, N + 1))
    J[N // 2, N // 2] = bad

    def solve(sim):
        keep = sim.get_state()
        st, _, _, _ = sim.nu_mg_solve(X, X, J)
        assert st != 0
        sim.set_state(particles=keep["particles"], fields=keep["fields"], xi=keep["xi"], dxi=keep["dxi"])

    for a, b in zip(_slices(N, None), _slices(N, solve)):
        assert torch_cuda.equal(a, b)
