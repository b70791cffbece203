"""nu_pre and nu_post of the non-uniform multigrid: on the levels of at most 64^2 a
cycle takes (nu + 1) / 2 line steps before and after the coarse correction, so
three sweeps asked for contract more than one.
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


@pytest.mark.parametrize("N", [32, 64])
@pytest.mark.parametrize("nu", [(3, 1), (1, 3), (3, 3)])
def test_more_sweeps_contract_more(torch_cuda, N, nu):
    from paper_2012_00881_amd import Simulation
    print(f"[case] line steps N={N} nu={nu}", flush=True)
    X = wi.nonuniform_axis(N, 4.0, "regions")
    rng = np.random.default_rng(N)
    J = rng.standard_normal((N + 1, N + 1))
    M = -rng.uniform(0.0, 3.0, (N + 1, N + 1))
    M[[0, -1]] = 0.0
    M[:, [0, -1]] = 0.0

    def rel_after(nu_pre, nu_post, cycles):
        sim = Simulation(wi.scaled(wi.config("C1"), n_cells=N, nu_pre=nu_pre, nu_post=nu_post,
                                   mg_max_cycles=cycles))
        _, _, cyc, rel = sim.nu_mg_solve(X, X, J, M=M)
        sim.close()
        assert cyc == cycles
        return rel

    one, more = rel_after(1, 1, 4), rel_after(*nu, 4)
    print(f"residual after 4 cycles {one:.2e}, with more sweeps {more:.2e}", flush=True)
    assert more < 0.5 * one
    assert rel_after(2, 2, 4) == one
