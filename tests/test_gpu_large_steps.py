"""Slices with steps of several times a workload's own, where the linear guess of
psi, E_z and B_z lies further off: a run from the cold plasma against the oracle's
slice by slice, as the other run tests, and no field that the exact solve settles
takes more than two iterations (whatever the guess, one exact solve leaves the
transform's rounding and a second one corrects that).
"""
import numpy as np
import pytest

import wandqs_inputs as wi
from parity import FIELD_TOL, check_fields

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("N,dxi", [(32, 0.5), (64, 0.25), (128, 0.2)])
def test_run_with_large_steps(torch_cuda, oracle_mod, N, dxi):
    from paper_2012_00881_amd import Simulation
    cfg = wi.scaled(wi.config("C1"), n_cells=N, dxi0=dxi, n_slices=10)
    orc = oracle_mod.Oracle(cfg)
    st = oracle_mod.initial_state(cfg)
    sim = Simulation(cfg)
    for k in range(cfg["n_slices"]):
        print(f"[case] large steps N={N} slice {k}", flush=True)
        F, info = sim.step(fields=True, info=True)
        assert orc.slice_step(st)["status"] == 0
        check_fields(F.cpu().numpy(), st["fields"], FIELD_TOL, f"slice {k}")
        assert max(info["vcycles"][:3]) <= 2, info["vcycles"]
    sim.close()
