"""Poisson and Helmholtz solves by turns on one context: the batch that a solve
starts with is sized by the last solve of its own kind, so the other kind between
them changes neither the bits nor the count.
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


@pytest.mark.parametrize("N", [64, 256, 512])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_alternating_solves_equal_repeated_ones(torch_cuda, N, precision):
    from paper_2012_00881_amd import Simulation
    t = torch_cuda
    print(f"[case] alternating solves N={N} {precision}", flush=True)
    rng = np.random.default_rng(N)
    f = np.zeros((1, N + 1, N + 1))
    f[:, 1:-1, 1:-1] = rng.standard_normal((1, N - 1, N - 1))
    k2 = rng.uniform(0.0, 3.0, (N + 1, N + 1))
    cfg = wi.scaled(wi.config("C1"), n_cells=N, precision=precision)

    def solves(kinds):
        sim = Simulation(cfg)
        out = []
        for helm in kinds:
            st, u, cyc, _ = sim.mg_solve(f, k2=k2 if helm else None)
            assert st == 0
            out.append((cyc, u.cpu()))
        sim.close()
        return out

    for helm in (False, True):
        other = solves([helm, not helm, helm, not helm, helm])[::2]
        for (ca, a), (cb, b) in zip(other, solves([helm] * 3)):
            assert ca == cb
            assert t.equal(a, b)
