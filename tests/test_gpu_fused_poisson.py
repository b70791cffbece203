"""The fused up-and-down pass of the finest level in Poisson V-cycles of the
tolerance mode, which a solve runs when mg_max_cycles is below 16 (from 16 on
it iterates with the exact solve), against the separate LDS-tile passes.

The same bits after the same number of cycles.  Where the norms' sums over other
tiles end the solves a cycle apart, both residuals are below mg_rtol ||f||, so the
solutions differ by at most 2 mg_rtol ||f|| / lambda, lambda = 2 (pi / 2L)^2 (1 -
1e-3) the smallest eigenvalue.
"""
import math

import pytest

import wandqs_inputs as wi

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("N", [128, 256, 512, 1024])
@pytest.mark.parametrize("nrhs", [1, 2])
@pytest.mark.parametrize("nu", [1, 2])
def test_fused_poisson_cycles_equal_separate_passes(torch_cuda, monkeypatch, N, nrhs, nu):
    from paper_2012_00881_amd import Simulation
    t = torch_cuda
    L, rtol = 6.0, 1e-9
    g = t.Generator().manual_seed(N + 10 * nu + nrhs)
    f = t.zeros(nrhs, N + 1, N + 1, dtype=t.float64)
    f[:, 1:-1, 1:-1] = t.randn(nrhs, N - 1, N - 1, dtype=t.float64, generator=g)
    cfg = wi.scaled(wi.config("C1"), n_cells=N, half_width=L, nu_pre=nu, nu_post=nu, mg_max_cycles=15,
                    mg_rtol=rtol)
    out = []
    for tiles in ("lds", None):
        if tiles:
            monkeypatch.setenv("WANDQS_MG_TILES", tiles)
        else:
            monkeypatch.delenv("WANDQS_MG_TILES", raising=False)
        print(f"[case] fused Poisson N={N} nrhs={nrhs} nu={nu} {tiles}", flush=True)
        sim = Simulation(cfg)
        sim.profile(True)
        for _ in range(2):  # the second batch is sized by the first solve
            st, u, cyc, _ = sim.mg_solve(f)
            assert st == 0
        names = {k["name"].split("<")[0] for k in sim.kernel_stats() if k["launches"] > 0}
        sim.close()
        assert ("k_mg_updown_reg" in names) == (tiles is None), names
        out.append((u.cpu(), cyc))
    (a, ca), (b, cb) = out
    assert abs(ca - cb) <= 1
    if ca == cb:
        assert t.equal(a, b)
    else:
        lam = 2.0 * (math.pi / (2.0 * L)) ** 2 * (1.0 - 1e-3)
        for r in range(nrhs):
            assert float((a[r] - b[r]).norm()) <= 2.0 * rtol * float(f[r].norm()) / lam
