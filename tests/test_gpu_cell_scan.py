"""The cell sort's prefix sum on grids whose blocks sum the totals before them
themselves (1024^2: 512 blocks) and on larger ones (2048^2 and 4096^2: 2048 and 8192
blocks), through the density that the deposit makes of the sorted particles: every
node against the same sum in NumPy, and the sum over all nodes.

A node adds at most a few tens of weights below 1 in FP64: 1e-13 of their size is
left to another order of the sum and the rounding of (x + L) / h (N / 2 units of
eps in a coordinate).
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


@pytest.mark.parametrize("N", [1024, 2048, 4096])
def test_sorted_density(torch_cuda, N):
    from paper_2012_00881_amd import Simulation
    print(f"[case] cell scan N={N}", flush=True)
    n0 = 0.02
    cfg = wi.scaled(wi.config("C1"), n_cells=N, ppc_side=1, n0=n0)
    st = wi.synthetic_state(cfg, seed=N, p_max=0.1, xi=1.0)
    x, y, L = st["x"], st["y"], cfg["half_width"]
    h = 2.0 * L / N
    # the right half empties into the middle: cells without particles and full ones
    right = x > 0.5 * L
    x[right] = 0.5 * x[right]
    sim = Simulation(cfg)
    sim.set_state(particles=np.stack([x, y, st["px"], st["py"]]), xi=1.0, dxi=0.01)
    sim.step()
    n = sim.moments()[0].cpu().numpy()
    sim.close()
    sx, sy = (x + L) / h, (y + L) / h
    a, b = np.minimum(sx.astype(np.int64), N - 1), np.minimum(sy.astype(np.int64), N - 1)
    dx, dy = sx - a, sy - b
    ref = np.zeros((N + 1) ** 2)
    for oy, wy in ((0, 1.0 - dy), (1, dy)):
        for ox, wx in ((0, 1.0 - dx), (1, dx)):
            ref += np.bincount((b + oy) * (N + 1) + a + ox, weights=wx * wy, minlength=ref.size)
    ref = n0 * ref.reshape(N + 1, N + 1)
    eps = np.finfo(np.float64).eps
    err = np.abs(n - ref).max() / ref.max()
    print(f"difference {err:.1e}", flush=True)
    assert err <= 1e-13 + N * eps
    assert abs(n.sum() - n0 * x.size) <= 1e-9 * n0 * x.size
