"""The deposits and the cell sort where cells hold 0, 1, 2, ... and a few hundred
particles (a blowout's sheath), on every number of lattice particles per cell,
against the oracle's slice: the node arrays to 1e-10 of their largest value and
the fields to the parity tolerance, and twice the same bits.
"""
import numpy as np
import pytest

import wandqs_inputs as wi
from parity import FIELD_TOL, check_fields, check_node_arrays

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("N", [16, 64, 128])
@pytest.mark.parametrize("side", [1, 2, 3, 4])
def test_crowded_cells_match_oracle(torch_cuda, oracle_mod, N, side):
    from paper_2012_00881_amd import Simulation
    print(f"[case] crowded cells N={N} side={side}", flush=True)
    # a thin plasma, in which such piles leave 1 + psi > 0
    cfg = wi.scaled(wi.config("C1"), n_cells=N, ppc_side=side, n0=0.02)
    st = wi.synthetic_state(cfg, seed=40 + N + side, p_max=0.3, xi=1.0, field_amp=0.0)
    L, h = cfg["half_width"], 2 * cfg["half_width"] / N
    # piles: the particles of the box's middle third go to the cells of one row and
    # of one column, with counts that grow along them
    x, y = st["x"], st["y"]
    mid = np.flatnonzero((np.abs(x) < L / 3) & (np.abs(y) < L / 3))
    u = wi.uniform01(7, 2 * mid.size)
    cells = np.repeat(np.arange(N), np.minimum(np.arange(N) ** 2 // 8, 300) + 1)[:mid.size]
    k = mid[:cells.size]
    half = k.size // 2
    x[k] = -L + h * (cells + u[:k.size])
    y[k] = -L + h * (N // 2 + u[mid.size:mid.size + k.size])
    x[k[half:]], y[k[half:]] = y[k[half:]].copy(), x[k[half:]].copy()
    count = np.bincount((np.minimum((y + L) // h, N - 1) * N + np.minimum((x + L) // h, N - 1)).astype(int),
                        minlength=N * N)
    print(f"cells hold 0 .. {count.max()} particles", flush=True)
    orc = oracle_mod.Oracle(cfg)
    ost = {k: (v.copy() if isinstance(v, np.ndarray) else v) for k, v in st.items()}
    r = orc.slice_step(ost, want_moments=True)
    assert r["status"] == 0
    seen = []
    for _ in range(2):
        sim = Simulation(cfg)
        sim.set_state(particles=np.stack([st["x"], st["y"], st["px"], st["py"]]), fields=st["fields"],
                      xi=st["xi"], dxi=st["dxi"])
        F, _ = sim.step(fields=True, info=True)
        seen.append((F.cpu().numpy(), sim.moments().cpu().numpy(), sim.get_state()["particles"].cpu().numpy()))
        sim.close()
    for a, b in zip(*seen):
        assert np.array_equal(a, b)
    check_node_arrays(seen[0][1], np.concatenate([r["moments"], r["extra"][:3]]), 1e-10)
    check_fields(seen[0][0], ost["fields"], FIELD_TOL, "crowded")
