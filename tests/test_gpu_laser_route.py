"""Which way a laser plane is solved, read from the kernels that ran: sine-transform
iterations where the grid has them (128^2 .. 2048^2), the susceptibility varies by
at most 0.4 (at 2048^2 0.1) of the shift's modulus on either side of the middle of its range, and
mg_max_cycles leaves room for them; V-cycles everywhere else.
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


# half range h of chi about its middle 1 + h against |1 + h + beta - i gam|, beta = 10, gam = 5
@pytest.mark.parametrize("N", [64, 128, 256, 512, 1024, 2048])
@pytest.mark.parametrize("half,cycles,direct", [  # direct: up to this N
    (0.0, 50, 2048),
    (1.0, 50, 2048),   # 1 / |12 - 5i| = 0.077
    (1.5, 50, 1024),   # 1.5 / |12.5 - 5i| = 0.111
    (7.5, 50, 1024),   # 7.5 / |18.5 - 5i| = 0.391
    (8.0, 50, 0),      # 8 / |19 - 5i| = 0.407
    (50.0, 50, 0),
    (1.0, 11, 0),      # 15 iterations (0.077^15 = 2e-17) and two more would not fit
    (1.0, 17, 2048),
])
def test_route_of_a_plane(torch_cuda, N, half, cycles, direct):
    from paper_2012_00881_amd import Simulation
    print(f"[case] laser route N={N} half range {half} cycles {cycles}", flush=True)
    L, nz, dxi, dt = 6.0, 2, 0.05, 8.0
    cfg = wi.scaled(wi.config("C1"), n_cells=N, half_width=L, beams=[], adaptive=0, laser_nz=nz,
                    laser_k0=10.0, dxi0=dxi, mg_max_cycles=cycles)
    rng = np.random.default_rng(N)
    chi = 1.0 + half * (1.0 + np.where(rng.uniform(size=(nz, N + 1, N + 1)) < 0.5, -1.0, 1.0))
    sim = Simulation(cfg)
    sim.laser_set(wi.laser_gaussian(N, L, nz, dxi, 0.1, 1.5, 1.5, 0.3))
    sim.profile(True)
    cyc = sim.laser_advance(dt, chi)
    names = {k["name"] for k in sim.kernel_stats() if k["launches"] > 0}
    sim.close()
    assert min(cyc) >= 1
    fst = any(n.startswith("k_las_fst") for n in names)
    vcycle = any(n.startswith("k_las_coarse") for n in names)
    expect = 128 <= N <= direct
    assert fst == expect and vcycle == (not expect), names
