"""Probe means over discs inside, across and outside the box, as small as one node
and larger than the box, against the mean over the same nodes of the slice's
field (node test in the same arithmetic).  Both add at most (N + 1)^2 values, in
different orders: they agree to (N + 1)^2 eps of the largest |value|.
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


@pytest.mark.parametrize("N", [8, 64, 128])
def test_probe_means(torch_cuda, N):
    from paper_2012_00881_amd import Simulation
    print(f"[case] probes N={N}", flush=True)
    L = 6.0
    h = 2 * L / N
    discs = [(0.0, 0.0, 2.5 * h), (L / 3, -L / 4, 1.7), (-L, L, 1.1), (0.3, 0.2, 100.0), (L + 1.0, 0.0, 1.5),
             (3 * L, 0.0, 1.0), (2 * h, h, 0.0), (0.0, -3.0, L)]
    probes = [dict(field=k % 5, slice_begin=1, slice_end=2, r_max=r, x0=x, y0=y)
              for k, (x, y, r) in enumerate(discs)]
    cfg = wi.scaled(wi.config("C1"), n_cells=N, half_width=L, probes=probes)
    st = wi.synthetic_state(cfg, seed=3 + N, p_max=0.3, xi=1.0)
    sim = Simulation(cfg, n_slices=2)
    sim.set_state(particles=np.stack([st["x"], st["y"], st["px"], st["py"]]), fields=st["fields"],
                  xi=st["xi"], dxi=st["dxi"])
    _, got = sim.run(2, probes=True)
    F = sim.get_state()["fields"].cpu().numpy()
    sim.close()
    g = -L + h * np.arange(N + 1)
    for k, (x, y, r) in enumerate(discs):
        rx, ry = (g - x)[None, :], (g - y)[:, None]
        v = F[k % 5][rx * rx + ry * ry <= r * r]
        want = v.mean() if v.size else 0.0
        err = abs(float(got[k]) - want)
        print(f"disc {k}: {v.size} nodes, difference {err:.1e}", flush=True)
        assert err <= (N + 1) ** 2 * np.finfo(float).eps * (np.abs(v).max() if v.size else 0.0)
