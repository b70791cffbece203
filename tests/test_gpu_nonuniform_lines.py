"""The line solves of the non-uniform multigrid at the sizes where their tiling
can go wrong: lines of 2 to 32 unknowns a lane (grids of 128^2 .. 2048^2), the
levels below 64^2 alone, strongly graded spacings (neighbouring cells of aspect
ratio up to 50) and a nonzero guess.

Each solution is checked by its own residual in the discrete equation written
out in the header (formed here in NumPy): the solve ends at the rounding floor,
||R J - L u|| <= 0.35 eps (2 max|d| ||u|| + ||R J||), or by stagnation within
10% of it; the check allows 4 of that bound for the residual's other summation
order.
"""
import numpy as np
import pytest

import wandqs_inputs as wi

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _weights(X):
    hm, hp = X[1:-1] - X[:-2], X[2:] - X[1:-1]
    ha, hb = hm + hp, hp - hm
    dxx = (2 / (hm * ha), -2 / (hm * hp), 2 / (hp * ha))
    dx = (-hp / (ha * hm), hp / (ha * hm) - hm / (ha * hp), hm / (ha * hp))
    return dxx, dx, hb / 3


def _residual(X, Y, u, M, J):
    ax, gx, bx = _weights(X)
    ay, gy, by = _weights(Y)

    def along_x(c, v):  # v given with its boundary columns
        return c[0] * v[:, :-2] + c[1] * v[:, 1:-1] + c[2] * v[:, 2:]

    def along_y(c, v):
        c = [w[:, None] for w in c]
        return c[0] * v[:-2] + c[1] * v[1:-1] + c[2] * v[2:]

    def pad(v):
        return np.pad(v, 1)

    dxx, dyy = along_x(ax, u)[1:-1], along_y(ay, u)[:, 1:-1]
    mu = M * u

    def third(v):
        return bx[None, :] * along_x(gx, v)[1:-1] + by[:, None] * along_y(gy, v)[:, 1:-1]

    Lu = (dxx + dyy + bx[None, :] * along_x(gx, pad(dyy))[1:-1] + by[:, None] * along_y(gy, pad(dxx))[:, 1:-1]
          + third(mu) + mu[1:-1, 1:-1])
    RJ = J[1:-1, 1:-1] + third(J)
    m = M[1:-1, 1:-1]
    g1x, g1y = (bx * gx[1])[None, :], (by * gy[1])[:, None]
    d = ax[1][None, :] + ay[1][:, None] + g1x * ay[1][:, None] + g1y * ax[1][None, :] + (g1x + g1y) * m + m
    return RJ - Lu, RJ, np.abs(d).max()


@pytest.mark.parametrize("N,grading", [(8, 1.3), (16, 1.5), (32, 1.2), (64, 1.12), (128, 1.05),
                                       (256, 1.02), (512, 1.01), (1024, 1.004), (2048, 1.0)])
@pytest.mark.parametrize("helm", [False, True])
def test_line_solves_reach_the_floor(torch_cuda, N, grading, helm):
    from paper_2012_00881_amd import Simulation
    print(f"[case] line solves N={N} helm={helm}", flush=True)
    # spacings growing by `grading` a cell from the axis out, one side faster than the other
    w = grading ** np.abs(np.arange(N) - N // 3)
    X = np.concatenate([[0.0], np.cumsum(w)])
    X = 8.0 * X / X[-1] - 4.0
    Y = -X[::-1].copy()
    rng = np.random.default_rng(N)
    J = rng.standard_normal((N + 1, N + 1))
    M = -rng.uniform(0.0, 3.0, (N + 1, N + 1)) if helm else np.zeros((N + 1, N + 1))
    M[0], M[-1], M[:, 0], M[:, -1] = 0.0, 0.0, 0.0, 0.0
    u0 = 0.01 * rng.standard_normal((N + 1, N + 1))
    sim = Simulation(wi.scaled(wi.config("C1"), n_cells=N, mg_max_cycles=200))
    st, u, cyc, rel = sim.nu_mg_solve(X, Y, J, u0=u0, M=M if helm else None)
    sim.close()
    assert st == 0, (st, cyc, rel)
    u = u.cpu().numpy()
    r, RJ, amax = _residual(X, Y, u, M, J)
    floor = 0.35 * EPS * (2 * amax * np.linalg.norm(u) + np.linalg.norm(RJ))
    print(f"cycles {cyc}, residual / floor {np.linalg.norm(r) / floor:.2f}", flush=True)
    assert np.linalg.norm(r) <= max(4 * floor, 1e-14 * np.linalg.norm(RJ))
    for edge in (u[0], u[-1], u[:, 0], u[:, -1]):
        assert np.all(edge == 0.0)
