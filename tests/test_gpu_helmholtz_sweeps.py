"""The sweeps of one Helmholtz V-cycle in the tolerance mode against the same cycle
in NumPy: nu_pre and nu_post act on every level, on those of at most 64^2 below a
finer one as two V(max(1, nu1 - 1), nu_post - 1) cycles (one V(nu1, 1) for
nu_post = 1), nu1 = nu_pre on the two finest levels and 1 below.

Those levels sweep in FP32 where they only correct a finer one: their correction
carries some tens of roundings of 6e-8, so the iterates agree to 1e-5; one sweep
more or fewer moves them by 1e-3 and more.
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


OMEGA, N0, L = 1.175, 1.0, 6.0


def _laplace(u, h):
    r = np.zeros_like(u)
    r[1:-1, 1:-1] = (u[:-2, 1:-1] + u[2:, 1:-1] + u[1:-1, :-2] + u[1:-1, 2:] - 4.0 * u[1:-1, 1:-1]) / h ** 2
    return r


def _smooth(u, f, k2, h, nu):
    n = u.shape[0] - 1
    Y, X = np.indices(u.shape)
    inner = (X > 0) & (Y > 0) & (X < n) & (Y < n)
    om = OMEGA if h * h <= 0.125 / N0 else 1.0
    for _ in range(nu):
        for colour in (0, 1):
            nb = np.zeros_like(u)
            nb[1:-1, 1:-1] = u[:-2, 1:-1] + u[2:, 1:-1] + u[1:-1, :-2] + u[1:-1, 2:]
            g = (nb - h * h * f) / (4.0 + h * h * k2)
            m = inner & ((X + Y) % 2 == colour)
            u[m] += om * (g[m] - u[m])


def _restrict(r):
    n = r.shape[0] - 1
    c = np.zeros((n // 2 + 1, n // 2 + 1))

    def at(dy, dx):
        return r[2 + dy:n - 1 + dy:2, 2 + dx:n - 1 + dx:2]

    c[1:-1, 1:-1] = (4 * at(0, 0) + 2 * (at(0, 1) + at(0, -1) + at(1, 0) + at(-1, 0))
                     + at(1, 1) + at(1, -1) + at(-1, 1) + at(-1, -1)) / 16
    return c


def _prolong(e):
    n = 2 * (e.shape[0] - 1)
    u = np.zeros((n + 1, n + 1))
    u[::2, ::2] = e
    u[1::2, ::2] = 0.5 * (e[1:] + e[:-1])
    u[:, 1::2] = 0.5 * (u[:, 2::2] + u[:, :-2:2])
    return u


def _cycle(u, f, k2s, l, h, pre, post):
    n = u.shape[0] - 1
    if n == 2:
        u[1, 1] = -f[1, 1] / (4.0 / h ** 2 + k2s[l][1, 1])
        return
    nu1, nu2, times = pre[l], post[l], 1
    if n == 64 and post[l - 1] >= 2:
        times = 2
    for _ in range(times):
        _smooth(u, f, k2s[l], h, nu1)
        r = f - _laplace(u, h) + k2s[l] * u
        r[[0, -1]] = 0.0
        r[:, [0, -1]] = 0.0
        e = np.zeros((n // 2 + 1, n // 2 + 1))
        _cycle(e, _restrict(r), k2s, l + 1, 2 * h, pre, post)
        u += _prolong(e)
        _smooth(u, f, k2s[l], h, nu2)


@pytest.mark.parametrize("N", [128, 256])
@pytest.mark.parametrize("nu_pre,nu_post", [(1, 1), (2, 2), (3, 3), (1, 3), (3, 1), (3, 2)])
def test_one_cycle_takes_the_sweeps_asked_for(torch_cuda, N, nu_pre, nu_post):
    from paper_2012_00881_amd import Simulation
    print(f"[case] Helmholtz sweeps N={N} nu=({nu_pre}, {nu_post})", flush=True)
    rng = np.random.default_rng(N)
    g = np.linspace(-L, L, N + 1)
    X, Y = g[None, :], g[:, None]
    f = np.exp(-((X - 1.0) ** 2 + Y ** 2)) * np.cos(3.0 * X) + 0.1 * rng.standard_normal((N + 1, N + 1))
    k2 = 0.2 + 0.5 * (1.0 + np.sin(X + 2.0 * Y))
    for a in (f, k2):
        a[[0, -1]] = 0.0
        a[:, [0, -1]] = 0.0
    sim = Simulation(wi.scaled(wi.config("C1"), n_cells=N, half_width=L, n0=N0, nu_pre=nu_pre, nu_post=nu_post,
                               mg_rtol=1e-14, mg_max_cycles=1))
    st, u, cyc, _ = sim.mg_solve(f, k2=k2)
    sim.close()
    assert cyc == 1
    k2s, l0 = [k2], {128: 1, 256: 2}[N]
    while k2s[-1].shape[0] > 3:
        k2s.append(_restrict(k2s[-1]))
    pre, post = [], []
    for l in range(len(k2s)):
        nu1, nu2 = (nu_pre if l < 2 else 1), nu_post
        if l >= l0 and nu_post >= 2:
            # (every level of the coarse kernel sweeps as its first one)
            nu1, nu2 = max(1, (nu_pre if l0 < 2 else 1) - 1), nu_post - 1
        elif l >= l0:
            nu1 = nu_pre if l0 < 2 else 1
        pre.append(nu1)
        post.append(nu2)
    ref = np.zeros_like(f)
    _cycle(ref, f, k2s, 0, 2 * L / N, pre, post)
    d = np.linalg.norm(u[0].cpu().numpy() - ref) / np.linalg.norm(ref)
    print(f"difference {d:.2e}", flush=True)
    assert d <= 1e-5
