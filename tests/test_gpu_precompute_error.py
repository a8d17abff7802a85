"""Error of the matrix-core propagator build against long double.

The powering multiplies the rounding of the one-step propagator by the number
of steps unless the build prevents it: a diffusion of a few hundred steps in
FP64 then carries some 1e-13.  Here the result has to be as good as its
transforms: an FFT of length L carries a relative rounding error of about
eps log2(L) / 2 per direction, at most 2 eps log2(M^2) in all, times four for
the products and the table itself.  Blocks of 2 to 32; weak and strong coupling
(a step of T beta / n below and above the 1/8 where the build changes its form)."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
L = np.longdouble
PI = L("3.14159265358979323846264338327950288")


def _reference(psi, T, beta, n):
    """n Crank-Nicolson steps of every mode in long double: Thomas and Sherman-Morrison on the N-cycle."""
    N, M, _ = psi.shape
    spec = np.fft.rfft2(psi.astype(L))
    h, beta = L(T) / n / 2, L(beta)
    s = np.sin(2 * PI * np.arange(M).astype(L) / M)
    e = 2 * PI * np.arange(N).astype(L) / N
    a = np.cos(e)[:, None, None] * s[None, None, :M // 2 + 1] + np.sin(e)[:, None, None] * s[None, :, None]
    V = 2 * beta + M * a * a
    d, off = 1 + h * V, -h * beta
    g = -d[0].copy()
    d[0] = d[0] - g
    d[N - 1] = d[N - 1] - off * off / g
    inv, cp = [1 / d[0]], []
    for r in range(1, N):
        cp.append(off * inv[r - 1])
        inv.append(1 / (d[r] - off * cp[r - 1]))

    def solve(y):
        for r in range(N):
            y[r] = (y[r] if r == 0 else y[r] - off * y[r - 1]) * inv[r]
        for r in range(N - 2, -1, -1):
            y[r] = y[r] - cp[r] * y[r + 1]
        return y

    z = [np.zeros_like(g) for _ in range(N)]
    z[0], z[N - 1] = g.copy(), np.full_like(g, off)
    z = solve(z)
    w = off / g
    den = 1 / (1 + z[0] + w * z[N - 1])
    x = list(spec)
    for _ in range(n):
        y = solve([x[r] + h * (beta * (x[(r + 1) % N] + x[r - 1]) - V[r] * x[r]) for r in range(N)])
        c = (y[0] + w * y[N - 1]) * den
        x = [y[r] - c * z[r] for r in range(N)]
    return np.fft.irfft2(np.stack(x), s=(M, M))


@pytest.mark.parametrize("N", [4, 5, 6, 8, 15, 16, 18, 31, 32, 34, 64])
@pytest.mark.parametrize("T,beta,n", [(0.9, 1.7, 399), (2.0, 1.0, 200), (3.0, 0.3, 64), (2.0, 4.0, 20)])
def test_fp64_diffusion_is_as_exact_as_its_transforms(N, T, beta, n):
    from paper_1304_2062_amd import se2n
    print(f"precompute error N={N} T={T} beta={beta} n={n}", flush=True)
    M = 24
    psi = np.random.default_rng(N * 7 + n).normal(size=(N, M, M))
    plan = se2n.Plan(M, N, torch.float64)
    t = torch.from_numpy(psi).cuda()
    plan.diffuse(t, T, beta, n)
    got = t.cpu().numpy().astype(L)
    plan.close()
    want = _reference(psi, T, beta, n)
    rel = float(np.linalg.norm(got - want) / np.linalg.norm(want))
    assert rel < 4 * 2 * 1.1e-16 * 2 * math.log2(M), rel
