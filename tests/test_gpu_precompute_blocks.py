"""The propagator build on the matrix cores at the edges of its tiles: blocks of
1 to 32 (even N up to 64, odd N up to 31), against the scalar build and the
oracle, as in test_gpu_precompute.py and with its tolerances."""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu


def _diffuse(monkeypatch, psi, M, N, T, beta, n, scheme, scalar):
    from paper_1304_2062_amd import se2n
    if scalar:
        monkeypatch.setenv("SE2N_SCALAR_PRECOMPUTE", "1")
    plan = se2n.Plan(M, N, torch.float64)
    t = torch.from_numpy(psi).cuda()
    plan.diffuse(t, T, beta, n, scheme)
    out, flags = t.cpu().numpy(), plan.propagator_flags(T, beta, n, scheme)
    plan.close()
    monkeypatch.delenv("SE2N_SCALAR_PRECOMPUTE", raising=False)
    return out, flags


@pytest.mark.parametrize("N", [5, 6, 15, 17, 31, 34, 48, 62, 64])
@pytest.mark.parametrize("scheme,n", [("cn", 1), ("cn", 2), ("cn", 5), ("cn", 64), ("cn", 399), ("exact", 1)])
def test_build_matches_scalar_build_and_oracle(monkeypatch, N, scheme, n):
    print(f"precompute N={N} {scheme} n={n}", flush=True)
    M, T, beta = 24, 0.9, 1.7
    psi = np.random.default_rng(N).normal(size=(N, M, M))
    a, fa = _diffuse(monkeypatch, psi, M, N, T, beta, n, scheme, False)
    b, fb = _diffuse(monkeypatch, psi, M, N, T, beta, n, scheme, True)
    assert np.linalg.norm(a - b) < 1e-12 * np.linalg.norm(b)
    assert np.array_equal(fa, fb)
    want = O.diffuse(psi, T, beta, n, scheme)
    assert np.linalg.norm(a - want) < 1e-10 * np.linalg.norm(want)
