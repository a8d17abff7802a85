"""FP32 tables of the matrix-core propagator build at the edges of its tiles
(blocks of 2 to 32: the kernels are compiled once per type and tile count),
against the FP64 oracle.

An FFT of length L carries a relative rounding error of about eps log2(L) / 2
per direction and the products less than that: at most 2 eps log2(M^2) in all,
times four for the volume's own rounding and the table's.  An element read too
early from the matrix cores is wrong in its leading digits."""
import math

import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [4, 5, 15, 16, 17, 31, 32, 34, 48, 64])
@pytest.mark.parametrize("scheme,n", [("cn", 1), ("cn", 4), ("cn", 5), ("cn", 399), ("exact", 1)])
def test_fp32_table_matches_the_oracle(N, scheme, n):
    from paper_1304_2062_amd import se2n
    print(f"precompute f32 N={N} {scheme} n={n}", flush=True)
    M, T, beta = 24, 0.9, 1.7
    psi = np.random.default_rng(N).normal(size=(N, M, M)).astype(np.float32)
    plan = se2n.Plan(M, N, torch.float32)
    t = torch.from_numpy(psi).cuda()
    plan.diffuse(t, T, beta, n, scheme)
    got = t.cpu().numpy().astype(np.float64)
    plan.close()
    want = O.diffuse(psi.astype(np.float64), T, beta, n, scheme)
    assert np.linalg.norm(got - want) < 4 * 2 * 6e-8 * 2 * math.log2(M) * np.linalg.norm(want)
