"""Which build the smallest blocks take: the scalar one where many classes make
the padded matrix-core products the bound (N <= 6 from a side of 384 on, even N
up to 10 from 768 on).  There the tables are those of SE2N_SCALAR_PRECOMPUTE bit
for bit; on either side of the line they agree with the oracle to the tolerance
of the other build tests."""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu


def _diffuse(psi, M, N, n):
    from paper_1304_2062_amd import se2n
    plan = se2n.Plan(M, N, torch.float64)
    t = torch.from_numpy(psi).cuda()
    plan.diffuse(t, 0.8, 1.3, n)
    out = t.cpu().numpy()
    plan.close()
    return out


@pytest.mark.parametrize("M,N,scalar", [(384, 4, True), (384, 5, True), (384, 6, True), (768, 8, True), (768, 10, True),
                                        (324, 6, False), (648, 8, False), (384, 7, False)])
def test_build_of_the_smallest_blocks(monkeypatch, M, N, scalar):
    print(f"precompute small M={M} N={N}", flush=True)
    psi = np.random.default_rng(M + N).normal(size=(N, M, M))
    got = _diffuse(psi, M, N, 50)
    if scalar:
        monkeypatch.setenv("SE2N_SCALAR_PRECOMPUTE", "1")
        assert np.array_equal(got, _diffuse(psi, M, N, 50))
    want = O.diffuse(psi, 0.8, 1.3, 50, "cn")
    assert np.linalg.norm(got - want) < 1e-10 * np.linalg.norm(want)
