"""The pair path with halved columns (sides whose column blocks are larger
than the LDS of a compute unit) against the five separate passes
(SE2N_NO_PAIR): the smallest and largest blocks of each side, even and odd N,
blocks whose workgroups share a compute unit, schemes and projections, volumes
and restorations; FP64, the only type that takes this way.

Both apply the same propagators with different transforms.  An FFT of length L
carries a relative rounding error of about eps log2(L) / 2 per direction, so
two results differ by at most about 2 eps log2(M^2); the restoration divides
by the orientation maximum at every mesh point, which amplifies the
difference, so it gets the library's own tolerance (1e-10)."""
import math

import numpy as np
import pytest
import torch

from paper_1304_2062_amd import synth

pytestmark = pytest.mark.gpu

F64 = torch.float64


def _tol(M):
    # four times the bound: the maximum and the lift add their own roundings
    return 4 * 2 * 1.1e-16 * 2 * math.log2(M)


def _plans(monkeypatch, M, N, dtype):
    from paper_1304_2062_amd import se2n
    pair = se2n.Plan(M, N, dtype)
    monkeypatch.setenv("SE2N_NO_PAIR", "1")
    five = se2n.Plan(M, N, dtype)
    monkeypatch.delenv("SE2N_NO_PAIR")
    return pair, five


def _rel(a, b):
    return float((a.double() - b.double()).norm() / b.double().norm())


CASES = [
    (384, 23, F64, "cn", "max"),
    (384, 44, F64, "exact", "max"),
    (384, 64, F64, "cn", "mean"),
    (768, 21, F64, "cn", "mean"),
    (768, 22, F64, "cn", "max"),
    (768, 42, F64, "cn", "max"),
    (512, 34, F64, "cn", "max"),
    (512, 64, F64, "exact", "mean"),
    (512, 31, F64, "cn", "max"),
    (1024, 18, F64, "cn", "mean"),
    (1024, 32, F64, "cn", "max"),
    (1024, 15, F64, "cn", "max"),
    (2048, 4, F64, "exact", "max"),
    (2048, 7, F64, "cn", "mean"),
    (2048, 16, F64, "cn", "max"),
]


@pytest.mark.parametrize("M,N,dtype,scheme,proj", CASES)
def test_halved_columns_equal_the_five_passes(monkeypatch, M, N, dtype, scheme, proj):
    print(f"halves {M} {N} {dtype} {scheme} {proj}", flush=True)
    pair, five = _plans(monkeypatch, M, N, dtype)
    f = torch.from_numpy(0.1 + 0.9 * synth.make_image(M + N, M, "small")).to(dtype).cuda()
    mask = torch.from_numpy(synth.mask_random(M + N + 1, M, 0.5)).cuda()
    args = (1.5, 1.0, 60)
    assert np.array_equal(pair.propagator_flags(*args, scheme), five.propagator_flags(*args, scheme))
    pair.workspace().fill_(255)  # NaN bytes: nothing is read before it is written
    got, rmap = pair.inpaint(f, mask, *args, scheme=scheme, proj=proj)
    want, rmap5 = five.inpaint(f, mask, *args, scheme=scheme, proj=proj)
    assert torch.equal(rmap, rmap5)
    assert _rel(got, want) < _tol(M)
    psi = pair.lift(f, mask, rmap)
    a = pair.diffuse(psi.clone(), *args, scheme)
    b = five.diffuse(psi.clone(), *args, scheme)
    assert _rel(a, b) < _tol(M)
    assert _rel(pair.project(a, proj), got) < _tol(M)


@pytest.mark.parametrize("M,N,dtype,dynamic", [(384, 44, F64, True), (768, 24, F64, False), (512, 34, F64, False), (512, 34, F64, True), (1024, 15, F64, True),
                                               (2048, 4, F64, False)])
def test_restoration_with_halved_columns(monkeypatch, M, N, dtype, dynamic):
    print(f"halves restore {M} {N} {dtype} dynamic={dynamic}", flush=True)
    pair, five = _plans(monkeypatch, M, N, dtype)
    f = torch.from_numpy(0.1 + 0.9 * synth.make_image(M + N, M, "small")).to(dtype).cuda()
    mask = torch.from_numpy(synth.mask_stripes(M, 3, 14)).cuda()
    args = (0.01, 2.0, 4, 0.5)
    got, _, join = pair.restore(f, mask, *args, dynamic=dynamic)
    want, _, join5 = five.restore(f, mask, *args, dynamic=dynamic)
    assert float(want.abs().max()) < 2.0
    assert torch.equal(join, join5)
    assert _rel(got, want) < 1e-10
