"""Halved columns of each side at its smallest and largest odd and even block,
against the five passes (SE2N_NO_PAIR), with the path that each plan took
asserted (a change to the fit rule cannot leave a plan compared with itself).

Both apply the same propagators with different transforms.  An FFT of length L
carries a relative rounding error of about eps log2(L) / 2 per direction, so two
results differ by at most about 2 eps log2(M^2); four times that for the maximum
and the lift."""
import math

import pytest
import torch

from paper_1304_2062_amd import synth

pytestmark = pytest.mark.gpu
F64 = torch.float64


def _rel(a, b):
    return float((a - b).norm() / b.norm())


@pytest.mark.parametrize("M,N,proj", [(384, 23, "mean"), (384, 39, "max"), (384, 44, "max"), (384, 64, "mean"),
                                      (512, 17, "max"), (512, 31, "mean"), (512, 34, "mean"), (512, 64, "max"),
                                      (768, 5, "max"), (768, 19, "mean"), (768, 10, "mean"), (768, 40, "max"),
                                      (1024, 9, "mean"), (1024, 15, "max"), (1024, 18, "max"), (1024, 32, "mean"),
                                      (2048, 5, "max"), (2048, 7, "mean"), (2048, 4, "mean"), (2048, 16, "max")])
def test_halved_columns_of_every_side(monkeypatch, M, N, proj):
    from paper_1304_2062_amd import se2n
    print(f"halves sides {M} {N} {proj}", flush=True)
    pair = se2n.Plan(M, N, F64)
    monkeypatch.setenv("SE2N_NO_PAIR", "1")
    five = se2n.Plan(M, N, F64)
    monkeypatch.delenv("SE2N_NO_PAIR")
    f = torch.from_numpy(0.1 + 0.9 * synth.make_image(M + N, M, "small")).to(F64).cuda()
    mask = torch.from_numpy(synth.mask_random(M + N + 1, M, 0.5)).cuda()
    args = (1.5, 1.0, 60)
    pair.workspace().fill_(255)  # NaN bytes: nothing is read before it is written
    for p in (pair, five):
        p.profile(True)
    got, rmap = pair.inpaint(f, mask, *args, proj=proj)
    want, rmap5 = five.inpaint(f, mask, *args, proj=proj)
    torch.cuda.synchronize()
    assert "col_solve" in pair.profile_stats() and "solve" not in pair.profile_stats()
    assert "solve" in five.profile_stats() and "col_solve" not in five.profile_stats()
    tol = 4 * 2 * 1.1e-16 * 2 * math.log2(M)
    assert torch.equal(rmap, rmap5)
    assert _rel(got, want) < tol
    psi = pair.lift(f, mask, rmap)
    assert _rel(pair.diffuse(psi.clone(), *args), five.diffuse(psi, *args)) < tol
    pair.close()
    five.close()
