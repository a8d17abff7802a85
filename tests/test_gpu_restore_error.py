"""Rounding of the transforms that a restoration repeats, FP32: the pair path is no
farther from the FP64 result than the five passes (SE2N_NO_PAIR) are.  The same
twiddles are applied at every mesh point, so their rounding adds up over the
intervals instead of averaging out.

With eps = 0 the mix multiplies by h / h = 1, and the mesh points are linear: a
restoration of an image proper divides by the orientation maximum, which can
amplify any rounding in single pixels.  5 % of slack for the spread of one image."""
import math

import pytest
import torch

from paper_1304_2062_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,n", [(256, 30, 200), (128, 24, 100), (384, 16, 100), (512, 16, 100), (64, 64, 100), (96, 30, 100),
                                   (1024, 24, 60)])
def test_repeated_transforms_are_as_exact_as_on_the_five_passes(monkeypatch, M, N, n):
    from paper_1304_2062_amd import se2n
    print(f"restore error {M} {N}", flush=True)
    f = torch.from_numpy(0.1 + 0.9 * synth.make_image(M + N, M, "medium")).float().cuda()
    mask = torch.from_numpy(synth.mask_stripes(M, 3, 14)).cuda()
    args = (0.1, 2.0 * (N / (2 * math.pi)) ** 2, n, 0.0)
    out, rmap = {}, None
    for name, dtype in (("pair", torch.float32), ("five", torch.float32), ("exact", torch.float64)):
        if name == "five":
            monkeypatch.setenv("SE2N_NO_PAIR", "1")
        plan = se2n.Plan(M, N, dtype)
        monkeypatch.delenv("SE2N_NO_PAIR", raising=False)
        if rmap is None:
            rmap = plan.orient(f, mask)
        out[name] = plan.restore(f.to(dtype), mask, *args, rmap_in=rmap)[0].double()
        plan.close()
    err = {k: float((out[k] - out["exact"]).norm() / out["exact"].norm()) for k in ("pair", "five")}
    print(f"  pair {err['pair']:.2e} five {err['five']:.2e}", flush=True)
    assert err["pair"] < 1.05 * err["five"], err
