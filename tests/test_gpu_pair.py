"""The pair path (three passes: lift and row FFT, column FFT with the per-mode
products and the inverse column FFT, inverse row FFT and projection) against
the five separate passes (SE2N_NO_PAIR), at the edges of its tiles: compiled
and other sides, even and odd N, blocks of one to 32 slices, both data types,
schemes and projections, and the restoration heuristics.

Both paths apply the same propagators with different transforms.  An FFT of
length L carries a relative rounding error of about eps log2(L) / 2 per
direction, so two FP32 results differ by at most about
2 * 2 * 6e-8 * log2(1024^2) / 2 = 2.4e-6 (FP64: 4.4e-15); the restoration
divides by the orientation maximum at every mesh point, which amplifies the
difference, so it gets the library's own tolerances (2e-5, 1e-10)."""
import numpy as np
import pytest
import torch

from paper_1304_2062_amd import synth

pytestmark = pytest.mark.gpu

TOL = {torch.float32: 2.4e-6, torch.float64: 1e-13}


def _plans(monkeypatch, M, N, dtype):
    from paper_1304_2062_amd import se2n
    pair = se2n.Plan(M, N, dtype)
    monkeypatch.setenv("SE2N_NO_PAIR", "1")
    five = se2n.Plan(M, N, dtype)
    monkeypatch.delenv("SE2N_NO_PAIR")
    return pair, five


def _image(M, seed, dtype):
    f = torch.from_numpy(0.1 + 0.9 * synth.make_image(seed, M, "small")).to(dtype).cuda()
    return f, torch.from_numpy(synth.mask_random(seed + 1, M, 0.5)).cuda()


def _rel(a, b):
    return float((a.double() - b.double()).norm() / b.double().norm())


CASES = [
    # M, N, dtype, scheme, proj
    (16, 4, torch.float32, "cn", "max"),
    (36, 5, torch.float32, "exact", "mean"),
    (48, 63, torch.float32, "cn", "max"),
    (64, 64, torch.float32, "cn", "mean"),
    (72, 10, torch.float64, "cn", "max"),
    (96, 9, torch.float64, "exact", "max"),
    (108, 31, torch.float64, "cn", "mean"),
    (128, 6, torch.float32, "exact", "max"),
    (192, 30, torch.float64, "cn", "max"),
    (256, 30, torch.float32, "cn", "max"),
    (256, 31, torch.float64, "cn", "max"),
    (324, 15, torch.float32, "exact", "mean"),
    (384, 48, torch.float32, "cn", "max"),
    (512, 32, torch.float32, "cn", "max"),
    (512, 32, torch.float64, "cn", "mean"),
    (768, 24, torch.float32, "cn", "max"),
    (972, 15, torch.float32, "cn", "max"),
    (1024, 32, torch.float32, "cn", "max"),
    (1024, 7, torch.float32, "cn", "mean"),
    (1024, 16, torch.float64, "exact", "max"),
]


@pytest.mark.parametrize("M,N,dtype,scheme,proj", CASES)
def test_pair_path_equals_the_five_passes(monkeypatch, M, N, dtype, scheme, proj):
    print(f"pair {M} {N} {dtype} {scheme} {proj}", flush=True)
    pair, five = _plans(monkeypatch, M, N, dtype)
    f, mask = _image(M, M + N, dtype)
    args = (1.5, 1.0, 60)
    assert np.array_equal(pair.propagator_flags(*args, scheme), five.propagator_flags(*args, scheme))
    pair.workspace().fill_(255)  # NaN bytes: nothing is read before it is written
    got, rmap = pair.inpaint(f, mask, *args, scheme=scheme, proj=proj)
    want, rmap5 = five.inpaint(f, mask, *args, scheme=scheme, proj=proj)
    assert torch.equal(rmap, rmap5)
    assert _rel(got, want) < TOL[dtype]
    # the volume path; the first call's map is one of its inputs
    psi = pair.lift(f, mask, rmap)
    a = pair.diffuse(psi.clone(), *args, scheme)
    b = five.diffuse(psi.clone(), *args, scheme)
    assert _rel(a, b) < TOL[dtype]
    assert _rel(pair.project(a, proj), got) < TOL[dtype]


@pytest.mark.parametrize("dynamic", [False, True])
@pytest.mark.parametrize("M,N,dtype", [(36, 5, torch.float64), (64, 16, torch.float64), (96, 31, torch.float64),
                                       (256, 30, torch.float64), (512, 32, torch.float64), (256, 30, torch.float32),
                                       (768, 40, torch.float32)])
def test_restoration_on_the_pair_path(monkeypatch, M, N, dtype, dynamic):
    """SR in both types; DR in FP64 (FP32 growth decisions may differ at
    near-ties).  Few short intervals keep every value bounded by the image's
    (checked): where the restoration diverges it amplifies any rounding."""
    if dynamic and dtype == torch.float32:
        pytest.skip("growth decisions near ties")
    print(f"pair restore {M} {N} {dtype} dynamic={dynamic}", flush=True)
    pair, five = _plans(monkeypatch, M, N, dtype)
    f, _ = _image(M, M + N, dtype)
    mask = torch.from_numpy(synth.mask_stripes(M, 3, 14)).cuda()
    args = (0.01, 2.0, 4, 0.5)
    got, _, join = pair.restore(f, mask, *args, dynamic=dynamic)
    want, _, join5 = five.restore(f, mask, *args, dynamic=dynamic)
    assert float(want.abs().max()) < 2.0
    assert torch.equal(join, join5)
    assert _rel(got, want) < (2e-5 if dtype == torch.float32 else 1e-10)


@pytest.mark.parametrize("shapes", [[(128, 4), (128, 64)], [(1024, 34), (1024, 32), (64, 16)], [(768, 40), (192, 6)],
                                    [(512, 32)] * 5 + [(256, 30), (384, 48)]])
def test_batch_on_the_pair_path(shapes):
    """Batched items against the single-image path: the smallest and largest
    blocks of a side, groups of several images and of one, both projections,
    beside items that keep the five passes (1024, N = 34 and sides without a
    compiled body), replayed with other work between."""
    from paper_1304_2062_amd import se2n
    items, want = [], []
    for i, (M, N) in enumerate(shapes):
        f, mask = _image(M, 100 + i, torch.float32)
        proj = "mean" if i % 3 == 1 else "max"
        items.append(se2n.BatchItem(f, mask, N, 1.0, 1.0, 50, proj=proj))
        plan = se2n.Plan(M, N, torch.float32)
        want.append(plan.inpaint(f, mask, 1.0, 1.0, 50, proj=proj))
        torch.cuda.synchronize()
        plan.close()
    ws = se2n.batch_workspace(items)
    ws.fill_(255)
    for replay in range(3):
        print(f"pair batch {shapes} replay {replay}", flush=True)
        for it in items:
            it.out.fill_(float("nan"))
        out = se2n.inpaint_batched(items, ws)
        for got, it, (ref, rmap) in zip(out, items, want):
            assert torch.equal(it.rmap_out, rmap)
            assert _rel(got, ref) < TOL[torch.float32]
        (torch.randn(1 << 20, device="cuda") * 2).sum().item()
    se2n.batch_clear()
