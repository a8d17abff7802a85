"""The row-blocked layout of the inverse passes against the in-place one where the
five passes run: plans too large for the pair path, and smaller ones kept off it
(SE2N_NO_PAIR).  Only the addresses differ, so every result is bit-identical; the
path that each plan took is asserted."""
import numpy as np
import pytest
import torch

from paper_1304_2062_amd import se2n, synth

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)


def _plans(monkeypatch, M, N, no_pair):
    if no_pair:
        monkeypatch.setenv("SE2N_NO_PAIR", "1")
    blocked = se2n.Plan(M, N, torch.float32)
    monkeypatch.setenv("SE2N_NO_ROW_BLOCKS", "1")
    flat = se2n.Plan(M, N, torch.float32)
    monkeypatch.delenv("SE2N_NO_ROW_BLOCKS")
    monkeypatch.delenv("SE2N_NO_PAIR", raising=False)
    assert blocked.workspace_bytes - flat.workspace_bytes >= N * (M // 2 + 1) * M * 8
    for p in (blocked, flat):
        p.profile(True)
    return blocked, flat


def _five(*plans):
    torch.cuda.synchronize()
    for p in plans:
        names = p.profile_stats()
        assert "col_solve" not in names and "col_fft_inv" in names
        p.close()


def _image(M, seed):
    f = torch.from_numpy(synth.make_image(seed, M, "medium")).to(DEV, torch.float32)
    return f, torch.from_numpy(synth.mask_random(seed + 1, M, 0.6)).to(DEV)


@pytest.mark.parametrize("M,N,proj,no_pair", [(1024, 34, "max", False), (1024, 21, "mean", False), (512, 33, "max", False),
                                              (1024, 16, "mean", True), (512, 31, "max", True)])
def test_inpaint(monkeypatch, M, N, proj, no_pair):
    print(f"layout five: inpaint {M}^2 N={N} {proj}", flush=True)
    blocked, flat = _plans(monkeypatch, M, N, no_pair)
    f, mask = _image(M, 3)
    a, ra = blocked.inpaint(f, mask, 4.0, 1.0, 400, proj=proj)
    b, rb = flat.inpaint(f, mask, 4.0, 1.0, 400, proj=proj)
    assert torch.equal(ra, rb) and torch.isfinite(a).all()
    assert torch.equal(a, b), float((a - b).abs().max())
    _five(blocked, flat)


@pytest.mark.parametrize("M,N,no_pair", [(1024, 34, False), (512, 33, False), (1024, 16, True)])
def test_diffuse(monkeypatch, M, N, no_pair):
    print(f"layout five: diffuse {M}^2 N={N}", flush=True)
    blocked, flat = _plans(monkeypatch, M, N, no_pair)
    psi = torch.from_numpy(np.random.default_rng(2).standard_normal((N, M, M)).astype(np.float32)).to(DEV)
    assert torch.equal(blocked.diffuse(psi.clone(), 0.7, 1.5, 30), flat.diffuse(psi.clone(), 0.7, 1.5, 30))
    _five(blocked, flat)


@pytest.mark.parametrize("M,N,no_pair", [(512, 33, False), (512, 30, True)])
@pytest.mark.parametrize("dynamic", [False, True])
def test_restoration(monkeypatch, M, N, no_pair, dynamic):
    print(f"layout five: restoration {M}^2 N={N} dynamic={dynamic}", flush=True)
    blocked, flat = _plans(monkeypatch, M, N, no_pair)
    f, _ = _image(M, 7)
    mask = torch.from_numpy(synth.mask_stripes(M, 6, 24)).to(DEV)
    kw = dict(T=2.0, beta=1.0, n_intervals=6, substeps=10, eps=0.5, dynamic=dynamic)
    a, ra, ja = blocked.restore(f, mask, **kw)
    b, rb, jb = flat.restore(f, mask, **kw)
    assert torch.equal(ra, rb)
    assert (ja is None and jb is None) or torch.equal(ja, jb)
    assert torch.equal(a, b)
    _five(blocked, flat)
