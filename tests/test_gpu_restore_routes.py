"""Which way a mesh point of a restoration takes on the pair path, and that both
ways agree with the five passes (SE2N_NO_PAIR): whole rows of every pair in LDS,
or the volume's own tiles where the rows outnumber the compute units and either
leave a unit no second workgroup (DR) or, on runtime radices, have more than 16
pairs (DR in FP32: take 16 elements per thread).  The sizes lie on both sides of
each line.

Few short intervals keep every value bounded.  SR and FP64 have the library's
tolerances (2e-5, 1e-10) and the same growth.  In FP32 a pixel joins or not by a
comparison of values that carry some 1e-6: among images with a spread of tenths
about one pixel in 1e5 per mesh point lies that near, so a thousandth of the map
may differ, each by a fraction of its value."""
import pytest
import torch

from paper_1304_2062_amd import synth

pytestmark = pytest.mark.gpu
F32, F64 = torch.float32, torch.float64


@pytest.mark.parametrize("M,N,dtype,dynamic,whole", [
    (1024, 16, F32, True, True), (1024, 20, F32, True, False), (1024, 32, F32, True, False), (864, 16, F32, True, True), (864, 20, F32, True, False),
    (512, 16, F64, True, True), (512, 20, F64, True, False), (256, 48, F64, True, True), (648, 16, F64, True, False),
    (288, 32, F32, False, True), (288, 34, F32, False, False), (432, 64, F32, False, False), (1024, 32, F32, False, True),
    (288, 40, F64, False, False), (192, 64, F64, False, True), (1024, 32, F64, False, False),
])
def test_restoration_routes(monkeypatch, M, N, dtype, dynamic, whole):
    from paper_1304_2062_amd import se2n
    print(f"restore route {M} {N} {dtype} dynamic={dynamic}", flush=True)
    pair = se2n.Plan(M, N, dtype)
    monkeypatch.setenv("SE2N_NO_PAIR", "1")
    five = se2n.Plan(M, N, dtype)
    monkeypatch.delenv("SE2N_NO_PAIR")
    f = torch.from_numpy(0.1 + 0.9 * synth.make_image(M + N, M, "small")).to(dtype).cuda()
    mask = torch.from_numpy(synth.mask_stripes(M, 3, 14)).cuda()
    args = (0.01, 2.0, 4, 0.5)
    pair.restore_workspace().fill_(255)  # NaN bytes: nothing is read before it is written
    pair.profile(True)
    got, _, join = pair.restore(f, mask, *args, dynamic=dynamic)
    torch.cuda.synchronize()
    names = pair.profile_stats()
    assert "col_solve" in names  # the pair path
    assert ("row_inv_volume" in names) == (not whole)
    want, _, join5 = five.restore(f, mask, *args, dynamic=dynamic)
    rel = float((got.double() - want.double()).norm() / want.double().norm())
    if dynamic and dtype == F32:
        assert float((join != join5).double().mean()) < 1e-3
        assert rel < 1e-3
    else:
        assert (join is None and join5 is None) or torch.equal(join, join5)
        assert rel < (2e-5 if dtype == F32 else 1e-10)
    pair.close()
    five.close()
