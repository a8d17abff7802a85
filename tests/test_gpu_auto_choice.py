"""Which schedule AUTO takes for a key it has not seen.

Where the table is cheap (few orientations) it is built at once, and the first
result is that of the propagator schedule bit for bit: the iterated steps,
which round n times in FP32, are left to the keys whose table costs more than
the steps do (few steps of many orientations)."""
import numpy as np
import pytest
import torch

from paper_1304_2062_amd import se2n, synth

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)

TABLE = ([(M, N, n) for M in (64, 256, 1024) for N in (4, 8, 12) for n in (50, 100)]
         + [(M, N, 200) for M in (64, 256, 1024) for N in (6, 10, 14, 16)]
         + [(64, 4, 400), (256, 6, 400), (256, 32, 200), (256, 48, 200), (256, 64, 400)])
STEPS = [(256, 32, 10), (256, 48, 10), (512, 64, 20), (1024, 24, 20)]


def _first(M, N, n, schedule):
    f = torch.from_numpy(synth.make_image(M + N, M, "small").astype(np.float32)).to(DEV)
    mask = torch.from_numpy(synth.mask_random(M + N + 1, M, 0.5)).to(DEV)
    plan = se2n.Plan(M, N, torch.float32)
    plan.set_schedule(schedule)
    out, _ = plan.inpaint(f, mask, 1.0, 1.0, n)
    used = plan.last_schedule()
    plan.close()
    return out, used


@pytest.mark.parametrize("M,N,n", TABLE)
def test_a_cheap_table_is_built_at_once(M, N, n):
    print(f"auto table {M} {N} n={n}", flush=True)
    got, used = _first(M, N, n, "auto")
    want, _ = _first(M, N, n, "propagator")
    assert used == "propagator"
    assert torch.equal(got, want)


@pytest.mark.parametrize("M,N,n", STEPS)
def test_few_steps_of_many_orientations_are_iterated(M, N, n):
    print(f"auto steps {M} {N} n={n}", flush=True)
    assert _first(M, N, n, "auto")[1] == "iterated"
