"""Results read on the caller's kinds of stream: the staged copy waits for the work before it."""
import numpy as np
import pytest

from paper_1812_05401_amd import binding as B
from paper_1812_05401_amd import inputs as I

pytestmark = pytest.mark.gpu

PER_THREAD = 2   # hipStreamPerThread: another stream in every thread that names it


@pytest.mark.parametrize("stream", [None, "torch", PER_THREAD], ids=["own", "torch", "per_thread"])
def test_results_wait_for_the_steps(gpu, stream):
    case = I.Case("copy", 1500, 900, storage="f64", tau=0.6, bc=I.CHANNEL, u_in=(0.04, 0.0), u0=(0.04, 0.0),
                  bodies=[I.body("disk", 400, 450, r=60)])
    want = B.Simulation(case, stream=None)
    sim = B.Simulation(case, stream=stream)
    for n in (400, 3, 400):
        want.step(n)
        fields, pop = want.fields(), want.populations()
        sim.step(n)
        assert bool((sim.populations() == pop).all())      # nothing waited for the steps before
        assert all(bool((a == b).all()) for a, b in zip(sim.fields(), fields))
        want_series, series = want.force_series(0, want.steps_done), sim.force_series(0, sim.steps_done)
        assert np.abs(series - want_series).max() <= 1e-12 * np.abs(want_series).max()
    want.close()
    sim.close()
