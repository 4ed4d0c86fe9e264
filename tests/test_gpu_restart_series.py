"""The per-step series across vplbm_set_populations: the steps before the restart that the ring holds stay,
the others read 0."""
import numpy as np
import pytest

from paper_1812_05401_amd import inputs as I
from tests.helpers import gpu_sim
from tests.test_gpu_two_step import env

pytestmark = pytest.mark.gpu


def make(nx, ny, storage, ring=0, **kw):
    case = I.Case("series", nx, ny, storage=storage, tau=0.6, bc=I.CHANNEL, u_in=(0.04, 0.0), u0=(0.04, 0.0),
                  bodies=[I.body("disk", 0.3 * nx, 0.45 * ny, r=ny / 8, omega=0.002)])
    with env(**kw):
        return gpu_sim(case, ring=ring)


def close(a, b):
    return np.abs(a - b).max() <= 1e-13 * np.abs(b).max()       # FP64 sums in another order


# launches of eight, six, four and two steps and of one
@pytest.mark.parametrize("nx,ny,storage,kw", [(96, 80, "f64", {}), (250, 200, "f32", {}), (1024, 800, "f32", {}),
                                              (1000, 900, "f16sr", {}), (96, 80, "f64", {"VPLBM_TWO_STEP": 0})])
def test_a_restart_keeps_the_steps_before(gpu, nx, ny, storage, kw):
    a, b = make(nx, ny, storage, **kw), make(nx, ny, storage, **kw)
    for n in (21, 30):
        a.step(n)
        b.step(n)
        done = a.steps_done
        a.set_populations(b.populations(), done)     # (nothing has read the series of the last steps)
        assert close(a.force_series(0, done), b.force_series(0, done))
        assert a.observables()["mass"] == pytest.approx(b.observables()["mass"], rel=1e-13)
    a.step(11)
    b.step(11)
    assert close(a.force_series(0, 62), b.force_series(0, 62))
    a.close()
    b.close()


def test_steps_that_the_ring_does_not_hold_read_zero(gpu):
    a, b = make(96, 80, "f64", ring=16), make(96, 80, "f64", ring=64)
    a.step(40)
    b.step(40)
    want = b.force_series(0, 40)
    pop = a.populations()
    a.set_populations(pop, 30)                       # back: steps 24 to 29 are there, 14 to 23 were overwritten
    got = a.force_series(14, 16)
    assert close(got[10:], want[24:30]) and not got[:10].any()
    a.set_populations(pop, 41)                       # on: steps 30 to 40 were not done after the restart
    got = a.force_series(25, 16)
    assert close(got[:5], want[25:30]) and not got[5:].any()
    assert a.observables()["mass"] == 0.0
    a.set_populations(pop, 1000)
    assert not a.force_series(984, 16).any()
    b.set_populations(pop, 10)
    assert close(b.force_series(0, 10), want[:10])
    b.set_populations(pop, 0)
    b.step(3)
    assert b.force_series(0, 3)[:, 0].all()
    a.close()
    b.close()
