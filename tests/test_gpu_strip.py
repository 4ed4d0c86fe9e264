"""The strip sweep and the patches against one step per launch: bitwise the same populations in every storage format,
over windows with and without x edges and solid nodes, strips of one row to all rows, remainders of
every length and graph replays; the per-step sums agree up to summation order (1e-13 relative)."""
import numpy as np
import pytest

from paper_1812_05401_amd import inputs as I
from tests.helpers import gpu_sim
from tests.test_gpu_parity import CASES, build_case
from tests.test_gpu_two_step import STORAGES, env, same_run

pytestmark = pytest.mark.gpu

CHANNEL = I.CHANNEL
OPEN = (I.VELOCITY, I.OUTFLOW, I.PERIODIC, I.PERIODIC)
SLIT = (I.PERIODIC, I.PERIODIC, I.FREESLIP, I.FREESLIP)


def bodies(nx, ny, moving=False):
    m = dict(ax=2.0, ay=3.0, freq=0.002) if moving else {}
    return [I.body("disk", 0.55 * nx, 0.4 * ny, r=ny / 7, omega=0.001, **m),
            I.body("rect", 0.2 * nx, 0.7 * ny, hx=7.0, hy=ny / 9)]


# nx, ny, edges, moving: windows with no edge (from 376 columns up) and lattices narrower than one
# window, pairs that straddle the wrap (odd nx, periodic), fewer rows than two strips' halo
LATTICES = [(611, 83, CHANNEL, False), (490, 61, I.CHANNEL_CONVECTIVE, False), (377, 40, OPEN, True),
            (503, 47, I.ALL_PERIODIC, True), (640, 30, SLIT, False), (131, 7, I.CHANNEL_CONVECTIVE, False),
            (57, 9, I.ALL_PERIODIC, False), (1024, 64, CHANNEL, True)]


def pair(case, storage, fields, ids=None, **kw):
    """The same simulation with the strip sweep and with one step per launch."""
    out = []
    for strip in (1, 0):
        with env(VPLBM_TWO_STEP=strip, VPLBM_THREE_STEP=strip, VPLBM_STRIP=strip, **{"VPLBM_STRIP_SHAPE": 0, "VPLBM_PATCH": 0, **kw}):
            s = gpu_sim(case, storage=storage, device_mask=ids is None)
            if ids is not None:
                s.set_mask(ids, case.bodies)
        s.init_fields(*fields)
        out.append(s)
    return out


@pytest.mark.parametrize("storage", STORAGES)
@pytest.mark.parametrize("spec", LATTICES, ids=lambda s: f"{s[0]}x{s[1]}_{s[2][1]}_{s[2][2]}{'_moving' if s[3] else ''}")
def test_strip_sweep_bitwise_equals_one_step(gpu, spec, storage):
    nx, ny, bc, moving = spec
    u = (0.04, 0.0)
    case = I.Case("strip", nx, ny, storage=storage, tau=0.6, bc=bc, u_in=u if bc[0] == I.VELOCITY else (0, 0),
                  u0=u, bodies=bodies(nx, ny, moving) if ny > 20 else [])
    fields = I.random_fields(nx, ny, 5, u_mean=u)
    for shape, slots in ((0, 1), (0, 60), (1, 4000)):     # the tallest strips, a few, one row each
        a, b = pair(case, storage, fields, VPLBM_GRAPH_STEPS=24, VPLBM_STRIP_SHAPE=shape, VPLBM_STRIP_SLOTS=slots)
        done = 0
        for n in (24, 13, 5, 1):
            a.step(n)
            b.step(n)
            done += n
        same_run(a, b, 0, done, f"{spec} {storage} shape {shape} slots {slots}")
        a.close()
        b.close()


@pytest.mark.parametrize("storage", STORAGES)
@pytest.mark.parametrize("spec", LATTICES + [(157, 153, I.CHANNEL_CONVECTIVE, True), (301, 251, OPEN, True), (421, 331, CHANNEL, True),
                                              (431, 400, OPEN, False)],
                         ids=lambda s: f"{s[0]}x{s[1]}_{s[2][1]}_{s[2][2]}{'_moving' if s[3] else ''}")
def test_patches_bitwise_equal_one_step(gpu, spec, storage):
    """The lattices above and one of each larger patch size, launches of every number of steps."""
    nx, ny, bc, moving = spec
    u = (0.04, 0.0)
    case = I.Case("patch", nx, ny, storage=storage, tau=0.6, bc=bc, u_in=u if bc[0] == I.VELOCITY else (0, 0),
                  u0=u, bodies=bodies(nx, ny, moving) if ny > 20 else [])
    a, b = pair(case, storage, I.random_fields(nx, ny, 6, u_mean=u), VPLBM_GRAPH_STEPS=16, VPLBM_PATCH=1000000)
    done = 0
    for n in (16, 1, 2, 3, 4, 5, 6, 7):
        a.step(n)
        b.step(n)
        done += n
    same_run(a, b, 0, done, f"{spec} {storage}")
    a.close()
    b.close()


@pytest.mark.parametrize("storage", STORAGES)
@pytest.mark.parametrize("spec", CASES, ids=[c[0] for c in CASES])
def test_strip_sweep_on_the_parity_cases(gpu, spec, storage):
    case, ids = build_case(*spec, seed=13)
    a, b = pair(case, storage, I.random_fields(case.nx, case.ny, 13, u_mean=case.u_in), ids)
    a.step(41)
    b.step(41)
    same_run(a, b, 0, 41, f"{spec[0]} {storage}")
    a.close()
    b.close()


@pytest.mark.parametrize("storage", ["f32", "f64", "f16sr"])
def test_strip_sweep_reports_a_bad_density(gpu, storage):
    """A node whose density is not positive, far from the lattice's edges, in a full row."""
    nx, ny = 400, 64
    case = I.Case("bad", nx, ny, storage=storage, tau=0.8)
    rho, ux, uy = (np.full((ny, nx), v) for v in (1.0, 0.0, 0.0))
    a, _ = pair(case, storage, (rho, ux, uy))
    a.step(12)
    assert a.observables()["status"] == 0
    rho[33, 201] = -20.0
    a.init_fields(rho, ux, uy)
    a.step(12)
    assert a.observables()["status"] == 1
