"""The serving pool's early stop where the kernel that advances a simulation is patches, tiles or strips,
or changes between two checks: each check compares with the one before it, as a single simulation's
residual does."""
import pytest

from paper_1812_05401_amd import inputs as I
from tests.test_gpu_residual import _drain

pytestmark = pytest.mark.gpu

SPL, EVERY = 32, 64


def channel(name, nx, ny, storage):
    return I.Case(name, nx, ny, storage=storage, tau=0.6, bc=I.CHANNEL, u_in=(0.04, 0.0), u0=(0.04, 0.0),
                  bodies=[I.body("disk", 0.3 * nx, 0.5 * ny, r=ny / 10)])


def single(case, n):
    """The residual at n - EVERY and at n, and the fields after n steps and one more."""
    from paper_1812_05401_amd import binding as B
    s = B.Simulation(case, stream=None)
    s.step(n - 2 * EVERY)
    s.residual()
    r = []
    for _ in range(2):
        s.step(EVERY)
        r.append(s.residual())
    s.step(1)
    fields = s.fields()
    s.close()
    return r[0], r[1], fields


# Nodes resident with the partner and without it: f16sr takes patches up to 0.42 million, tiles up to
# 3.8 million and strips above; f32 patches up to 1.2 million and strips above.  The partner ends at 96
# steps, between the first check and the second.
@pytest.mark.parametrize("storage,nx,ny,partner", [("f16sr", 700, 700, None), ("f16sr", 600, 600, (500, 500)),
                                                   ("f16sr", 600, 600, (2000, 1900)), ("f16sr", 900, 700, (2000, 1900)),
                                                   ("f16sr", 2000, 1950, None), ("f32", 700, 700, (2000, 1900))])
def test_checks_compare_with_the_check_before(gpu, storage, nx, ny, partner):
    B = gpu
    case = channel("a", nx, ny, storage)
    before, last, fields = single(case, 3 * EVERY)
    assert 0.0 < last < before
    # a tolerance never met: all steps run and the last check (the end itself is none) is the third's;
    # one between the third's residual and the second's: the third stops it
    for tol, steps in ((1e-300, 4 * EVERY), (0.5 * (last + before), 3 * EVERY + 1)):
        pool = B.Pool(4 << 30, max_slots=4, steps_per_launch=SPL)
        ids = [pool.submit(case, 4 * EVERY, keep_fields=True, stop=(tol, EVERY))]
        if partner:
            ids.append(pool.submit(channel("b", *partner, storage), 96, keep_fields=True))
        state, done, residual, obs, got = _drain(pool, ids)[ids[0]]
        pool.close()
        print(f"{storage} {nx}x{ny} with {partner}: {done} steps, residual {residual:.6e}, single {last:.6e}", flush=True)
        assert state == B.DONE and done == steps and obs["step"] == steps - 1
        assert abs(residual - last) <= 1e-9 * last      # FP64 sums in another order
    assert all((a == b).all() for a, b in zip(got, fields))
