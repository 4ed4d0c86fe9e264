"""GPU tests of the serving pool's kernels: patches, strips of one or more blocks and tiles, a change
between them, lattices of hardly more rows than a launch has steps, simulations that end anywhere in a replay."""
import numpy as np
import pytest

from paper_1812_05401_amd import inputs as I
from tests.test_gpu_pool import run

pytestmark = pytest.mark.gpu

STORAGES = ["f32", "f64", "f32d", "f16s", "bf16s", "bf16sr", "f16sr"]


def cases(storage):
    """Rows around the steps per launch and the blocks' 4, 6 and 8; columns around one and two windows."""
    out = []
    for k, (nx, ny) in enumerate([(57, 3), (58, 4), (64, 5), (120, 6), (33, 9), (178, 17), (117, 40), (250, 73)]):
        bc = (I.ALL_PERIODIC, I.CHANNEL, I.CHANNEL_CONVECTIVE)[k % 3]
        u = (0.03, 0.01) if bc == I.ALL_PERIODIC else (0.04, 0.0)
        bodies = [I.body("disk", nx / 2, ny / 2, r=min(nx, ny) / 6, omega=0.002)] if ny >= 9 else []
        out.append(I.Case(f"strip{k}", nx, ny, collision="mrt" if k % 2 else "srt", storage=storage, tau=0.62 + 0.03 * k, bc=bc,
                          u_in=u if bc != I.ALL_PERIODIC else (0.0, 0.0), u0=u, bodies=bodies, steps=17 + 3 * k))
    return out


@pytest.mark.parametrize("spl", [1, 3, 14])
@pytest.mark.parametrize("storage", STORAGES)
def test_fields_are_the_single_simulations_in_any_mix(gpu, storage, spl):
    B = gpu
    small = cases(storage)
    # alone they take patches; beside this one strips (of several blocks) or tiles, until it has gone
    large = [I.Case("large", 2500, 1800, storage=storage, tau=0.7, bc=I.CHANNEL, u_in=(0.04, 0.0), u0=(0.04, 0.0),
                    bodies=[I.body("disk", 600, 900, r=60)], steps=16)]
    mix = run(B.Pool, small + large, 4 << 30, spl=spl)[0]
    for k, c in enumerate(small):
        obs, fields = mix[k]
        alone, alone_fields = run(B.Pool, [c], 1 << 30, spl=spl)[0][0]
        s = B.Simulation(c)
        s.step(c.steps)
        so, *want = s.observables(fields=True)
        s.close()
        for a, b, w in zip(fields, alone_fields, want):
            assert np.array_equal(a, b) and np.array_equal(a, w), c.name
        assert obs["mass"] == alone["mass"] and obs["step"] == so["step"] == c.steps - 1
        assert np.array_equal(obs["fx"], alone["fx"]) and np.array_equal(obs["fy"], alone["fy"])
        # sums of the same FP64 terms in another order
        assert abs(obs["mass"] - so["mass"]) <= 1e-13 * so["mass"]
        # a body's force: sums of at most 4000 terms of size 1 at most
        assert np.abs(np.array(obs["fx"]) - np.array(so["fx"])).max(initial=0.0) <= 4000 * 4000 * 2.0 ** -53
