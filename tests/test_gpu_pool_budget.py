"""The pool's memory budget counts the sums of the bodies' forces that a request takes memory for."""
import pytest

from paper_1812_05401_amd import inputs as I
from tests.test_gpu_pool import run

pytestmark = pytest.mark.gpu


def case(storage, nbodies, bc=I.CHANNEL):
    """580 x 256 nodes; one small body, or eight that share the lattice among them."""
    nx, ny = 580, 256
    bodies = [I.body("disk", 150, 120, r=20)] if nbodies == 1 else [
        I.body("rect", (k % 4 + 0.5) * nx / 4, (k // 4 + 0.5) * ny / 2, hx=nx / 10, hy=ny / 5) for k in range(nbodies)]
    return I.Case("budget", nx, ny, storage=storage, tau=0.7, bc=bc, u_in=(0.03, 0.0), u0=(0.03, 0.0), bodies=bodies, steps=24)


@pytest.mark.parametrize("storage", ["f32", "f64", "f16s", "f16sr"])
@pytest.mark.parametrize("nbodies,together", [(1, 2), (8, 1)])
def test_two_requests_in_twice_the_memory_of_one(gpu, storage, nbodies, together):
    B = gpu
    c = case(storage, nbodies)
    need = B.vplbm_pool_bytes_needed(c)
    s = B.Simulation(c, stream=None)
    s.step(c.steps)
    so, *want = s.observables(fields=True)
    s.close()
    # one of eight bodies takes more than `need`: two do not fit together, and one still runs in `need`
    for budget, n in ((2 * need, 2), (need, 1)):
        res, most = run(B.Pool, [c] * n, budget, spl=8)
        assert most == (together if n == 2 else 1)
        for k in range(n):
            obs, fields = res[k]
            assert all(bool((a == b).all()) for a, b in zip(fields, want))
            assert abs(obs["mass"] - so["mass"]) <= 1e-13 * so["mass"]
            scale = max(abs(so["fx"]).max(), abs(so["fy"]).max())
            assert abs(obs["fx"] - so["fx"]).max() <= 1e-9 * scale and abs(obs["fy"] - so["fy"]).max() <= 1e-9 * scale
    with pytest.raises(B.VplbmError) as e:
        run(B.Pool, [c], need - 1, spl=8)
    assert e.value.code == B.EBUDGET
