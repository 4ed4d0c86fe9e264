"""Calls of few steps on lattices that take patches: what remains takes patches or the tiled kernels by size
and format, bitwise as one step per launch."""
import pytest

from paper_1812_05401_amd import inputs as I
from tests.test_gpu_strip import CHANNEL, OPEN, bodies, pair
from tests.test_gpu_two_step import STORAGES, same_run

pytestmark = pytest.mark.gpu


# on either side of 50,000, 90,000, 250,000 and 350,000 nodes
@pytest.mark.parametrize("storage", STORAGES)
@pytest.mark.parametrize("nx,ny,bc,moving", [(249, 200, CHANNEL, True), (253, 199, OPEN, False), (301, 301, I.CHANNEL_CONVECTIVE, True),
                                             (499, 503, I.CHANNEL_CONVECTIVE, False), (601, 590, I.ALL_PERIODIC, True)])
def test_remainders_bitwise_equal_one_step(gpu, nx, ny, bc, moving, storage):
    u = (0.04, 0.0)
    case = I.Case("remainders", nx, ny, storage=storage, tau=0.6, bc=bc, u_in=u if bc[0] == I.VELOCITY else (0, 0),
                  u0=u, bodies=bodies(nx, ny, moving))
    a, b = pair(case, storage, I.random_fields(nx, ny, 9, u_mean=u), VPLBM_PATCH=-1)
    done = 0
    for n in (1, 2, 3, 1, 4, 5, 6, 7, 8):
        a.step(n)
        b.step(n)
        done += n
    same_run(a, b, 0, done, f"{nx}x{ny} {storage}")
    a.close()
    b.close()
