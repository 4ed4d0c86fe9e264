"""Moving bodies on lattices of an odd number of columns, in device memory that other data has filled
before: the masks of a launch's steps hold no ids beyond the last column."""
import pytest

from paper_1812_05401_amd import inputs as I
from tests.test_gpu_strip import CHANNEL, OPEN, bodies, pair
from tests.test_gpu_two_step import same_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f32", "f32d", "f16sr", "bf16sr"])
@pytest.mark.parametrize("nx,ny,bc", [(377, 40, OPEN), (1023, 64, CHANNEL)])
def test_moving_bodies_in_used_memory(gpu, nx, ny, bc, storage):
    import torch
    case = I.Case("used", nx, ny, storage=storage, tau=0.6, bc=bc, u_in=(0.04, 0.0), u0=(0.04, 0.0),
                  bodies=bodies(nx, ny, True))
    fill = [torch.full((n,), 0xEE, dtype=torch.uint8, device="cuda") for n in (1 << 22, 1 << 20, 1 << 18, 1 << 16) for _ in range(8)]
    torch.cuda.synchronize()
    del fill
    torch.cuda.empty_cache()
    a, b = pair(case, storage, I.random_fields(nx, ny, 8, u_mean=(0.04, 0.0)))
    a.step(25)
    b.step(25)
    same_run(a, b, 0, 25, f"{nx}x{ny} {storage}")
    a.close()
    b.close()
