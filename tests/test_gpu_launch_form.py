"""The kernel and the steps of a full launch that the library names are those that it takes."""
import pytest

from paper_1812_05401_amd import inputs as I
from tests.test_gpu_two_step import STORAGES, env

pytestmark = pytest.mark.gpu


def form(nx, ny, storage, moving=False, **kw):
    from paper_1812_05401_amd import binding as B
    m = dict(ay=2.0, freq=0.001) if moving else {}
    with env(**kw):
        s = B.Simulation(I.Case("form", nx, ny, storage=storage, bodies=[I.body("disk", nx / 2, ny / 2, r=5, **m)]), stream=None)
    try:
        return s.launch_form, s.steps_per_launch
    finally:
        s.close()


@pytest.mark.parametrize("storage", STORAGES)
def test_forms_by_size(gpu, storage):
    wide = {"f32": 6, "f64": 5, "f32d": 4, "f16s": 4, "bf16s": 4, "f16sr": 3, "bf16sr": 3}[storage]
    tiled = 3 if storage == "f32" else 2
    assert form(100, 100, storage) == (("patches", 8), tiled)
    assert form(100, 100, storage, moving=True) == (("patches", 8), tiled)
    assert form(4096, 2048, storage) == (("strips", wide), tiled)
    assert form(4096, 2048, storage, moving=True) == (("strips", wide), tiled)
    assert form(4096, 2048, storage, VPLBM_STRIP=0) == (("tiles", tiled), tiled)
    assert form(100, 100, storage, VPLBM_PATCH=0) == (("tiles", tiled), tiled)
    assert form(4096, 2048, storage, VPLBM_THREE_STEP=0) == (("tiles", 2), 2)
    assert form(100, 100, storage, VPLBM_TWO_STEP=0) == (("tiles", 1), 1)
    # too few rows for the steps of a strip
    assert form(3000000, 3, storage)[0] == (("tiles", tiled) if wide > 3 else ("strips", 3))
