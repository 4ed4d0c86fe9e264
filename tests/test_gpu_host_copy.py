"""Results in a caller's arrays: the staged copy to pageable memory at the sizes where its chunks, slots
and threads change, with some of the arrays left out, and to pinned memory."""
import ctypes as C

import numpy as np
import pytest

from paper_1812_05401_amd import binding as B
from paper_1812_05401_amd import inputs as I

pytestmark = pytest.mark.gpu

# nodes of 24 (fields) and 72 (populations) bytes: below and above 64 KB, 512 KB, 2, 8 and 64 MB
SIZES = [(30, 29), (67, 41), (131, 167), (301, 291), (613, 571), (1201, 583), (1601, 701)]


def same(got, want):
    # neighbouring values are 2^-30 apart; storing less the lattice weight rounds by 2^-53
    assert np.abs(got - want).max() <= 2.0 ** -50


@pytest.mark.parametrize("nx,ny", SIZES)
def test_results_arrive_whole(gpu, nx, ny):
    import torch
    case = I.Case("copy", nx, ny, storage="f64", tau=0.6, bc=I.ALL_PERIODIC, u0=(0.02, 0.01))
    sim = B.Simulation(case)
    try:
        n = nx * ny
        w = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)
        pop = w[:, None, None] + (np.arange(9 * n) % 1048573).reshape(9, ny, nx) * 2.0 ** -30
        sim.set_populations(pop)
        for _ in range(2):
            same(sim.populations(), pop)
        pinned = torch.empty((9, ny, nx), dtype=torch.float64, pin_memory=True)
        B.check(B.load().vplbm_get_populations(sim.h, C.cast(pinned.data_ptr(), C.POINTER(C.c_double))))
        same(pinned.numpy(), pop)
        straight = torch.empty((3, ny, nx), dtype=torch.float64, pin_memory=True)
        at = [C.cast(straight[i].data_ptr(), C.POINTER(C.c_double)) for i in range(3)]
        B.check(B.load().vplbm_observables(sim.h, None, *at))
        fields = straight.numpy()
        assert all((a == b).all() for a, b in zip(sim.fields(), fields)) and np.unique(fields[0]).size > 100
        for left_out in ((0,), (1,), (2,), (0, 1), (0, 2), (1, 2)):
            out = [np.full((ny, nx), np.nan) for _ in range(3)]
            ptr = [None if i in left_out else a.ctypes.data_as(C.POINTER(C.c_double)) for i, a in enumerate(out)]
            B.check(B.load().vplbm_observables(sim.h, None, *ptr))
            for i in range(3):
                assert np.isnan(out[i]).all() if i in left_out else (out[i] == fields[i]).all()
    finally:
        sim.close()
