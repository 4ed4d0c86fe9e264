"""The pinned memory of staged copies is shared by the handles of a process: many handles hold no more than
one does, and handles read by several threads at once get their own results."""
import ctypes as C
import os
import threading

import numpy as np
import pytest

from paper_1812_05401_amd import binding as B
from paper_1812_05401_amd import inputs as I

pytestmark = pytest.mark.gpu


def address_space():
    return int(open("/proc/self/statm").read().split()[0]) * os.sysconf("SC_PAGE_SIZE")


def read(sim, out):
    B.check(B.load().vplbm_observables(sim.h, None, *(a.ctypes.data_as(C.POINTER(C.c_double)) for a in out)))


def sims(n, nx, ny):
    """Handles of different states, their device staging memory allocated."""
    out = []
    for k in range(n):
        s = B.Simulation(I.Case("shared", nx, ny, storage="f16s", tau=0.6, bc=I.ALL_PERIODIC, u0=(0.01 + 0.002 * k, 0.0)), stream=None)
        s.init_fields(np.ones((ny, nx)), np.full((ny, nx), 0.01 + 0.002 * k), np.zeros((ny, nx)))
        out.append(s)
    return out


def test_many_handles_hold_one_handles_memory(gpu):
    nx, ny = 2000, 1500                                     # 72 MB of fields: the copy of eight threads
    handles = sims(20, nx, ny)
    out = [np.zeros((ny, nx)) for _ in range(3)]
    read(handles[0], out)                                   # the slots, and eight threads' stacks and heaps
    before = address_space()
    for s in handles[1:]:
        read(s, out)
    grown = address_space() - before
    print(f"20 handles: {grown / 2**20:.0f} MB more than one", flush=True)
    for s in handles:
        s.close()
    assert grown < 5 * (32 << 20)                           # 19 x 32 MB if each held its own


def test_handles_read_by_several_threads(gpu):
    nx, ny = 1201, 900
    handles = sims(12, nx, ny)
    want = []
    for s in handles:
        s.step(5)
        want.append(s.fields())
    bad = []

    def work(k):
        out = [np.zeros((ny, nx)) for _ in range(3)]
        for _ in range(5):
            for a in out:
                a.fill(np.nan)
            read(handles[k], out)
            if not all(bool((a == b).all()) for a, b in zip(out, want[k])):
                bad.append(k)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(handles))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for s in handles:
        s.close()
    assert not bad
