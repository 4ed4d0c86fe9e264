"""The serving pool after an advance that ended in an error: a cancelled simulation whose result could not
be stored is released by the next advance, and the device steps it no more."""
import contextlib
import os
import resource

import numpy as np
import pytest

from paper_1812_05401_amd import inputs as I
from tests.test_gpu_residual import _drain

pytestmark = pytest.mark.gpu


@contextlib.contextmanager
def little_host_memory(room):
    """At most `room` bytes of address space more than the process has now."""
    old = resource.getrlimit(resource.RLIMIT_AS)
    now = int(open("/proc/self/statm").read().split()[0]) * os.sysconf("SC_PAGE_SIZE")
    resource.setrlimit(resource.RLIMIT_AS, (now + room, old[1]))
    try:
        yield
    finally:
        resource.setrlimit(resource.RLIMIT_AS, old)


def channel(name, nx, ny, storage):
    return I.Case(name, nx, ny, storage=storage, tau=0.6, bc=I.CHANNEL, u_in=(0.04, 0.0), u0=(0.04, 0.0),
                  bodies=[I.body("disk", 0.3 * nx, 0.5 * ny, r=ny / 10)])


def test_a_failed_release_is_done_by_the_next_advance(gpu):
    B = gpu
    a, b, c = channel("a", 200, 150, "f32"), channel("b", 4032, 3000, "f16s"), channel("c", 4033, 3000, "f16s")
    need = [B.vplbm_pool_bytes_needed(x) for x in (a, b, c)]
    pool = B.Pool(need[2] + need[0] // 2, max_slots=4, steps_per_launch=8)   # b beside a, c alone
    # the same size once before, so that the pool's own memory for a result is there
    first = pool.submit(b, 8, keep_fields=True)
    while pool.status(first)[0] != B.DONE:
        pool.advance()
    pool.result(first)                                      # (not its fields: no freed arrays to take a result from)
    ra, rb, rc = pool.submit(a, 400, keep_fields=True), pool.submit(b, 400, keep_fields=True), pool.submit(c, 16, keep_fields=True)
    for _ in range(3):
        running, queued, _ = pool.advance()
        assert (running, queued) == (2, 1)
    pool.cancel(rb)
    with little_host_memory(24 << 20):                      # b's fields take 290 MB
        with pytest.raises(B.VplbmError) as e:
            pool.advance()
    assert e.value.code == B.ENOMEM
    assert pool.status(rb)[0] == B.RUNNING
    running, queued, _ = pool.advance()
    assert (running, queued) == (1, 1)                      # c waits for a
    state, done = pool.status(rb)
    assert state == B.CANCELLED and done < 400
    s = B.Simulation(b, stream=None)
    s.step(done)
    assert all(np.array_equal(x, y) for x, y in zip(pool.result(rb, fields=True)[1], s.fields()))
    s.close()
    res = _drain(pool, [ra, rc])
    for rid, case, n in ((ra, a, 400), (rc, c, 16)):
        state, done, _, obs, fields = res[rid]
        assert state == B.DONE and done == n and obs["status"] == 0
        s = B.Simulation(case, stream=None)
        s.step(n)
        assert all(np.array_equal(x, y) for x, y in zip(fields, s.fields()))
        s.close()
    assert pool.advance() == (0, 0, 4)
    pool.close()
