"""CPU model of the strip sweep's indexing (strip.hpp): which source every step's pull reads, on
ragged lattices and every edge combination, and that every node is stored once.

The model moves identities through the same registers: a population is the tuple (step, direction,
x, y) of the node that produced it.  A pull is right when its nine values are those that the edge
rules name (edge_source in lattice.hpp), and a result is valid only if its pull was; the strip's own
nodes of the last step have to be valid, and so have all they depend on."""
import itertools
import os
import random
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1812_05401_amd", "csrc")

CX = [0, 1, 0, -1, 0, 1, -1, -1, 1]
CY = [0, 0, 1, 0, -1, 1, 1, -1, -1]
MIRROR = [0, 1, 4, 3, 2, 8, 7, 6, 5]


def halo(k_steps, cols):
    return k_steps - 1 if cols == 1 else (k_steps + 1) // 2 * 2


def edge_source(a, x, y, nx, ny, xper, yper):
    sx, sy, pa = x - CX[a], y - CY[a], a
    if sy < 0 or sy >= ny:
        if yper:
            sy %= ny
        else:
            sy, pa = y, MIRROR[a]
    if sx < 0 or sx >= nx:
        sx = sx % nx if xper else min(max(sx, 0), nx - 1)
    return pa, sx, sy


class Strip:
    """One wave: 64 lanes of `cols` columns, kept here as a flat list of 64 * cols columns."""

    def __init__(self, nx, ny, xper, yper, x0, y0, y1, k_steps, cols, shifted_loads):
        self.__dict__.update(locals())
        self.hx = halo(k_steps, cols)
        self.n = 64 * cols
        first, last = x0 - self.hx, x0 - self.hx + self.n - 1
        self.edge = first < 1 or last > nx - 2
        self.pull = cols == 1 or (not self.edge and shifted_loads)
        self.u = [first + i for i in range(self.n)]
        self.xw = [x for i in range(0, self.n, cols) for x in self.columns(self.u[i])]
        self.inlet = [self.edge and not xper and self.u[i] == 0 for i in range(self.n)]
        assert all(i % cols == 0 for i in range(self.n) if self.inlet[i])

    def columns(self, u):
        """Lattice columns of the lane whose first unwrapped column is u."""
        nx, cols = self.nx, self.cols
        if not self.edge:
            assert u >= 1 and u + cols <= nx - 1
            x = u
        elif self.xper:
            x = u % nx
        else:
            x = 0 if u < 0 else (nx - 1) // cols * cols if u > nx - 1 else u
        if cols == 1:
            return [x]
        if self.edge and self.xper and nx % 2:
            return [x, (x + 1) % nx]                # two loads
        assert x % 2 == 0 or not self.edge          # one load of a pair, inside the row's pitch
        assert x + 1 < (nx + 63) // 64 * 64
        return [x, x + 1]

    def source_column(self, i, shift):
        """Column that a load shifted by -1, 0 or 1 reads for column i."""
        if not self.edge:
            return self.xw[i] + shift
        if self.xper:
            return (self.xw[i] + shift) % self.nx
        return min(max(self.xw[i] + shift, 0), self.nx - 1) if shift else self.xw[i]

    def left(self, p):
        return [None] + p[:-1]

    def right(self, p):
        return p[1:] + [None]

    def from_right(self, p):
        q = self.right(p)
        if self.edge and not self.xper:
            q = [p[i] if self.u[i] == self.nx - 1 else v for i, v in enumerate(q)]
        return q

    def load_row(self, y):
        assert 0 <= y < self.ny
        rows = [y - 1, y, y + 1]
        low, high = y == 0, y == self.ny - 1
        if low:
            rows[0] = self.ny - 1 if self.yper else 0
        if high:
            rows[2] = 0 if self.yper else self.ny - 1
        f = []
        for a in range(9):
            ghost = not self.yper and (low if CY[a] > 0 else high if CY[a] < 0 else False)
            pa, r = MIRROR[a] if ghost else a, rows[1 - CY[a]]
            assert 0 <= r < self.ny
            col = [(0, pa, self.source_column(i, -CX[a] if self.pull else 0), r) for i in range(self.n)]
            if not self.pull and CX[a]:
                col = self.left(col) if CX[a] > 0 else self.from_right(col)
            f.append(col)
        return f

    def relax(self, k, f, y):
        """Results of step k on row y: valid where the whole pull is what the edge rules name."""
        yw = y % self.ny if self.yper else y
        out = [[None] * self.n for _ in range(9)]
        for i in range(self.n):
            if self.edge and not self.xper and not 0 <= self.u[i] < self.nx:
                continue
            ok = True
            for a in range(9):
                if self.inlet[i] and CX[a] > 0:
                    continue                      # the inlet rule overwrites these
                pa, sx, sy = edge_source(a, self.xw[i], yw, self.nx, self.ny, self.xper, self.yper)
                ok &= f[a][i] == (k, pa, sx, sy)
            if ok:
                for a in range(9):
                    out[a][i] = (k + 1, a, self.xw[i], yw)
        return out

    def sweep(self):
        """The nodes stored, each with whether its result is valid."""
        K, stored = self.k_steps, []
        yb, n = self.y0 - (K - 1), self.y1 - self.y0 + 2 * (K - 1)
        none = [None] * self.n
        win = [dict.fromkeys(("up2", "up5", "up6", "m0", "m1", "m3", "m2", "m5", "m6"), none) for _ in range(K - 1)]
        wrap = lambda y: y + self.ny if y < 0 else y - self.ny if y >= self.ny else y  # noqa: E731
        inside = lambda y: self.yper or 0 <= y < self.ny  # noqa: E731
        for i in range(n):
            y = yb + i
            f = self.load_row(wrap(y) if self.yper else min(max(y, 0), self.ny - 1))
            out = [none] * 9
            for k in range(K):
                y = yb + i - k
                if k:
                    w = win[k - 1]
                    if not self.yper and y + 1 == self.ny:
                        out[4], out[7], out[8] = w["m2"], w["m6"], w["m5"]
                    f = [w["m0"], w["m1"], w["up2"], w["m3"], out[4], w["up5"], w["up6"],
                         self.from_right(out[7]), self.left(out[8])]
                    w["up2"], w["up5"], w["up6"] = w["m2"], self.left(w["m5"]), self.from_right(w["m6"])
                    if not self.yper and y + 1 == 0:
                        w["up2"], w["up5"], w["up6"] = out[4], f[8], f[7]
                    w["m0"], w["m1"], w["m3"] = out[0], self.left(out[1]), self.from_right(out[3])
                    w["m2"], w["m5"], w["m6"] = out[2], out[5], out[6]
                    # a mirrored population keeps the name of the plane it comes from
                if i >= 2 * k and inside(y):
                    out = self.relax(k, f, y)
            if i >= 2 * (K - 1):
                y = yb + i - (K - 1)
                assert self.y0 <= y < self.y1
                for c in range(self.hx, self.n - self.hx):
                    if not self.edge or self.u[c] < self.nx:
                        stored.append((self.u[c], y, out[0][c] == (K, 0, self.xw[c], y)))
        return stored


def check(nx, ny, xper, yper, k_steps, cols, shifted_loads, rows):
    width = 64 * cols - 2 * halo(k_steps, cols)
    seen = {}
    for y0 in range(0, ny, rows):
        for x0 in range(0, nx, width):
            s = Strip(nx, ny, xper, yper, x0, y0, min(y0 + rows, ny), k_steps, cols, shifted_loads)
            for x, y, valid in s.sweep():
                assert 0 <= x < nx and 0 <= y < ny and valid, (x, y, valid)
                assert (x, y) not in seen
                seen[x, y] = 1
    assert len(seen) == nx * ny


FORMS = [(6, 2, True), (4, 2, False), (4, 1, True), (3, 1, True), (2, 2, False)]


@pytest.mark.parametrize("xper,yper", itertools.product((True, False), repeat=2))
@pytest.mark.parametrize("form", FORMS, ids=lambda f: f"{f[0]}steps_{f[1]}cols_{'shifted' if f[2] else 'aligned'}")
def test_every_pull_reads_the_source_the_edge_rules_name(form, xper, yper):
    for nx, ny, rows in [(3, 3, 4), (5, 4, 3), (61, 7, 4), (120, 9, 8), (129, 6, 5), (250, 5, 64),
                         (373, 21, 4)]:
        if ny >= form[0]:                           # fewer rows than steps take other kernels
            check(nx, ny, xper, yper, *form, rows)


@pytest.mark.parametrize("xper,yper", itertools.product((True, False), repeat=2))
@pytest.mark.parametrize("form,nsteps", [((8, 8, 8), 8), ((8, 8, 8), 3), ((16, 16, 6), 6), ((24, 16, 5), 5), ((24, 16, 5), 1),
                                         ((16, 16, 4), 3), ((26, 18, 4), 4), ((20, 17, 3), 2)])
def test_patch_pulls_read_the_source_the_edge_rules_name(form, nsteps, xper, yper):
    """The patches of patch.hip: every LDS read of a step lies in the region, on a node that the step
    before wrote, and is the source that edge_source names; every node is stored once."""
    tw, th, top = form
    ew, eh, skip = tw + 2 * (top - 1), th + 2 * (top - 1), top - nsteps
    for nx, ny in [(3, 3), (5, 4), (21, 9), (40, 25), (33, 50)]:
        stored = {}
        for x0, y0 in itertools.product(range(0, nx, tw), range(0, ny, th)):
            nodes = {}
            for ex, ey in itertools.product(range(ew), range(eh)):
                ux, uy = x0 + ex - (top - 1), y0 + ey - (top - 1)
                if (xper or 0 <= ux < nx) and (yper or 0 <= uy < ny):
                    nodes[ex, ey] = ux % nx, uy % ny, min(ex, ew - 1 - ex, ey, eh - 1 - ey)
            mid = {}
            for k in range(nsteps):
                out = {}
                for (ex, ey), (x, y, ring) in nodes.items():
                    if ring < skip + k:
                        continue
                    plain = (xper or 0 < x < nx - 1) and (yper or 0 < y < ny - 1)
                    ux, uy = x0 + ex - (top - 1), y0 + ey - (top - 1)
                    for d in range(9):
                        pa, sx, sy = edge_source(d, x, y, nx, ny, xper, yper)
                        if k and not (not xper and x == 0 and CX[d] > 0):
                            px, py, pd = ex - CX[d], ey - CY[d], d
                            if not plain:
                                if not yper and not 0 <= uy - CY[d] < ny:
                                    py, pd = ey, MIRROR[d]
                                if not xper and not 0 <= ux - CX[d] < nx:
                                    px = ex
                            assert mid[px, py] == (sx, sy) and pd == pa
                    out[ex, ey] = x, y
                    if k == nsteps - 1 and ring >= top - 1 and ux < nx and uy < ny:
                        assert (x, y) not in stored
                        stored[x, y] = 1
                mid = out
        assert len(stored) == nx * ny


def test_reduction_sets_are_distinct_and_folded_before_cleared():
    """The reduction sets of reduce.hpp (kMaxSteps, kAccSets of kernels.hpp) over random mixes of
    launches of 1 to kMaxSteps steps, as tests/test_two_step_indexing.py has them for three."""
    text = open(os.path.join(CSRC, "kernels.hpp")).read()
    most, sets = (int(re.search(rf"constexpr int {k} = (\d+);", text).group(1)) for k in ("kMaxSteps", "kAccSets"))
    assert sets >= 3 * most and sets & (sets - 1) == 0
    rng = random.Random(3)
    for _ in range(200):
        t, cleared, written = 0, {}, {}
        for li in range(60):
            n = rng.randint(1, most)
            fold = [t - 1 - d for d in range(most) if t - 1 - d >= 0]
            write, clear = list(range(t, t + n)), list(range(t + n, t + n + most))
            ids = [s % sets for s in fold + write + clear]
            assert len(set(ids)) == len(ids)
            assert all(cleared.get(s % sets, -1) < written[s] for s in fold)
            assert all(s < sets or cleared[s % sets] > written[s - sets] for s in write)
            written.update({s: li for s in write})
            cleared.update({s % sets: li for s in clear})
            t += n
