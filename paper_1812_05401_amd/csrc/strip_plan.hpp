// How a lattice is cut into the strips of a strip sweep, and which mask rows a strip reads (plain C++,
// no device code), kept apart from the runtime so it can be checked on its own.
#pragma once

#include <algorithm>
#include <vector>

namespace vplbm {

// A strip: its window's first own column, its rows y0 .. y1 - 1, and its form (StripForm).
struct StripTile {
    int x0, y0, y1, form;
};
enum StripForm { kPlain = 0, kMasked = 1, kEdge = 2 };

struct StripPlan {
    int nx, ny;
    bool xper, yper;
    int window, halo;        // columns of a window, and those on either side that are not its own
    int steps;               // per launch
    int nbox;                // boxes (x0, y0, w, h) inside the lattice that hold every solid node at every time
    const int (*box)[4];
};

// Time of one row of a strip, relative to a plain one: rows that may hold solid nodes load ids and
// may take the penalized collision; windows at an x edge load column by column.
inline double strip_row_cost(int form) { return form == kPlain ? 1.0 : form == kMasked ? 2.0 : 1.4; }

// The rows of each window that take one form (a StripTile each), to be cut into strips.
inline std::vector<StripTile> strip_segments(const StripPlan &p)
{
    std::vector<StripTile> segs;
    const int own = p.window - 2 * p.halo, reach = p.steps - 1;
    std::vector<char> solid(p.ny);
    for (int x0 = 0; x0 < p.nx; x0 += own) {
        const int first = x0 - p.halo, last = first + p.window - 1;
        if (first < 1 || last > p.nx - 2) {
            segs.push_back({x0, 0, p.ny, kEdge});
            continue;
        }
        // rows whose strip rows may see a solid node
        std::fill(solid.begin(), solid.end(), 0);
        bool clear = true;
        for (int b = 0; b < p.nbox; b++) {
            const int *q = p.box[b];
            if (q[0] > last || q[0] + q[2] <= first) continue;
            clear = false;
            for (int y = q[1] - reach; y < q[1] + q[3] + reach; y++) {
                if (y >= 0 && y < p.ny) solid[y] = 1;
                else if (p.yper) solid[((y % p.ny) + p.ny) % p.ny] = 1;
            }
        }
        for (int y = 0; y < p.ny;) {
            int e = clear ? p.ny : y + 1;
            while (e < p.ny && solid[e] == solid[y]) e++;
            segs.push_back({x0, y, e, solid[y] ? kMasked : kPlain});
            y = e;
        }
    }
    return segs;
}

// Rows of a strip of one form within time t: it computes 2 (steps - 1) rows beyond its own.
inline int strip_rows(double t, int form, int steps)
{
    const int r = (int)(t / strip_row_cost(form)) - 2 * (steps - 1);
    return r < 1 ? 1 : r;
}

// The least time (most: of a strip of that many rows) with count(time) <= slots, count falling with time.
template <typename F> double strip_time(int steps, int most, int slots, const F &count)
{
    double lo = 2 * (steps - 1) + 1, hi = 2.0 * (most + 2 * (steps - 1) + 1);
    for (int i = 0; i < 40; i++) {
        const double mid = 0.5 * (lo + hi);
        if (count(mid) <= slots) hi = mid;
        else lo = mid;
    }
    return hi;
}

// The strips of a lattice, at most `slots` of them if that can be: every strip takes about the same
// time, so that strips resident together end together.  Sorted by rows, then columns.
inline std::vector<StripTile> plan_strips(const StripPlan &p, int slots)
{
    const std::vector<StripTile> segs = strip_segments(p);
    const double t = strip_time(p.steps, p.ny, slots, [&](double t) {
        long long n = 0;
        for (const StripTile &s : segs) {
            const int r = strip_rows(t, s.form, p.steps);
            n += (s.y1 - s.y0 + r - 1) / r;
        }
        return n;
    });
    // f(strip) for every strip, by columns
    auto each = [&](auto f) {
        for (const StripTile &s : segs) {
            const int r = strip_rows(t, s.form, p.steps), h = s.y1 - s.y0, n = (h + r - 1) / r;
            for (int i = 0; i < n; i++)
                f(StripTile{s.x0, s.y0 + (int)((long long)h * i / n), s.y0 + (int)((long long)h * (i + 1) / n), s.form});
        }
    };
    std::vector<int> at(p.ny + 1);       // strips that begin below row y: a counting sort by rows
    each([&](const StripTile &s) { at[s.y0 + 1]++; });
    for (int y = 0; y < p.ny; y++) at[y + 1] += at[y];
    std::vector<StripTile> out(at[p.ny]);
    each([&](const StripTile &s) { out[at[s.y0]++] = s; });
    return out;
}

// Entries that hold the strips of a lattice whatever its `boxes` boxes are: plan_strips makes at most
// `slots` strips, or one of each segment if those are more.  Rows of a window that boxes reach form at
// most one run per box and, across a periodic edge, one more at either end; between and beside them lie
// the plain ones.
inline int strip_entries(int nx, int ny, int own, int boxes, int slots)
{
    const long long segments = (long long)((nx + own - 1) / own) * std::min(ny, 2 * boxes + 5);
    return (int)std::max<long long>(slots, segments);
}

// Whether step k (of 0 .. steps - 1) works in iteration i of a strip, on row y0 - (steps - 1) + i - k.  Before
// that its row may lie more than a lattice of few rows below row 0, where strip_row has no answer.
constexpr bool strip_begun(int i, int k) { return i >= 2 * k; }

// The row of the lattice that stands for row y of a strip: the wrapped one (rows that steps work on wrap
// once at most where ny >= steps), or beyond a free-slip edge the nearest.
constexpr int strip_row(int y, int ny, bool yper)
{
    if (yper) return y < 0 ? y + ny : y >= ny ? y - ny : y;
    return y < 0 ? 0 : y >= ny ? ny - 1 : y;
}

// The lattice column of a lane whose first column is ux: the wrapped one, or beyond a non-periodic edge
// the nearest inside that a load of `cols` columns may start at.
constexpr int strip_column(int ux, int cols, int nx, bool xper)
{
    if (xper) return ux % nx < 0 ? ux % nx + nx : ux % nx;
    return ux < 0 ? 0 : ux > nx - 1 ? (nx - 1) & ~(cols - 1) : ux;
}

// The id of column c of a lane whose ids, a byte each, were loaded together: where the second column (x1)
// lies beyond the last of an odd lattice, its byte is the row's padding and stands for no body.  (Where
// an id is used: made of the loaded ids it cost 1% of the sweep at 8192 x 2048, 26% at the load itself,
// which then waits.)
constexpr int strip_id(unsigned ids, int c, int x1, int nx) { return c == 0 ? int(ids & 0xFFu) : x1 < nx ? int(ids >> 8 & 0xFFu) : 0; }

// Strips to cut a lattice into: as many rounds of the `resident` waves that the GPU holds at once as
// leave a strip about `rows` rows (36, measured at 8192 x 2048 and 8192 x 8192: fewer, taller strips end
// less evenly, more compute too many rows twice), and one round of three quarters of them where that
// makes strips of under eight rows.
inline int strip_slots(long long nodes, int own, int resident, int rows)
{
    const double rounds = double(nodes) / own / rows / resident;
    if (nodes < 0.22 * 36.0 * own * resident) return resident * 3 / 4;
    const int n = rounds < 0.4 ? 1 : (int)(rounds + 0.6);
    return (int)std::min<long long>((long long)resident * 39 / 40 * n, 1 << 20);
}

// Entry of the sorted list that workgroup b of n takes: workgroups are dealt to the 8 XCDs
// round-robin, and each XCD takes one contiguous range of the list, so that windows that share
// cache lines stay in one L2.
inline int xcd_entry(int b, int n)
{
    const int q = n >> 3, r = n & 7;
    const int xcd = b & 7, j = b >> 3;
    return xcd < r ? xcd * (q + 1) + j : r * (q + 1) + (xcd - r) * q + j;
}

}  // namespace vplbm
