// The strips of random lattices and boxes (plan_strips): every node of every window in exactly one strip, of
// the form its rows need, in order of rows and columns, and no more strips than strip_entries says.  Prints "ok", or the first fault.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "strip_plan.hpp"

using namespace vplbm;

int main()
{
    std::mt19937 rng(7);
    auto pick = [&](int a, int b) { return a + (int)(rng() % (unsigned)(b - a + 1)); };
    for (int n = 0; n < 20000; n++) {
        const int cols = pick(1, 2), steps = pick(2, 6), halo = cols == 1 ? steps - 1 : (steps + 1) / 2 * 2, window = 64 * cols;
        const int nx = pick(3, 700), ny = pick(steps < 3 ? 3 : steps, n % 3 ? 90 : 16), nbox = pick(0, 8), slots = n % 4 ? pick(1, 60) : pick(60, 4000);
        int box[8][4];
        for (int b = 0; b < nbox; b++) {
            box[b][0] = pick(0, nx - 1);
            box[b][1] = pick(0, ny - 1);
            box[b][2] = pick(1, nx - box[b][0]);
            box[b][3] = pick(1, ny - box[b][1] < 6 ? ny - box[b][1] : 6);
        }
        const StripPlan p{nx, ny, (n & 1) != 0, (n & 2) != 0, window, halo, steps, nbox, box};
        const std::vector<StripTile> list = plan_strips(p, slots);
        const int own = window - 2 * halo;
        bool bad = (int)list.size() > strip_entries(nx, ny, own, 8, slots);
        std::vector<int> seen((size_t)((nx + own - 1) / own) * ny);
        for (size_t i = 1; i < list.size(); i++)
            bad |= list[i].y0 < list[i - 1].y0 || (list[i].y0 == list[i - 1].y0 && list[i].x0 <= list[i - 1].x0);
        for (const StripTile &s : list) {
            bad |= s.x0 % own != 0 || s.y0 < 0 || s.y1 <= s.y0 || s.y1 > ny;
            if (bad) break;
            for (int y = s.y0; y < s.y1; y++) seen[(size_t)(s.x0 / own) * ny + y]++;
            // no box within reach of a plain strip
            for (int b = 0; b < nbox && s.form == kPlain; b++)
                for (int y = s.y0 - (steps - 1); y < s.y1 + steps - 1; y++) {
                    const int yw = p.yper ? ((y % ny) + ny) % ny : y;
                    bad |= yw >= box[b][1] && yw < box[b][1] + box[b][3] && box[b][0] < s.x0 - halo + window && box[b][0] + box[b][2] > s.x0 - halo;
                }
        }
        for (int v : seen) bad |= v != 1;
        if (bad) {
            std::printf("lattice %d: %dx%d, %d boxes, %d slots, %d strips, room for %d\n", n, nx, ny, nbox, slots, (int)list.size(), strip_entries(nx, ny, own, 8, slots));
            return 1;
        }
    }
    std::puts("ok");
    return 0;
}
