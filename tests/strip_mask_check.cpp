// What the strip sweep reads of a mask.  Rows (strip_begun, strip_row): inside the lattice for every strip
// of every lattice of `steps` rows and up, and the row of the step.  Columns (strip_column,
// strip_id): of a row whose padding holds anything, only ids of the lattice's columns come through.
// Prints "ok", or the first fault.
#include <cstdio>
#include <vector>

#include "strip_plan.hpp"

using namespace vplbm;

static bool columns()
{
    for (int nx = 3; nx <= 300; nx++)
        for (int per = 0; per < (nx & 1 ? 1 : 2); per++) {   // (an odd periodic lattice takes two loads)
            std::vector<unsigned char> row((nx + 63) / 64 * 64, 0xEE);
            for (int x = 0; x < nx; x++) row[x] = (unsigned char)(x % 9);
            for (int ux = -6; ux < nx + 128; ux += 2) {
                const int x0 = strip_column(ux, 2, nx, per != 0), x1 = x0 + 1;
                const bool inside = x0 >= 0 && x0 < nx && x1 < (int)row.size() && x0 % 2 == 0;
                const unsigned ids = inside ? row[x0] | row[x1] << 8 : 0u;
                const int id0 = strip_id(ids, 0, x1, nx), id1 = strip_id(ids, 1, x1, nx);
                if (!inside || id0 != x0 % 9 || id1 != (x1 < nx ? x1 % 9 : 0)) {
                    std::printf("nx %d periodic %d column %d: ids %d %d\n", nx, per, ux, id0, id1);
                    return false;
                }
            }
        }
    return true;
}

int main()
{
    if (!columns()) return 1;
    for (int steps = 1; steps <= 8; steps++)
        for (int ny = steps < 3 ? 3 : steps; ny <= 24; ny++)
            for (int per = 0; per < 2; per++)
                for (int y0 = 0; y0 < ny; y0++)
                    for (int y1 = y0 + 1; y1 <= ny; y1++)
                        for (int i = 0; i < y1 - y0 + 2 * (steps - 1); i++)
                            for (int k = 0; k < steps; k++) {
                                if (!strip_begun(i, k)) continue;
                                const int y = y0 - (steps - 1) + i - k, row = strip_row(y, ny, per != 0);
                                const bool used = per || (y >= 0 && y < ny);
                                if (row < 0 || row >= ny || (used && row != (y + ny) % ny)) {
                                    std::printf("steps %d ny %d periodic %d strip %d..%d iteration %d step %d: row %d\n", steps, ny, per, y0, y1, i, k, row);
                                    return 1;
                                }
                            }
    std::puts("ok");
    return 0;
}
