// Mask rows of the strip sweep (strip_id_row): inside the lattice for every strip of every lattice of
// `steps` rows and up, and the row of the step once the step has begun.  Prints "ok", or the first fault.
#include <cstdio>

#include "strip_plan.hpp"

using namespace vplbm;

int main()
{
    for (int steps = 1; steps <= 8; steps++)
        for (int ny = steps < 3 ? 3 : steps; ny <= 24; ny++)
            for (int per = 0; per < 2; per++)
                for (int y0 = 0; y0 < ny; y0++)
                    for (int y1 = y0 + 1; y1 <= ny; y1++)
                        for (int i = 0; i < y1 - y0 + 2 * (steps - 1); i++)
                            for (int k = 0; k < steps; k++) {
                                const int row = strip_id_row(y0, steps, i, k, ny, per != 0);
                                const int y = y0 - (steps - 1) + i - k;
                                const bool used = i >= 2 * k && (per || (y >= 0 && y < ny));
                                if (row < 0 || row >= ny || (used && row != (y + ny) % ny)) {
                                    std::printf("steps %d ny %d periodic %d strip %d..%d iteration %d step %d: row %d\n", steps, ny, per, y0, y1, i, k, row);
                                    return 1;
                                }
                            }
    std::puts("ok");
    return 0;
}
