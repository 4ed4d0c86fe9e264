// Steps per launch of the moving bodies' mask update (place_steps): the nodes of its steps, and the stride
// of its grid beyond them, fit an int, for up to eight boxes of the largest lattice.  Prints "ok".
#include <cstdio>

#include "step_plan.hpp"

int main()
{
    const int largest = 0x7FFFFFFF / 9;
    for (int steps = 1; steps <= 8; steps++)
        for (int boxes = 0; boxes <= 8; boxes++)
            for (int part = 1; part <= 64; part++) {
                const long long area = (long long)boxes * (largest / 64 * part);
                const int n = vplbm::place_steps(steps, (int)area);
                const long long last = n * area + 1024 * 256;
                if (last > 0x7FFFFFFF || (n != steps && n != 1) || (steps * area < (1LL << 30) && n != steps)) {
                    std::printf("%d steps of %lld nodes: %d\n", steps, area, n);
                    return 1;
                }
            }
    std::puts("ok");
    return 0;
}
