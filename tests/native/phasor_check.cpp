// Reads lines "q x" (hexadecimal floating point) and writes the cosine and sine parts of
// exp(-i q x) by phasor_fast, those by phasor_library, and the range limit for q, compiled
// from the kernels' own source.
#include <cstdio>
#include <cstdlib>

#include "phasor.h"

int main()
{
    char line[512];
    while (fgets(line, sizeof line, stdin) != nullptr) {
        char *end = nullptr;
        const double q = strtod(line, &end), x = strtod(end, nullptr);
        const numag::HalfTurns h = numag::half_turns(q);
        const double range = numag::phasor_range(q);
        double2 f = make_double2(0.0, 0.0);
        if (fabs(x) < range) f = numag::phasor_fast(h, x);
        const double2 l = numag::phasor_library(h, x);
        printf("%a %a %a %a %a\n", f.x, f.y, l.x, l.y, range);
    }
    return 0;
}
