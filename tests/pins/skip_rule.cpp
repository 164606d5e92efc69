// Reads "b sigma d2" (binary64, hexadecimal) per line and prints the steps
// that real_skip.hpp lets a block of beads at squared distance d2 be skipped.
#include <cstdio>

#include "real_skip.hpp"

int main()
{
    double b, sigma, d2;
    while (std::scanf("%la %la %la", &b, &sigma, &d2) == 3) {
        const double bs = b + sigma, cull2 = bs * bs * (1.0 + 0x1p-30);
        const double unit = rsaw::skip_unit(b);
        std::printf("%d\n", rsaw::skip_steps((float)(d2 * unit), rsaw::skip_reach(cull2, unit)));
    }
    return 0;
}
