// Reads "geometry N k n_chains b sigma" per line and prints the estimated
// growth time in ms of the serving loop's size classes (request_cost.hpp).
#include <cstdio>
#include <cstring>

#include "request_cost.hpp"

int main()
{
    rsaw_config c;
    std::memset(&c, 0, sizeof(c));
    unsigned long long m;
    while (std::scanf("%d %d %d %llu %lf %lf", &c.geometry, &c.n_monomers, &c.k_trials, &m, &c.bond_length,
                      &c.bead_diameter) == 6) {
        c.n_chains = m;
        std::printf("%.17g\n", rsaw::estimate_ms(c));
    }
    return 0;
}
