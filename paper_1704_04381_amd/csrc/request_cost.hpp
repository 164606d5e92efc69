// Growth time of a request alone on the device, for the serving loop's size
// classes only (it never affects a result).  Host code.
//
// Fitted to the built-in kernels on one MI355X, growth kernels in ns per chain
// with enough chains to fill it (measured / model):
//   six neighbours   N = 64 0.113 / 0.123; 256 2.15 / 1.97; 1000 30.8 / 30.0 (a
//                    scan's N^2); 2048 95.5 / 95.0; 5000 387 / 397; 16384 2325 /
//                    2646 (site set: a step's time, and fewer chains resident)
//   26 neighbours    N = 64 0.474 / 0.471; 256 7.84 / 7.54; 400 19.3 / 17.0;
//                    2048 251 / 251; 8000 3710 / 2374
//   hard spheres     k = 8, sigma = b: N = 64 7.0 / 10.3; 256 67 / 95; 1000 261 /
//                    206; 3000 351 / 206.  k = 16, N = 1000 702 / 843; sigma = 0.3 b,
//                    N = 3000 4020 / 4860
// A hard-sphere chain ends after about 5 e^2 beads, e = k b / sigma.
#pragma once

#include <algorithm>
#include <cmath>

#include "rsaw.h"

namespace rsaw {

inline double estimate_ms(const rsaw_config &c)
{
    const double N = c.n_monomers;
    double ns;
    if (c.geometry == RSAW_REAL_HS) {
        const double e = c.k_trials * (c.bond_length / c.bead_diameter); // sigma = 0: infinite
        const double n = std::min(N, 6.5 * e * e);
        ns = 95.0 * std::pow(n / 256.0, 1.6) * std::max(1.0, c.k_trials / 16.0);
    } else if (c.geometry == RSAW_LATTICE_26) {
        ns = N <= 300 ? 1.15e-4 * N * N : 251.0 * std::pow(N / 2048.0, 1.65);
    } else {
        ns = N <= 1024 ? 3.0e-5 * N * N : 95.0 * std::pow(N / 2048.0, 1.6);
    }
    return (double)c.n_chains * ns * 1e-6;
}

} // namespace rsaw
