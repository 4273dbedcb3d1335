// A forward step shared between 256-row and 64-row workgroups: every 64 rows of every head are in exactly one of the two launches.
// Reads "nq n_q_tiles n_units" per line (n_units of 256 rows to the large workgroups) and prints how many of the line's row tiles are not
// covered exactly once.
#include <cstdio>
#include <iostream>
#include <vector>
#include "hexi_internal.h"

int main()
{
    int nq, n_q_tiles, n_units;
    while (std::cin >> nq >> n_q_tiles >> n_units) {
        const QShare share = {n_units / nq, n_units % nq};
        std::vector<int> seen((size_t)nq * n_q_tiles * 4, 0);
        for (int u = 0; u < share.n_units(nq); ++u) {
            int h, p;
            share.unit(u, &h, &p);
            for (int i = 0; i < 4; ++i) ++seen.at((size_t)h * n_q_tiles * 4 + 4 * (n_q_tiles - 1 - p) + i);
        }
        const QuadRest rest = rest_of(share, n_q_tiles);
        for (int h = 0; h < nq; ++h)
            for (int t = 0; t < rest.tiles; ++t)
                if (rest.has(h, t)) ++seen.at((size_t)h * n_q_tiles * 4 + t);
        int wrong = share.n_units(nq) != n_units;
        for (int n : seen) wrong += n != 1;
        std::printf("%d\n", wrong);
    }
    return 0;
}
