// The stretch of the NUFFT's grid that a plan's channels occupy (plain C++, no
// HIP types, so that it can be checked on the host).
#pragma once

#include <vector>

struct NufftStretch {
    int b1;  // the FFT's first 2^b1-fold copy is skipped: 6, 3 or 0
    int p0;  // first point of the stretch (0 with b1 = 0)
};

// occupied[p]: some channel's kernel reaches point p.  The widest cyclic run of
// other points ends where the stretch starts; it takes 1/64 or 1/8 of the n
// points when it fits them and they are at least 16.
inline NufftStretch nufft_stretch(const std::vector<bool>& occupied)
{
    const int n = (int)occupied.size();
    int p0 = 0, gap = 0;
    for (int pp = 0, run = 0; pp < 2 * n; ++pp) {
        if (!occupied[pp % n]) {
            if (++run > gap && run <= n) {
                gap = run;
                p0 = (pp + 1) % n;
            }
        } else {
            run = 0;
        }
    }
    for (int b1 = 6; b1 > 0; b1 -= 3)
        if (n - gap <= n >> b1 && n >> b1 >= 16) return NufftStretch{b1, p0};
    return NufftStretch{0, 0};
}
