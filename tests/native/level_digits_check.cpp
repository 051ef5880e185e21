// Prints, for each codebook read from stdin (bits, then 2^bits levels), the
// number of digit sets, whether the short sum does, and the values that the digits stand for, level by
// level, as the logit kernel sums them.
#include <cmath>
#include <cstdio>
#include <vector>

#include "isoq_internal.h"

int main()
{
    int bits;
    while (std::scanf("%d", &bits) == 1) {
        const int K = 1 << bits;
        float lev[16];
        for (int k = 0; k < K; k++)
            if (std::scanf("%f", lev + k) != 1)
                return 1;
        std::vector<isoq::LevelDigits> sets;
        const bool narrow = isoq::build_level_digits(bits, lev, sets);
        std::printf("%zu %d", sets.size(), (int)narrow);
        for (int k = 0; k < K; k++) {
            double v = 0;
            for (const isoq::LevelDigits &s : sets) {
                // 4 bits: magnitude k - 8, or the complement of magnitude 7 - k
                const int at = bits < 4 ? k : k >= 8 ? k - 8 : 7 - k;
                long n = 0;
                for (int t = 0; t < 3; t++) {
                    int d = (int)reinterpret_cast<const signed char *>(s.tab[t])[at];
                    if (bits == 4 && k < 8)
                        d = ~d;
                    n = 256 * n + d;
                }
                v += bits == 4 ? (n + 32896.5) * ((double)s.quantum / 32768.0) : n * ((double)s.quantum / 65536.0);
            }
            std::printf(" %.17g", std::ldexp(v, sets[0].exp));
        }
        std::printf("\n");
    }
    return 0;
}
