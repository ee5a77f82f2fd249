// The shifted and the skewed tile order visit every tile once: the one XCD by
// XCD within its band, the other row by row.
#include <cstdio>
#include <vector>

#include "fw2.h"
#include "fake_runtime.hpp"

int main()
{
    int bad = 0;
    for (int n = 1; n < 400; ++n)
        for (int shift : {1, 3, 24, 51, 1000}) {
            std::vector<int> seen(n, 0);
            for (int b = 0; b < n; ++b) {
                const int t = fw2::shifted_tile(b, n, shift), x = b % 8, rem = n % 8;
                const int begin = x * (n / 8) + (x < rem ? x : rem), end = begin + n / 8 + (x < rem ? 1 : 0);
                if (t < begin || t >= end || seen[t]++) ++bad;
            }
        }
    if (fw2::shifted_tile(8 * 5 + 2, 800, 7) != 200 + 5 + 14 || fw2::shifted_tile(8 * 99 + 1, 800, 7) != 100 + 6) ++bad;
    for (int nbx = 1; nbx < 40; ++nbx)
        for (int nby : {1, 2, 7, 30}) {
            std::vector<int> seen(nbx * nby, 0);
            for (int b = 0; b < nbx * nby; ++b) {
                const int t = fw2::skewed_tile(b, nbx);
                if (t / nbx != b / nbx || seen[t]++) ++bad;
            }
        }
    if (fw2::skewed_tile(3 * 64 + 60, 64) != 3 * 64 + 11) ++bad;
    std::printf("bands: %d failed\n", bad);
    return bad ? 1 : 0;
}
