// row_split.cpp -- TEST INFRASTRUCTURE: the share of every wave of the
// signal-speed kernels, over grids of many and few, long and short rows.
#include "ppmlr_rows.hpp"

#include <cstdio>
#include <vector>

using ppmlr::RowSplit;

// every zone is taken once, and no wave works through more columns in turn
// than an even share of them, rounded up, and one more
static bool covers(int nx, int rows, int waves)
{
    const RowSplit w(nx, rows, waves);
    std::vector<unsigned char> seen((size_t)nx * rows, 0);
    long long longest = 0;
    for (int wave = 0; wave < waves; ++wave) {
        long long chain = 0;
        for (long long n = wave; n < w.units(); n += waves) {
            const int group = (int)(n / w.parts), part = (int)(n % w.parts);
            const int end = (part + 1) * w.width < w.cols ? (part + 1) * w.width : w.cols;
            for (int col = part * w.width; col < end; ++col, ++chain)
                for (int lane = 0; lane < 64; ++lane) {
                    const int row = group * w.per + lane / w.lanes, i = col * w.lanes + lane % w.lanes;
                    if (row < rows && i < nx) ++seen[(size_t)row * nx + i];
                }
        }
        if (chain > longest) longest = chain;
    }
    for (unsigned char s : seen)
        if (s != 1) { std::printf("nx=%d rows=%d waves=%d: a zone taken %d times\n", nx, rows, waves, (int)s); return false; }
    // (groups that outnumber the waves keep their columns together)
    const long long total = (long long)w.groups * w.cols, even = (total + waves - 1) / waves;
    const long long limit = w.groups > waves ? even + w.cols : 2 * even;
    if (longest > limit) {
        std::printf("nx=%d rows=%d waves=%d: %lld columns in turn, even share %lld\n", nx, rows, waves, longest, even);
        return false;
    }
    return true;
}

int main()
{
    int n = 0;
    for (int nx : {1, 2, 3, 8, 9, 16, 17, 32, 33, 63, 64, 65, 97, 128, 129, 256, 300, 1000, 4000, 40001})
        for (int rows : {1, 2, 3, 7, 16, 63, 256, 1000, 5063})
            for (int waves : {4, 8, 60, 256, 1266, 8192}) {
                if ((long long)nx * rows > 6000000) continue;
                ++n;
                if (!covers(nx, rows, waves)) return 1;
            }
    std::printf("%d splits\n", n);
    return 0;
}
