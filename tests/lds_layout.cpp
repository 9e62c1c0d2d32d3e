// lds_layout.cpp -- TEST INFRASTRUCTURE: every LDS slot that the lanes of a sweep
// workgroup touch, over all shapes that the library launches, against the
// bytes that the launch asks for.  Prints the shapes looked at; the first
// access outside ends it with exit code 1.
#include "ppmlr_march.hpp"

#include <cstdio>
#include <set>
#include <tuple>

using namespace ppmlr;

static long long shapes = 0;

// One workgroup of `lanes` lanes on P pencils of M zones (L of them owned, a
// march) or of a whole tile (L = 0), rows of S slots, `rows` rows.
static bool inside(bool x, int P, int M, int L, int S, int lanes, int rows, int elem)
{
    const long long bytes = (long long)lds_bytes(rows, S, elem, P), front = (long long)lds_front(P, elem);
    const int use = P * M, d = x ? 1 : P;
    long long lo = 0, hi = 0, wr = 0;
    for (int tid = 0; tid < lanes; ++tid) {
        const int n = L ? march_lane(tid, use) : tid, p = x ? n / M : n % P, i = x ? n - p * M : n / P;
        const int t = L ? march_slot(x, n, p, P) : n;
        if (t - 2 * d < lo) lo = t - 2 * d;          // the zones i - 2 .. i + 2, unbounded
        if (t + 2 * d > hi) hi = t + 2 * d;
        if (L && tid >= use) continue;               // (padding lanes of a march write nothing)
        if (t > wr) wr = t;
        // what a chunk leaves to the next: three sets, two of each in turn
        if (L && i == L - 1 && t - d * (L + 5) < (x ? p * (M + kCarry) : 0)) return false;
        if (L && i == 0 && t - d * (1 + 2 * 2 + 1) < (x ? p * (M + kCarry) : 0)) return false;
    }
    ++shapes;
    // the last row is read one zone to the right only, the others two
    const long long last = (long long)(rows - 1) * S, end = front + (last + hi - d + 1) * elem;
    const long long end2 = front + (last - S + hi + 1) * elem;
    if (front + lo * elem < 0 || end > bytes || end2 > bytes || wr >= S) {
        std::printf("%s P=%d M=%d L=%d S=%d lanes=%d rows=%d elem=%d: slots %lld..%lld, written to %lld, %lld of %lld bytes\n",
                    x ? "x" : "y/z", P, M, L, S, lanes, rows, elem, lo, hi, wr, end > end2 ? end : end2, bytes);
        return false;
    }
    return true;
}

int main()
{
    // marches: every shape of one context's sweep, and of an ensemble's (256
    // lanes whatever the shape, one row length)
    std::set<std::tuple<int, int, int, int, int>> seen;      // P, M, S, lanes, elem
    for (int N = 1; N <= 1100; ++N)
        for (int P = 1; P <= 128; ++P)
            for (int C = 1; C <= 80; ++C)
                for (int elem = 4; elem <= 8; elem += 4) {
                    const March m = march_shape(N, P, C, 320);
                    if (m.P)
                        for (int trace = 0; trace < 2; ++trace)
                            seen.insert({P, m.M, march_stride(m, elem, trace != 0), block_threads(P, m.M), elem});
                    const int S = elem == 4 ? 320 : 256;
                    const March e = march_shape(N, P, C, S);
                    if (e.P) seen.insert({P, e.M, S, 256, elem});
                }
    for (const auto &[P, M, S, lanes, elem] : seen)
        for (int x = 0; x < 2; ++x)
            for (int rows : {kSlotsA + kSlotsB, kSlotsAGuess + kSlotsB}) {
                if (rows > kSlotsA + kSlotsB && elem == 8) continue;
                if (!inside(x != 0, P, M, M - kG, S, lanes, rows, elem)) return 1;
            }
    std::printf("%lld marches\n", shapes);
    // tiles of segments and of whole pencils: rows as long as the workgroup or longer
    shapes = 0;
    for (int M = 15; M <= 1024; ++M)
        for (int P = 1; block_threads(P, M) <= 1024; ++P)
            for (int x = 0; x < 2; ++x)
                for (int elem = 4; elem <= 8; elem += 4)
                    if (!inside(x != 0, P, M, 0, block_threads(P, M), block_threads(P, M), kSlotsA + kSlotsB, elem))
                        return 1;
    std::printf("%lld tiles\n", shapes);
    return 0;
}
