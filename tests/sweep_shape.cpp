// sweep_shape.cpp -- TEST INFRASTRUCTURE: the shapes that the library chooses for
// sweeps of whole pencils, over grids of many and few, long and short pencils.
#include "ppmlr_march.hpp"

#include <cstdio>

using namespace ppmlr;

static bool bad(const Sweep &s, int P_req, const March &m, const char *why)
{
    std::printf("%dx%dx%d axis %d elem %d trace %d learned %d, %d asked: P=%d C=%d L=%d M=%d SM=%d: %s\n", s.n[0], s.n[1],
                s.n[2], s.axis, s.elem, s.trace, s.learned, P_req, m.P, m.C, m.L, m.M, m.SM, why);
    return false;
}

// A shape that a kernel exists for, whose chunks end where the pencil does.
static bool launchable(const Sweep &s, int P_req, const March &m)
{
    const int N = s.n[s.axis], threads = block_threads(m.P, m.M);
    if (m.P == 0) return true;
    if (P_req > 0 && m.P != P_req) return bad(s, P_req, m, "not the pencils asked for");
    if (m.C == 1) {
        if (m.M != N + 2 * kG || threads > 1024 || (m.SM > 0 && threads > m.SM)) return bad(s, P_req, m, "tile");
        if (!s.learned && m.SM != stride_for(threads, s.elem)) return bad(s, P_req, m, "not the tile kernel's rows");
        return true;
    }
    if (m.M != m.L + kG || (m.C - 1) * m.L >= N + kG || m.C * m.L < N + kG) return bad(s, P_req, m, "chunks");
    if (threads > 256 || threads > m.SM) return bad(s, P_req, m, "lanes");
    if (m.SM != 128 && m.SM != 192 && m.SM != 256 && m.SM != 320 && !(m.SM == 208 && s.elem == 8 && !s.trace))
        return bad(s, P_req, m, "rows");
    return true;
}

int main()
{
    long long n = 0, marches = 0;
    const int sizes[] = {1, 2, 3, 8, 14, 28, 32, 61, 97, 189, 192, 239, 300, 512, 1000, 1011, 4000};
    for (int nx : sizes)
        for (int ny : sizes)
            for (int nz : sizes)
                for (int axis = 0; axis < 3; ++axis)
                    for (int kind = 0; kind < 5; ++kind) {
                        const Sweep s = {{nx, ny, nz}, axis, kind < 3 ? 4 : 8, kind == 1 || kind == 4, kind == 2, nx % 2 == 0};
                        const March m = sweep_shape(s, 0);
                        ++n;
                        marches += m.C > 1;
                        if (!launchable(s, 0, m)) return 1;
                        for (int P : {1, 3, 8, 11, 40})
                            if (!launchable(s, P, sweep_shape(s, P))) return 1;
                        // tiles of one pencil read 4 B of every line they touch: not on a
                        // grid that fills the chip several times over
                        if (kind == 0 && axis > 0 && nx > 8 && m.C == 1 && m.P == 1 &&
                            (double)nx * ny * nz / s.n[axis] > 4000)
                            return bad(s, 0, m, "narrow rows on a full chip"), 1;
                        // FP64 tiles that spill are for grids that no march holds
                        if (m.C == 1 && s.elem == 8 && block_threads(m.P, m.M) > (s.trace ? 512 : 768) &&
                            march_shape(s.n[axis], m.P, 8, 320).P > 0)
                            return bad(s, 0, m, "a tile that spills"), 1;
                        // asked for the pencils that were chosen, the shape is the same
                        const March r = sweep_shape(s, m.P);
                        if (r.P != m.P || r.C != m.C || r.L != m.L || r.SM != m.SM) return bad(s, m.P, r, "not the shape chosen"), 1;
                        // one pencil per CU or fewer: nothing is gained by taking a
                        // pencil that a tile holds in parts that wait for each other
                        // (FP64 characteristic tiles of 9 waves and more spill)
                        const double pencils = (double)nx * ny * nz / s.n[axis];
                        const int threads = block_threads(1, s.n[axis] + 2 * kG);
                        if (pencils <= 256 && threads <= (kind == 4 ? 512 : 1024) && stride_for(threads, s.elem) > 0 && m.C != 1)
                            return bad(s, 0, m, "chunks in turn on an empty chip"), 1;
                    }
    std::printf("%lld sweeps, %lld marches\n", n, marches);
    return marches > 1000 ? 0 : 1;
}
