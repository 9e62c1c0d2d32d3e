// ppmlr_march.hpp -- LDS layout of a sweep workgroup and the shapes of a march
// (whole pencils in chunks): plain functions of sizes, the same on the host, in
// the kernels and in the CPU test of the layout.
#pragma once
#include <stddef.h>

#if defined(__HIPCC__)
#define PPMLR_HD __host__ __device__
#else
#define PPMLR_HD
#endif

namespace ppmlr {

constexpr int kG = 7;           // ghost zones per side
constexpr int kSlotsA = 16;     // values per zone in LDS buffer A
constexpr int kSlotsAGuess = 19;  // buffer A of the learned / harvest sweeps (3 more face values)
constexpr int kSlotsB = 8;       // values per zone in LDS buffer B
constexpr int kStatWords = 37;  // iteration histogram [32], floors, nonconverged, nonphys,
                                // learned-guess faces, learned-guess fallbacks

// Dynamic LDS of a sweep workgroup: the workgroup's scalars (16 doubles of
// per-wave signal-speed maxima, the kStatWords counters, the learned guess's
// face count or a persistent launch's barrier flag, and a persistent launch's
// tile claim), then the tile buffers A and B (slots values per zone, stride
// S).  A zone reads its neighbours' slots up to two zones away without a
// bounds test: what a zone at the end of a tile reads beyond it (another
// value's slot, the scalars in front, the guard of two zones behind) reaches
// ghost zones only, as the tile's 7 ghost zones are the radius of the whole
// sweep.  P: pencils per workgroup (the zones of y and z tiles are P slots
// apart).
constexpr int kLdsScalars = 16 * 8 + (kStatWords + 2) * 4;
PPMLR_HD constexpr size_t lds_guard(int P, int elem) { return ((size_t)2 * P * elem + 15) / 16 * 16; }
PPMLR_HD constexpr size_t lds_front(int P, int elem)
{
    constexpr size_t head = (kLdsScalars + 15) / 16 * 16;
    return lds_guard(P, elem) > head ? lds_guard(P, elem) : head;
}
PPMLR_HD constexpr size_t lds_bytes(int slots, int S, int elem, int P)
{
    return lds_front(P, elem) + ((size_t)slots * (size_t)S * (size_t)elem + 15) / 16 * 16 + lds_guard(P, elem);
}
// A march keeps the old first kG zones of a periodic axis behind the rows.
PPMLR_HD constexpr size_t lds_wrap_bytes(int P, int elem) { return (size_t)8 * kG * P * elem; }
constexpr int kCarry = 6;       // slots of every row that a march keeps for each pencil

// The zone slot n of a march's P * M that lane tid works on: its own, and for
// the lanes past them (padding to whole waves) the last one, which they read
// and do not write.  (With slots of their own, behind the carries, they read up
// to 63 slots past a row, and in the last row past the allocation.)
PPMLR_HD constexpr int march_lane(int tid, int S) { return tid < S ? tid : S - 1; }
// Its place in a row: kCarry slots stand before each pencil's zones (x), or
// before the zones of all pencils (y and z).
PPMLR_HD constexpr int march_slot(bool x, int n, int p, int P) { return n + kCarry * (x ? p + 1 : P); }

// Threads needed for a tile of P pencils, rounded to whole waves.
constexpr int block_threads(int P, int M) { return ((P * M + 63) / 64) * 64; }

// Shape of a march (whole pencils in chunks, see sweep_tile): P pencils per
// workgroup, C chunks of L zones, M = L + 7 zones per chunk, LDS stride SM.
struct March {
    int P = 0, C = 0, L = 0, M = 0, SM = 0;
};

// The march of P pencils of N zones in C chunks; P = 0 where the last chunk would
// be empty, a chunk shorter than 14 zones (but for a single one), or its zones
// and carries more than 4 waves or max_slots LDS slots per row.
inline March march_shape(int N, int P, int C, int max_slots)
{
    March m;
    m.L = (N + kG + C - 1) / C;
    if ((C > 1 && m.L < 2 * kG) || (C - 1) * m.L >= N + kG) return m;
    m.M = m.L + kG;
    const int slots = P * (m.M + kCarry);
    m.SM = slots <= 128 ? 128 : (slots + 63) / 64 * 64;
    if (block_threads(P, m.M) > 256 || m.SM > max_slots) return m;
    m.C = C;
    m.P = P;
    return m;
}

// LDS stride of a march as it is launched.  (FP64, three waves: four workgroups
// per CU with rows of 208 slots, three with 256: x sweep of 256x192x192, two
// pencils of 95 zones, 680 and 769 us; four waves are more lanes than that kernel
// is built for.)
inline int march_stride(const March &m, int elem, bool trace)
{
    const int waves = block_threads(m.P, m.M) / 64;
    return elem == 8 && !trace && waves <= 3 && m.SM == 256 && m.P * (m.M + kCarry) <= 208 ? 208 : m.SM;
}

}  // namespace ppmlr
