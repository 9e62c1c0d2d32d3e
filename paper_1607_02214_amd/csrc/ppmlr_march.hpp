// ppmlr_march.hpp -- LDS layout of a sweep workgroup and the shapes of a sweep of
// whole pencils (one tile of them, or a march through them in chunks): plain
// functions of sizes, the same on the host, in the kernels and in the CPU tests.
#pragma once
#include <algorithm>
#include <cmath>
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

// LDS stride of a tile with `threads` lanes: the smallest of the compile-time
// strides 256, 384, ..., 1024 (steps of 128) that holds them and whose two
// buffers fit the 160 KB LDS; 0 = the exact runtime stride (an FP64 tile of 832
// lanes, whose rounded stride would not fit); -1 = does not fit.  A stride
// close to the workgroup size leaves LDS for more resident workgroups per CU.
inline int stride_for(int threads, int elem)
{
    if (threads > 1024) return -1;
    const int sm = threads <= 256 ? 256 : (threads + 127) / 128 * 128;
    const int P = threads / (2 * kG + 1) + 1;   // at most: a tile's pencils have 15 zones or more
    if (lds_bytes(kSlotsA + kSlotsB, sm, elem, P) <= 160 * 1024) return sm;
    if (lds_bytes(kSlotsA + kSlotsB, threads, elem, P) <= 160 * 1024 && elem == 8) return 0;
    return -1;
}

// A sweep along axis, as far as its shape depends on it.
struct Sweep {
    int n[3];
    int axis, elem;
    bool trace, learned;        // characteristic tracing; the learned guess (FP32)
    bool wrap;                  // periodic axis
};

inline size_t march_lds(const Sweep &s, int P, int SM)
{
    return lds_bytes((s.learned ? kSlotsAGuess : kSlotsA) + kSlotsB, SM, s.elem, P) +
           (s.wrap ? lds_wrap_bytes(P, s.elem) : 0);
}

// How much a y or z sweep is slowed by rows of w 4-byte words (see march_time).
inline double row_cost(int axis, int w, bool cached)
{
    if (axis == 0) return 1.0;
    if (cached) return w >= 4 ? 1.0 : (w == 3 ? 1.1 : (w == 2 ? 1.15 : 1.7));
    return w >= 8 ? 1.0 : (w == 4 ? (axis == 1 ? 1.03 : 1.25) : (w > 4 ? 1.12 : (w == 3 ? 1.2 : (w == 2 ? 1.35 : 1.8))));
}

// What the estimates below start from: workgroups of P pencils that take C
// chunks one after the other, `waves` waves and `lds` bytes each, wps waves of
// that kernel on a SIMD; the workgroups of the sweep, how many of them a CU
// holds, the rounds of the whole chip that they make; and the us of a chunk
// alone, and for each wave on its CU.
struct Load {
    int nq, waves, places;
    double t0, t1, per_cu, wgs, rounds;
    bool cached;
    Load(const Sweep &s, int P, int waves_, size_t lds, int wps) : waves(waves_)
    {
        nq = s.axis == 0 ? s.n[1] : s.n[0];
        t0 = s.elem == 4 ? (s.trace ? 5.0 : 4.5) : 4.2;
        t1 = s.elem == 4 ? (s.trace ? 0.22 : 0.155) : (s.trace ? 0.78 : 0.52);
        // (waves of a workgroup of more than four meet on a SIMD: 5 take the places
        // of 8)
        places = waves > 4 ? (waves + 3) / 4 * 4 : waves;
        per_cu = std::max(1, std::min((int)(160 * 1024 / ((lds + 1279) / 1280 * 1280)), 4 * wps / places));
        wgs = (double)((nq + P - 1) / P) * (s.axis == 2 ? s.n[1] : s.n[2]);
        rounds = wgs / (256.0 * per_cu);
        cached = 8.0 * s.n[0] * s.n[1] * s.n[2] * s.elem < 128e6;
    }
};

// Estimated us of a march, for the choice among marches: the chunks, times the
// rounds, times the time of a chunk, which grows with the waves that share a CU
// (FP32, us: 4.5 + 0.155 per wave, from 256x192x192 sweeps at 8, 12, 16 and 20
// waves per CU: 560, 413, 336, 295 us).  In y and z, rows narrower than 32 B
// cost more (y, z sweep: 16 B 1.03, 1.25; 8 B 1.35; widths other than powers of
// two 1.1 to 1.2); less so where the state stays in the last-level cache
// (128x96x96: 16 B 1.0, 8 B 1.15).
inline double march_time(const Sweep &s, int P, int C, const Load &l)
{
    const double row = row_cost(s.axis, P * s.elem / 4, l.cached);
    // (a last round that is not full takes a round's time; with many rounds
    // workgroups follow each other and it is less)
    return l.rounds <= 1.0 ? C * row * (l.t0 + l.t1 * l.waves * std::ceil(l.wgs / 256.0))
                           : C * row * (l.t0 + l.t1 * l.waves * l.per_cu) * (l.rounds + 0.2);
}

// Estimated us of tiles (C = 1) and of a march, for the choice between them: as
// above, with what tells in few rounds.  On 362 sweeps of 150 random grids (24 to
// 420 zones an axis, every mode and precision) whose shape is not the one of
// march_time over tiles and marches alike: 0.88 of its time in the mean, 12 of
// them 3 to 13 % slower.  On 27 other grids the shape chosen was within 6 % of
// the fastest count of pencils on all but 20 of 330 sweeps.
inline double sweep_time(const Sweep &s, int P, int C, const Load &l)
{
    // (rows of the whole grid that are as narrow are one piece for all workgroups.
    // Tiles suffer more from narrow ones than marches do: 100x100x100, y and z,
    // rows of 8 B 1.3; 36x123x241, z, rows of 4 B 2.7, 33x167x189, y, 2.3)
    const int w = P * s.elem / 4;
    const double row = l.cached && l.nq * s.elem <= 32 ? 1.0
                       : l.cached && w <= 2 && s.axis > 0 ? (w == 2 ? (s.elem == 8 ? 1.3 : 1.4) : 2.4) : row_cost(s.axis, w, l.cached);
    const double full = row * (l.t0 + l.t1 * l.waves * l.per_cu);
    // a round that leaves room (where narrow rows cost what the waves of a CU wait
    // for each other): so many workgroups on the fullest CU
    auto part = [&](double n) { return l.t0 + row * l.t1 * 0.5 * (l.waves + l.places) * std::ceil(n / 256.0); };
    // a march sets up more (32^3 in FP64: 688 us for 20 steps, as tiles 661 us; x
    // sweep of 80^3 in FP32: 24.9 and 22.7 us.  The other modes' chunks are longer:
    // 128x96x96, x, characteristic, 57.4 us in two chunks, 64.7 us as a tile)
    const double n = C == 1 ? 1.0 : C * ((s.trace || s.learned ? 1.0 : 1.075) + 0.01 * (C - 2));
    // (the chip's loads come all at once as it fills)
    if (l.rounds <= 1.0) return n * part(l.wgs) * (1.0 + 0.2 * l.rounds);
    // (the second round, in step with those before and after it: 1.2 and 2.2 whole
    // rounds; a few workgroups of it find room as the first ones end)
    const double more = l.wgs - 256.0 * l.per_cu;
    if (l.rounds <= 2.0) return n * (1.2 * full + part(more) * std::min(1.0, 25.0 * (l.rounds - 1.0)));
    return n * full * (l.rounds + 0.2);
}

// The shape of a sweep of whole pencils, P_req of them per workgroup (0: chosen),
// or none (P = 0) where no workgroup holds them.  C = 1 is one tile of the
// pencils (M and SM are the tile's), C > 1 a march.
//
// A march's workgroups are held to 4 waves: one per SIMD, so that a CU fills
// evenly (with 5 or 7 waves, two of a workgroup meet on a SIMD, and half as many
// workgroups were resident: y sweep of 256x192x192 431 and 409 us against 304 us
// with 4).  Tiles of more waves are for grids of so few pencils that all are
// resident at once (FP32, one pencil: in two rounds), where the chunks of a
// march only wait for each other (x sweep of 1000x1x1 zones: 10 us as a tile, 24
// us in five chunks; of 500x500x1: 13 and 19 us; of 1000x1000x1, four rounds of
// tiles: 42 us in either).  More than 8 pencils are taken by tiles of four waves
// only: axes of up to 14 zones (3x300x300, x: 54 us with 7 or 8
// pencils, 36 us with 15).
inline March sweep_shape(const Sweep &s, int P_req)
{
    if (P_req > 0) {                                 // the pencils that are chosen: the shape that is
        const March m = sweep_shape(s, 0);
        if (m.P == P_req) return m;
    }
    const int N = s.n[s.axis], nq = s.axis == 0 ? s.n[1] : s.n[0];
    const int wps = s.elem == 4 ? (s.trace || s.learned ? 4 : 5) : (s.trace ? 2 : 3);     // waves per SIMD (registers)
    March march, tile;
    double march_t = 1e300, march_s = 1e300, tile_t = 1e300;
    for (int P = P_req > 0 ? P_req : 1; P <= (P_req > 0 ? P_req : 8); ++P)
        for (int C = 2; C <= 64 && (N + kG) / C >= kG; ++C) {
            March m = march_shape(N, P, C, 320);
            if (m.P == 0) continue;
            m.SM = march_stride(m, s.elem, s.trace);
            const Load l(s, P, block_threads(P, m.M) / 64, march_lds(s, P, m.SM), wps);
            const double t = march_time(s, P, C, l);
            if (t < march_t - 1e-9) { march_t = t; march_s = sweep_time(s, P, C, l); march = m; }
        }
    for (int P = P_req > 0 ? P_req : 1; P <= (P_req > 0 ? P_req : std::min(16, nq)); ++P) {
        const int threads = block_threads(P, N + 2 * kG);
        const int stride = s.learned ? (threads <= 256 ? 256 : (threads <= 512 ? 512 : 1024)) : stride_for(threads, s.elem);
        const bool wide = threads > 256;
        if (threads > 1024 || stride < 0 || (wide && P > 8 && P_req == 0)) continue;
        // (FP64 tiles of more than 12 waves, 8 with characteristic tracing, spill a
        // third of their registers: 189x26x36, x, four pencils 35 us, one 22 us)
        const bool spills = s.elem == 8 && threads > (s.trace ? 512 : 768);
        // (FP32 tiles have the registers for 6 waves per SIMD, of which the sixth is
        // room and no gain: z sweep of 100x100x100, 4 waves, 45 us, and 38 us as two
        // chunks at 5 per SIMD)
        const int tile_wps = wide && wps == 5 ? 6 : wps;
        const Load l(s, P, threads / 64, lds_bytes((s.learned ? kSlotsAGuess : kSlotsA) + kSlotsB,
                                                   stride > 0 ? stride : threads, s.elem, P), tile_wps);
        if ((spills || (wide && l.rounds > (P == 1 && tile_wps == 6 ? 2.0 : 1.0))) &&
            (P_req == 0 || march.P > 0))
            continue;
        const double t = sweep_time(s, P, 1, l);
        if (t < tile_t - 1e-9) {
            tile_t = t;
            tile.P = P; tile.C = 1; tile.L = N; tile.M = N + 2 * kG; tile.SM = stride;
        }
    }
    return tile.P > 0 && (march.P == 0 || tile_t <= march_s) ? tile : march;
}

}  // namespace ppmlr
