// ppmlr_sweep.hpp -- gfx950 device code of one dimensionally split PPMLR-MHD
// sweep (paper, Section II: zone-centred averages, parabolic distribution in
// each zone, characteristic edge values, Lagrangian update with an interface
// Riemann solve, remap onto the Eulerian grid; Section III-A: one independent
// 1D problem per pencil).
//
// Execution model: one thread per zone, a workgroup owns one tile of P
// pencil segments (L interior zones + 7 ghosts per side each; one segment =
// the whole pencil) or marches along P whole pencils in chunks, and every
// stencil is served from LDS.  Successive stages
// exchange only what a neighbour needs, through two LDS buffers (A, B) with
// one barrier per exchange:
//   R1 load + primitives                                  -> A
//   R2 limited slopes (mass coordinate), shock test   A -> B
//      edge values                                   A, B -> A (slots 9..15)
//   R3 parabolas, tracing, interface states       A, B -> A
//   R4 Riemann solves, Lagrangian fluxes              A -> B
//   R5 Lagrangian zone contents                       B -> A
//   R6 limited slopes (volume coordinate)             A -> B
//      remap edge values                           A, B -> A (slots 8..14)
//   R7 remap parabolas, donor-cell fluxes             A -> B
//   R8 conservative update, sources, store            B
// The pencil axis is a template parameter so that all component indexing is
// static.  Private arrays are in registers, but for the wave structure of the
// characteristic mode (Waves7, 68 B a lane in FP32, 136 B in FP64): a choice
// between two of its members by a sign is compiled to a store at a computed
// address.
#pragma once
#include "ppmlr_char.hpp"
#include "ppmlr_march.hpp"
#include "ppmlr_mlp.hpp"
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ppmlr {

// The signal-speed maximum is accumulated in kCflSlots words kCflStride
// words apart (workgroup b uses slot b mod kCflSlots), so that the
// workgroups' atomics do not all queue on one address; readers take the
// maximum of the slots.
constexpr int kCflSlots = 64;
constexpr int kCflStride = 32;
constexpr int kStatSlots = 64;  // copies of the counters (workgroup b adds to copy b % 64)

enum { kPeriodic = 0, kOutflow = 1, kInflow = 2 };

// Arithmetic helpers: FP64 uses Newton-refined reciprocals and reciprocal
// square roots and the IEEE square root, FP32 the hardware reciprocal /
// square-root approximations (1 ulp).
template <typename T> struct Ar;
// FP64: the hardware reciprocal and reciprocal square root refined by two
// Newton steps each (quadratic convergence: faithfully rounded results for
// the positive, finite arguments of the sweep), in place of the
// correctly rounded division sequence (~10 instructions each).
__device__ inline double rcp64(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    double e = __builtin_fma(-x, r, 1.0);
    r = __builtin_fma(r, e, r);
    e = __builtin_fma(-x, r, 1.0);
    return __builtin_fma(r, e, r);
}
__device__ inline double rsqrt64(double x)
{
    double y = __builtin_amdgcn_rsq(x);
    const double h = 0.5 * x;
    double t = __builtin_fma(-h * y, y, 0.5);
    y = __builtin_fma(y, t, y);
    t = __builtin_fma(-h * y, y, 0.5);
    return __builtin_fma(y, t, y);
}
template <> struct Ar<double> {
    __device__ static inline double rcp(double x) { return rcp64(x); }
    __device__ static inline double div(double a, double b) { return a * rcp64(b); }
    __device__ static inline double sqrt_(double x) { return __builtin_sqrt(x); }
    // square root: x rsqrt(x) with one correction; zero and +infinity (class
    // bits 5, 6 and 9) are their own roots, where that form has no value
    __device__ static inline double sqrtp(double x)
    {
        const double y = rsqrt64(x), r = x * y;
        const double s = __builtin_fma(__builtin_fma(-r, r, x), 0.5 * y, r);
        return __builtin_amdgcn_class(x, 0x260) ? x : s;
    }
    __device__ static inline double rsqrt(double x) { return rsqrt64(x); }
};
template <> struct Ar<float> {
    __device__ static inline float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
    __device__ static inline float div(float a, float b) { return a * __builtin_amdgcn_rcpf(b); }
    __device__ static inline float sqrt_(float x) { return __builtin_amdgcn_sqrtf(x); }
    __device__ static inline float sqrtp(float x) { return __builtin_amdgcn_sqrtf(x); }
    __device__ static inline float rsqrt(float x) { return __builtin_amdgcn_rsqf(x); }
};

template <typename T> __device__ inline T tmin(T a, T b) { return a < b ? a : b; }
template <typename T> __device__ inline T tmax(T a, T b) { return a > b ? a : b; }
template <typename T> __device__ inline T tabs(T a) { return a < T(0) ? -a : a; }
// Element i of a global array at a uniform base address, addressed by a 32-bit
// byte offset (every array the sweep reads is below 4 GiB), so that the load
// or store takes the scalar-base + vector-offset form.  The address space is
// stated, as a base read from a descriptor in memory does not show it.
template <typename T> using global_t = __attribute__((address_space(1))) T;
template <typename T> __device__ inline T load(const T *base, unsigned int i)
{
    return *(const global_t<T> *)((const global_t<char> *)(const char *)base + i * (unsigned int)sizeof(T));
}
template <typename T> __device__ inline void store(T *base, unsigned int i, T v)
{
    *(global_t<T> *)((global_t<char> *)(char *)base + i * (unsigned int)sizeof(T)) = v;
}
// IEEE min / |x| / copysign in the type's own precision (the unsuffixed
// builtins are the double versions and would convert FP32 operands)
__device__ inline float fmin_(float a, float b) { return __builtin_fminf(a, b); }
__device__ inline double fmin_(double a, double b) { return __builtin_fmin(a, b); }
__device__ inline float fmax_(float a, float b) { return __builtin_fmaxf(a, b); }
__device__ inline double fmax_(double a, double b) { return __builtin_fmax(a, b); }
__device__ inline float fabs_(float a) { return __builtin_fabsf(a); }
__device__ inline double fabs_(double a) { return __builtin_fabs(a); }
__device__ inline float copysign_(float a, float b) { return __builtin_copysignf(a, b); }
__device__ inline double copysign_(double a, double b) { return __builtin_copysign(a, b); }
template <typename T> __device__ inline T tsgn(T a) { return a > T(0) ? T(1) : (a < T(0) ? T(-1) : T(0)); }

template <typename T>
struct SweepArgs {
    T *u;                       // state, SoA [8][nz][ny][nx]
    long long vol;              // zones per variable
    int N, M;                   // zones along the pencil; zones of one tile's segment, L + 2G
    int L, nseg;                // interior zones per segment (the last may be shorter), segments per pencil
    int nchunk;                 // march: chunks per pencil of L zones each (the left ghosts included)
    int Mext;                   // N + 2G: extent of the geometry tables along the pencil
    int P;                      // pencils per workgroup
    int S;                      // LDS slots = P * M
    long long stride_n, stride_q, stride_r;   // element strides
    float inv_div;              // 1 / M (x sweep) or 1 / P (y, z): lane -> (pencil, zone)
    const T *vin[8];            // base of each conserved variable of the input state
    T *var[8];                  // ... and of the output state (the same when whole pencils are swept in place)
    int nq, nr;                 // pencils along q (memory-fastest transverse) and r
    int tiles_q, ntiles, tiles_per_xcd;   // ntiles: tiles of one segment band (tiles_q * nr)
    int nslots;                 // tiles of one segment band: tiles_q * nr
    int seg_fast;               // 1: consecutive tiles are the segments of one pencil group; 0: bands in turn
    const T *dx, *xc, *xf;      // sweep axis: extended widths [Mext], centres [Mext], faces [Mext+1]
    const T *xc_q, *xc_r;       // transverse centres (interior zones)
    const T *rdx, *rdc;         // sweep axis, interior zones: 1 / dx, 1 / (x_{i+1} - x_{i-1})
    const T *rdx_q, *rdx_r;     // transverse 1 / dx (interior zones)
    int bc_lo, bc_hi;
    T gamma;
    T dt;                       // used when dt_dev == nullptr
    const double *dt_dev;       // device-resident dt (advance loop)
    // The first sweep of a step that advances the time: t_out += dt, with dt =
    // step, or, with dt_slots, step (the CFL number) over the maximum of the
    // signal-speed slots; dt_out receives it for the step's other sweeps.  A
    // kernel of its own for this took 3.3 us and a launch gap per step.
    double *t_out;
    double step;
    const unsigned long long *dt_slots;
    double *dt_out;
    unsigned long long *clear_slots;   // slots to clear (the step's second sweep), or null
    int has_bd;                 // background field present
    T dip_m, dir_x, dir_y, dir_z, bext_x, bext_y, bext_z;
    T in_rho, in_vx, in_vy, in_vz, in_bx, in_by, in_bz, in_p;   // inflow (total B)
    const double *in_dev;       // inflow of this step on the device (time series) or nullptr
    T r_inner2, inner_rho, inner_E;
    int has_inner;
    const double *inner_v;      // drift of the reset zones [3][box] (ionosphere coupling) or nullptr: at rest
    int ib[6];                  // its index box i0, i1, j0, j1, k0, k1 (half-open)
    int flatten, janhunen, max_iter;
    T tol, p_floor;
    unsigned long long *stats;  // kStatSlots x kStatWords counters or nullptr
    unsigned long long *cfl_max;// fused signal-speed max (double bits, kCflSlots slots) or nullptr
    // learned Riemann guess (FP32 single-run sweeps)
    const unsigned short *mlp_frag;       // packed BF16 weight fragments
    const float *mlp_theta;               // FP32 parameters (biases)
    T gate_p, gate_u;                     // relative pressure / velocity jump that selects a face
    float *harvest;                       // [harvest_cap][28] interface records or nullptr
    long long harvest_cap;
    unsigned long long *harvest_count;    // records offered (may exceed the capacity)
};

// Riemann initial-guess modes of the sweep body
enum { kGuessPlain = 0, kGuessLearned = 1, kGuessHarvest = 2 };

// Background field B_d = M [3 (m.r) r / r^5 - m / r^3] + b_ext along a
// pencil, in the pencil frame (n, t1, t2): t1, t2 are the cyclic successors of
// the sweep axis.  What depends on the pencil alone is set up once for the
// zone's two evaluations (centre and right face).
template <int AX, typename T>
struct PencilField {
    T c1, c2, ct2, mt3;            // transverse position, its square, 3 (m.r) of the transverse part
    T en, e1, e2, mn, m1, m2;      // uniform field, dipole direction
    template <typename A>
    __device__ inline PencilField(const A &a, T c1_, T c2_) : c1(c1_), c2(c2_)
    {
        const T e[3] = {a.bext_x, a.bext_y, a.bext_z}, m[3] = {a.dir_x, a.dir_y, a.dir_z};
        en = e[AX]; e1 = e[(AX + 1) % 3]; e2 = e[(AX + 2) % 3];
        mn = m[AX]; m1 = m[(AX + 1) % 3]; m2 = m[(AX + 2) % 3];
        ct2 = c1 * c1 + c2 * c2;
        mt3 = T(3) * (m1 * c1 + m2 * c2);
    }
    template <typename A>
    __device__ inline void at(const A &a, T n, T &bn, T &b1, T &b2) const
    {
        bn = en;
        b1 = e1;
        b2 = e2;
        if (a.dip_m != T(0)) {
            const T ir = Ar<T>::rsqrt(n * n + ct2);
            const T ir2 = ir * ir;
            const T g = a.dip_m * (ir2 * ir);                       // M / r^3
            const T c = ((T(3) * mn) * n + mt3) * ir2 * g;          // 3 M (m.r) / r^5
            bn = c * n + (bn - g * mn);
            b1 = c * c1 + (b1 - g * m1);
            b2 = c * c2 + (b2 - g * m2);
        }
    }
};

// Pencil-frame coordinates (n, t1, t2) of axis AX as (x, y, z).
template <int AX, typename T>
__device__ inline void to_xyz(T n, T t1, T t2, T &x, T &y, T &z)
{
    if (AX == 0) { x = n; y = t1; z = t2; }
    else if (AX == 1) { y = n; z = t1; x = t2; }
    else { z = n; x = t1; y = t2; }
}
template <int AX, typename T>
__device__ inline void to_pencil(T bx, T by, T bz, T &bn, T &b1, T &b2)
{
    if (AX == 0) { bn = bx; b1 = by; b2 = bz; }
    else if (AX == 1) { bn = by; b1 = bz; b2 = bx; }
    else { bn = bz; b1 = bx; b2 = by; }
}

// Median of three.
__device__ inline float med3_(float x, float y, float z) { return __builtin_amdgcn_fmed3f(x, y, z); }
__device__ inline double med3_(double x, double y, double z)
{
    return fmax_(fmin_(x, y), fmin_(fmax_(x, y), z));
}

// Half of the Eq. 1.8 limited slope sgn(da) min(|da|, 2|dm|, 2|dp|) (zero
// where dm and dp differ in sign), from hd = da / 2.  When dm and dp share a
// sign da shares it too (the weights of Eq. 1.7 are positive).  In single
// precision this is two medians: med(dm, dp, 0) is the one-sided difference
// nearer zero when the signs agree and zero otherwise, and med(hd, that, 0)
// clips hd to it.  The slopes travel halved (the edge weights take the factor
// back, exactly), which saves the doubling of every variable's clip value.
__device__ inline float limit_half(float hd, float dm, float dp) { return med3_(hd, med3_(dm, dp, 0.0f), 0.0f); }
__device__ inline double limit_half(double hd, double dm, double dp)
{
    const double r = copysign_(fmin_(fmin_(fabs_(hd), fabs_(dm)), fabs_(dp)), dp);
    return (dp * dm > 0.0) ? r : 0.0;
}

// Width weights of a zone on widths wm, w0, wp, wpp of zones j-1 .. j+2,
// shared by all variables: the (halved) average slope times width da_j / 2 =
// A (a_{j+1} - a_j) + B (a_j - a_{j-1}) (CW84 Eq. 1.7) and the right edge
// a_{j+1/2} = a_j + E0 (a_{j+1} - a_j) + E3 da_j / 2 - E2 da_{j+1} / 2
// (Eq. 1.6).
template <typename T>
struct Weights {
    T A, B, E0, E2, E3;
    __device__ inline Weights(T wm, T w0, T wp, T wpp)
    {
        const T sm = wm + w0, s0 = w0 + wp, sp = wp + wpp;
        const T i0 = Ar<T>::rcp(s0), q = wp + s0;                    // q = w0 + 2 wp
        const T cs = T(0.5) * w0 * Ar<T>::rcp(sm + wp);
        A = cs * (wm + sm) * i0;
        B = cs * q * Ar<T>::rcp(sm);
        const T f0 = w0 * i0, inv = Ar<T>::rcp(sm + sp);
        const T r1 = sm * Ar<T>::rcp(w0 + s0), r2 = sp * Ar<T>::rcp(q);
        const T u0 = (w0 + w0) * inv, up = (wp + wp) * inv;
        E0 = f0 + up * f0 * (r1 - r2);
        E2 = u0 * r1;
        E3 = up * r2;
    }
};

// Domain-of-dependence fraction y with its two shared coefficients: y / 2 and
// 6 (y / 2) (1 - 2 y / 3).
template <typename T>
struct Frac {
    T h, c;
    __device__ inline explicit Frac(T y) : h(T(0.5) * y), c(y * (T(3) - T(2) * y)) {}
};

// Zone parabola after the CW84 Eq. 1.10 monotonicity constraint: left and
// right edge L, R, their difference D and a sixth of the curvature, S = a -
// (L + R) / 2.  At a local extremum both edges take the zone average;
// otherwise the edge on the far side of an overshooting parabola is moved to
// 3a - 2a_other.  Both rules are one median each: for a monotone profile (say
// a_L < a < a_R) the overshoot test a6 > dA reads a_L < 3a - 2a_R, so the new
// left edge is max(a_L, 3a - 2a_R) = med(a_L, 3a - 2a_R, a) (a is the largest
// of the three); at an extremum 3a - 2a_R lies beyond a on the far side from
// a_L, so the median is a.  Likewise on the right with a_L and a_R exchanged.
template <typename T>
struct Para {
    T L, R, D, S;
    __device__ inline void set(T a, T aL, T aR)
    {
        const T a3 = T(3) * a;
        edges(a, med3_(aL, a3 - T(2) * aR, a), med3_(aR, a3 - T(2) * aL, a));
    }
    __device__ inline void edges(T a, T l, T r)
    {
        L = l;
        R = r;
        D = R - L;
        S = a - T(0.5) * (L + R);
    }
    // averages over the fraction y next to the right or left edge (Eq. 1.12)
    __device__ inline T right(const Frac<T> &f) const { return R - f.h * D + f.c * S; }
    __device__ inline T left(const Frac<T> &f) const { return L + f.h * D + f.c * S; }
};

// Counter update aggregated per wave: the lowest active lane of each group of
// lanes with the same bin adds the group's population to the workgroup's LDS
// counters (flushed to global memory once per workgroup).
__device__ inline void wave_add(unsigned int *s_ctr, bool pred)
{
    unsigned long long m = __ballot(pred);
    if (m != 0ull && __lane_id() == __ffsll((long long)m) - 1) atomicAdd(s_ctr, (unsigned int)__popcll(m));
}
__device__ inline void wave_hist(unsigned int *s_hist, bool counted, int bin)
{
    // bin 0 (a face whose linear guess already meets the tolerance) is by far
    // the most common: one ballot for it, then a loop over the other bins
    const unsigned long long zero = __ballot(counted && bin == 0);
    if (zero != 0ull && __lane_id() == __ffsll((long long)zero) - 1)
        atomicAdd(&s_hist[0], (unsigned int)__popcll(zero));
    unsigned long long active = __ballot(counted && bin != 0);
    while (active) {
        int leader = __ffsll((long long)active) - 1;
        int lb = __shfl(bin, leader);
        unsigned long long same = __ballot(counted && bin == lb);
        if (__lane_id() == leader) atomicAdd(&s_hist[lb], (unsigned int)__popcll(same));
        active &= ~same;
    }
}

// Inputs of the learned guess for one face (see the Riemann block of
// sweep_tile): sides s = (rho, u, v_t1, v_t2, B_t1, B_t2, P), normalised by
// the pair means; Pbar and cbar are the mean pressure and sqrt(P/rho).
template <typename T>
__device__ inline void guess_features(const T *L, const T *R, T *feat, T &Pbar, T &cbar)
{
    const T rbar = T(0.5) * (L[0] + R[0]);
    Pbar = T(0.5) * (L[6] + R[6]);
    const T irb = Ar<T>::rcp(rbar), iPb = Ar<T>::rcp(Pbar);
    cbar = Ar<T>::sqrt_(Pbar * irb);
    const T icb = Ar<T>::rcp(cbar), ibs = Ar<T>::rsqrt(Pbar);
    const T ub = T(0.5) * (L[1] + R[1]), v1b = T(0.5) * (L[2] + R[2]), v2b = T(0.5) * (L[3] + R[3]);
    const T *side[2] = {L, R};
#pragma unroll
    for (int sd = 0; sd < 2; ++sd) {
        const T *x = side[sd];
        T *f = feat + 7 * sd;
        f[0] = x[0] * irb;
        f[1] = (x[1] - ub) * icb;
        f[2] = (x[2] - v1b) * icb;
        f[3] = (x[3] - v2b) * icb;
        f[4] = x[4] * ibs;
        f[5] = x[5] * ibs;
        f[6] = x[6] * iPb;
    }
}

// Whether a face is selected: a strong jump of the pressure or the velocity.
template <typename T>
__device__ inline bool guess_selects(T rl, T rr, T ul, T ur, T pl, T pr, T gate_p, T gate_u)
{
    const T cbar = Ar<T>::sqrt_(T(0.5) * (pl + pr) * Ar<T>::rcp(T(0.5) * (rl + rr)));
    return tabs(pr - pl) > gate_p * tmin(pl, pr) || tabs(ur - ul) > gate_u * cbar;
}

// One tile of a sweep, executed by one workgroup: P pencils, each cut to
// segment `seg` (interior zones seg*L .. seg*L + L - 1 with G zones on either
// side; one segment = the whole pencil).  A zone's result depends on the
// zones within G of it only, so segments give the whole-pencil result
// bit for bit.  Neighbours are read without a bounds test (see the LDS layout):
// what a zone at an end of the tile reads beyond it has no meaning, and reaches
// no further than the G ghosts there, the radius of all stages together; a stage
// that reads further needs more ghosts.  tq, r: tile position (q tiles of P
// pencils, r the slow transverse index).  The state is read through a.vin
// and written through a.var: the same buffer for whole pencils, different
// buffers for segments (a segment's ghost zones are other segments' interior
// zones).  dt: the time step; cfl_max: target
// of the fused signal-speed maximum (FUSE_CFL); stat_slot: which copy of the
// counters this workgroup adds to.
// SM: LDS stride per stored value (so that every LDS access uses an immediate
// offset), or 0 for a runtime stride, the workgroup size.
// MARCH: the workgroup takes its P pencils whole, in a.nchunk chunks of L zones
// plus 7 ghosts on the right, one after the other and in place.  What a chunk's
// first zone needs of the zones on its left (primitives, edges, fluxes,
// Lagrangian contents, remap edges and fluxes) the chunk before left in LDS,
// so each zone is computed once but for the 7, and bit for bit as in a whole
// pencil.  A tile of a whole 192-zone pencil needs 13 waves in step and leaves
// one workgroup on a CU; chunks of 25 zones of 8 pencils are 4 waves, five
// workgroups a CU, rows of 32 B in y and z.  256x192x192, one sweep, x / y / z:
// FP32 456 / 515 / 553 us as whole-pencil tiles, 306 / 295 / 291 us as marches;
// FP64 1394 / 1167 / 1266 us against 680 / 665 / 700 us.  Requesting the next
// chunk's zones ahead was measured and is not done (315 / 302 / 299 us): with
// 20 waves on a CU the loads are covered, and the registers are not there; nor
// by a load or two per lane that only bring its rows into the L2 (6 % slower,
// 15 % at 512x384x384; loads return in order, and the later ones of the chunk
// would wait behind them).
// GUESS: initial guess of the normal-pair Newton iteration: the plain linear
// guess, the learned (MLP) guess on selected faces, or the plain guess with
// the selected faces' states and solutions recorded for training.  s_guess:
// one LDS counter (learned mode).
// Margin of the shock detector's compression test, in sound speeds
// sqrt(P / rho): no shock compresses by less, and a strict u_{j-1} > u_{j+1}
// at a pressure jump at rest would let rounding noise decide flattening.
constexpr double kCompMin = 1e-5;

template <int AX, typename T, bool STATS, bool FUSE_CFL, int SM, int GUESS = kGuessPlain, bool TRACE = false,
          bool MARCH = false, typename ARGS>
__device__ __forceinline__ void sweep_tile(const ARGS &args, const int tq, const int r, const int seg, const T dt,
                                           unsigned long long *cfl_max, const int stat_slot,
                                           unsigned char *smem_raw, double *s_red, unsigned int *s_stat,
                                           unsigned int *s_guess = nullptr)
{
    static_assert(GUESS == kGuessPlain || (SM > 0 && sizeof(T) == 4 && STATS),
                  "learned / harvest modes are FP32 sweeps with a compile-time stride and counters");
    static_assert(!TRACE || GUESS == kGuessPlain, "the characteristic mode takes the plain interface solve");
    const int S = SM > 0 ? SM : (int)blockDim.x;          // LDS stride
    if (STATS && threadIdx.x < kStatWords) s_stat[threadIdx.x] = 0u;   // ordered by the first barrier
    constexpr int kn = AX, k1 = (AX + 1) % 3, k2 = (AX + 2) % 3;
    T cq;                                                 // the pencil's coordinate along q
    // signal-speed maximum in the sweep's precision: a maximum selects one
    // value, so reducing in FP32 and converting the result gives the FP64
    // maximum of the converted values exactly
    T smax = T(0);
    const int nch = MARCH ? args.nchunk : 1;
    for (int ch = 0; ch < nch; ++ch) {
    // A march's arguments and lane indices are formed anew in every chunk:
    // held over the loop they take more scalar and vector registers than there
    // are, and are spilled (134 lane reads per chunk, measured).
    const ARGS *ap = &args;
    int tid = threadIdx.x;
    if (MARCH) {
        asm volatile("" : "+s"(ap));
        asm volatile("" : "+v"(tid));
    }
    const ARGS &a = *ap;
    T *sA = reinterpret_cast<T *>(smem_raw + lds_front(a.P, (int)sizeof(T)));
    T *sB = sA + (GUESS == kGuessPlain ? kSlotsA : kSlotsAGuess) * S;
    const int q0 = tq * a.P;
    const int Suse = a.S, M = a.M, N = a.N, P = a.P;
    const bool slot_ok = tid < Suse;
    // this lane's zone of the tile or chunk (the lanes that pad a workgroup to
    // whole waves load the last one's line and no lines of their own: y sweep of
    // 192x160x160 in tiles of one pencil, 94 zones in 128 lanes, 454 and 403 us)
    const int zn = march_lane(tid, Suse);
    int p, i;
    // zn / divisor as floor((zn + 1/2) * (1/divisor)): exact for zn < 2^12
    // and divisors up to 2^11 (the distance to the next integer, >= 1/(2 div),
    // exceeds the rounding error, < zn * 2^-23 / div)
    const int qd = (int)(((float)zn + 0.5f) * a.inv_div);
    if (AX == 0) { p = qd; i = zn - p * M; }              // zones of a pencil adjacent
    else { i = qd; p = zn - i * P; }                      // pencils adjacent (coalesced)
    // slot offset of zone i+1 (kept from the compiler for x, which would fold
    // it into address arithmetic per slot)
    int d = (AX == 0) ? 1 : P;
    if (AX == 0) asm("" : "+s"(d));
    const int q = q0 + p;
    const int Mext = a.Mext, L = a.L;
    // This lane's LDS slot and those of the zones i+1, i+2 (see the LDS layout
    // for the ends of a tile).  A march keeps kCarry slots of every row before
    // each pencil's zones, what a chunk's last zone leaves to the next chunk: three
    // sets, two of each in turn.
    const int t = MARCH ? march_slot(AX == 0, zn, p, P) : tid;
    const int sp1 = t + d, sp2 = sp1 + d;
    T *sP = sB + kSlotsB * S;                             // march on a periodic axis: old zones 0 .. 6
    const bool wrap = MARCH && a.bc_hi == kPeriodic;
    const T gam = a.gamma;

    const int qq = q < a.nq ? q : a.nq - 1;
    // q is t1 for the x and z sweeps, t2 for the y sweep
    const int j1 = AX == 1 ? r : qq, j2 = AX == 1 ? qq : r;
    (void)j1; (void)j2;
    // 32-bit element offsets within one variable (the host keeps a variable
    // below 4 GiB); each variable's base pointer is uniform
    const unsigned int base = (unsigned int)(qq * (int)a.stride_q + r * (int)a.stride_r);

    // ------------------------------------------------------------ R1
    const bool first = !MARCH || ch == 0;                 // ghosts on the left
    const int ie = (MARCH ? ch : seg) * L + i;            // index into the extended tables
    if (first) cq = load(a.xc_q, qq);
    const int ic = ie < Mext ? ie : Mext - 1;
    const T dxi = load(a.dx, ic);
    const T xci = load(a.xc, ic);
    const T xfr = load(a.xf, ic + 1);
    int src = ie - kG;
    if (src < 0) {
        if (a.bc_lo == kPeriodic) { src = src % N; if (src < 0) src += N; }
        else src = 0;
    } else if (src >= N) {
        src = a.bc_hi == kPeriodic ? src % N : N - 1;
    }
    // conserved state in pencil frame: rho, mn, m1, m2, bn, b1, b2, E (every
    // lane loads a zone of the pencil, inflow ghosts are replaced below)
    T Q[8];
    {
        const unsigned int o = base + (unsigned int)(src * (int)a.stride_n);
        Q[0] = load(a.vin[0], o);
        Q[1] = load(a.vin[1 + kn], o);
        Q[2] = load(a.vin[1 + k1], o);
        Q[3] = load(a.vin[1 + k2], o);
        Q[4] = load(a.vin[4 + kn], o);
        Q[5] = load(a.vin[4 + k1], o);
        Q[6] = load(a.vin[4 + k2], o);
        Q[7] = load(a.vin[7], o);
    }
    // transverse coordinates of the pencil
    const T cr = load(a.xc_r, r);
    const T c1 = AX == 1 ? cr : cq, c2 = AX == 1 ? cq : cr;
    const int g = ie - kG;                                // zone index along the pencil
    const bool pen = slot_ok && q < a.nq && ie < Mext;
    // zones that this tile or chunk updates, and the faces it owns (counted
    // and recorded once per pencil): -1/2 .. N-1/2 over all of them
    const int glo = MARCH ? (ch == 0 ? 0 : ch * L - kG) : seg * L;
    const int gend = min(MARCH ? (ch + 1) * L - kG : glo + L, N);
    const int own_lo = (MARCH ? ch == 0 : seg == 0) ? -1 : glo;
    const bool interior = pen && g >= glo && g < gend;
    const bool face_ok = pen && i >= (first ? 3 : 0) && i <= M - 5;   // faces whose two states are complete
    if (GUESS == kGuessLearned && tid == 0) s_guess[0] = 0u;
    // lanes past the tile do not write in a march: the slots behind are taken
    const bool keeps = !MARCH || slot_ok;
    // March: a chunk's first zone takes what it needs of the zones on its left
    // from the slots where the chunk before left them, so that no ghost zone
    // is computed again there.
    const bool carried = MARCH && ch > 0 && i == 0;
    const bool leaves = MARCH && slot_ok && i == L - 1;   // the next chunk's left neighbour
    auto left = [&](int set) -> int { return t - d - (carried ? d * (2 * set + (ch & 1)) : 0); };
    auto cslot = [&](int set) -> int { return t - d * (L + 2 * set + ((ch + 1) & 1)); };
    if (wrap && nch > 1) {
        // the zones behind a periodic end are the first ones, which chunk 0 updates
        if (ch == 0 && slot_ok && g >= 0 && g < kG) {
#pragma unroll
            for (int k = 0; k < 8; ++k) sP[(k * kG + g) * P + p] = Q[k];
        }
        if (ch > 0 && slot_ok && g >= N) {
            const int z = min(g - N, kG - 1);
#pragma unroll
            for (int k = 0; k < 8; ++k) Q[k] = sP[(k * kG + z) * P + p];
        }
    }
    const bool inflow_zone = (g < 0 && a.bc_lo == kInflow) || (g >= N && a.bc_hi == kInflow);
    // centre and right-face background field (pencil frame)
    T bdn = 0, bd1 = 0, bd2 = 0, bfn = 0, bf1 = 0, bf2 = 0;
    if (a.has_bd) {
        const PencilField<AX, T> fld(a, c1, c2);
        fld.at(a, xci, bdn, bd1, bd2);
        fld.at(a, xfr, bfn, bf1, bf2);
    }
    if (inflow_zone) {
        // inflow ghost: primitive inflow state with B' = B_in - B_d(centre)
        // (a time series of inflow states puts this step's in a.in_dev)
        T in[8] = {a.in_rho, a.in_vx, a.in_vy, a.in_vz, a.in_bx, a.in_by, a.in_bz, a.in_p};
        if (a.in_dev) {
#pragma unroll
            for (int k = 0; k < 8; ++k) in[k] = (T)a.in_dev[k];
        }
        T vn, v1, v2, Bn, B1, B2;
        to_pencil<AX>(in[1], in[2], in[3], vn, v1, v2);
        to_pencil<AX>(in[4], in[5], in[6], Bn, B1, B2);
        T pbn = Bn - bdn, pb1 = B1 - bd1, pb2 = B2 - bd2;
        Q[0] = in[0];
        Q[1] = in[0] * vn;
        Q[2] = in[0] * v1;
        Q[3] = in[0] * v2;
        Q[4] = pbn;
        Q[5] = pb1;
        Q[6] = pb2;
        Q[7] = in[7] / (gam - T(1)) + T(0.5) * in[0] * (vn * vn + v1 * v1 + v2 * v2) +
               T(0.5) * (pbn * pbn + pb1 * pb1 + pb2 * pb2);
    }
    const T rho = Q[0];
    const T irho = Ar<T>::rcp(rho);
    const T un = Q[1] * irho, v1 = Q[2] * irho, v2 = Q[3] * irho;
    const T bn = Q[4], b1 = Q[5], b2 = Q[6];
    const T bt2 = b1 * b1 + b2 * b2;
    T pth = (gam - T(1)) * (Q[7] - T(0.5) * ((Q[1] * un + Q[2] * v1 + Q[3] * v2) + (bn * bn + bt2)));
    const bool floored = pth < a.p_floor;
    if (floored) pth = a.p_floor;
    const T dm = rho * dxi;
    const T Pt = pth + bd1 * b1 + bd2 * b2 + T(0.5) * bt2;
    const T Pa = Pt + T(0.5) * (bd1 * bd1 + bd2 * bd2);
    const bool cnt_floor = interior && floored;
    const bool cnt_bad = interior && (!(rho > T(0)) || !__builtin_isfinite(rho) || !__builtin_isfinite(Q[7]));
    // primitive set used for reconstruction: rho, u, v1, v2, b1, b2, p
    const T W[7] = {rho, un, v1, v2, b1, b2, pth};
    if (keeps) {
#pragma unroll
        for (int k = 0; k < 7; ++k) sA[k * S + t] = W[k];
        sA[7 * S + t] = dm;
        sA[8 * S + t] = bn;
        sA[9 * S + t] = Pt;
        sA[10 * S + t] = Pa;
        sA[11 * S + t] = bfn;
        sA[12 * S + t] = bf1;
        sA[13 * S + t] = bf2;
    }
    if (leaves) {
        const int w = cslot(0);
#pragma unroll
        for (int k = 0; k < 7; ++k) sA[k * S + w] = W[k];
        sA[7 * S + w] = dm;
        sA[8 * S + w] = bn;
        sA[9 * S + w] = Pt;
        sA[10 * S + w] = Pa;
        sA[11 * S + w] = bfn;
        sA[12 * S + w] = bf1;
        sA[13 * S + w] = bf2;
    }
    if (MARCH && slot_ok && i == L - 2) sA[15 * S + cslot(0) + d] = Pt;
    __syncthreads();

    // ------------------------------------------------------------ R2
    const int sm1 = left(0);
    // P~ of the zone i-2 (row 9; carried in row 15)
    const int sm2 = !MARCH || ch == 0 || i > 1 ? t - 2 * d : (i == 1 ? t - d * (2 + (ch & 1)) : sm1 + 6 * S);
    const T dmm = sA[7 * S + sm1], dmp = sA[7 * S + sp1], dmp2 = sA[7 * S + sp2];
    const T bnm = sA[8 * S + sm1], bnp = sA[8 * S + sp1];
    const T bln = sA[11 * S + sm1], bl1 = sA[12 * S + sm1], bl2 = sA[13 * S + sm1];  // left face
    const T Ptm = sA[9 * S + sm1], Ptp = sA[9 * S + sp1];
    // Each zone limits its own slopes (CW84 Eq. 1.7-1.8) and hands them to
    // the zone on its left through buffer B; the right-edge value then needs
    // the neighbour's slope only.  The edges go to buffer A, slots 9..15
    // (the face values of R1 there have been read by then).
    T edgeR[7];
    T ftil = T(0);
    {
        const Weights<T> w(dmm, dm, dmp, dmp2);
        // (the edge without the right neighbour's slope waits in edgeR)
        T da0[7];
#pragma unroll
        for (int k = 0; k < 7; ++k) {
            const T dmv = W[k] - sA[k * S + sm1], dpv = sA[k * S + sp1] - W[k];
            da0[k] = limit_half(w.A * dpv + w.B * dmv, dmv, dpv);
            edgeR[k] = W[k] + w.E0 * dpv + w.E3 * da0[k];
        }
        if (a.flatten) {
            T Ptm2 = sA[9 * S + sm2], Ptp2 = sA[9 * S + sp2];
            T Pam = sA[10 * S + sm1], Pap = sA[10 * S + sp1];
            T um = sA[1 * S + sm1], up = sA[1 * S + sp1];
            T d1 = Ptp - Ptm, d2 = Ptp2 - Ptm2;
            // compression with a margin of kCompMin sound speeds
            // sqrt(P_min / rho), so that equal velocities (a pressure jump at
            // rest) and rounding noise about them never flatten
            const T pmin = tmin(Pap, Pam), du = um - up;
            if (tabs(d1) > T(0.33) * pmin && du > T(0) && du * du * rho > T(kCompMin * kCompMin) * pmin) {
                if (d2 != T(0)) ftil = tmax(T(0), tmin(T(1), T(10) * (Ar<T>::div(d1, d2) - T(0.75))));
                else ftil = T(1);
            }
        }
        if (keeps) {
#pragma unroll
            for (int k = 0; k < 7; ++k) sB[k * S + t] = da0[k];
            sB[7 * S + t] = ftil;
        }
        if (leaves) sB[7 * S + cslot(0)] = ftil;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 7; ++k) edgeR[k] -= w.E2 * sB[k * S + sp1];
    }
    if (keeps) {
#pragma unroll
        for (int k = 0; k < 7; ++k) sA[(9 + k) * S + t] = edgeR[k];
    }
    if (leaves) {
        const int w = cslot(1);
#pragma unroll
        for (int k = 0; k < 7; ++k) sA[(9 + k) * S + w] = edgeR[k];
    }
    __syncthreads();

    // ------------------------------------------------------------ R3
    T fl = T(0);
    if (a.flatten) {
        T fm = sB[7 * S + sm1], fp = sB[7 * S + sp1];
        fl = tmax(ftil, (Ptp - Ptm < T(0)) ? fp : fm);
    }
    // Flattening toward the zone average.  Few zones are near a shock, so a
    // wave without one skips it (x + 0 (a - x) = x).
    const bool flat = a.flatten && __any(fl != T(0));
    T edgeL[7];
    {
        const int e = left(1);
#pragma unroll
        for (int k = 0; k < 7; ++k) edgeL[k] = sA[(9 + k) * S + e];
    }
    if (flat) {
#pragma unroll
        for (int k = 0; k < 7; ++k) {
            edgeL[k] += fl * (W[k] - edgeL[k]);
            edgeR[k] += fl * (W[k] - edgeR[k]);
        }
    }
    Para<T> pc[7];
#pragma unroll
    for (int k = 1; k < 4; ++k) pc[k].set(W[k], edgeL[k], edgeR[k]);
    // tracing speeds (Lagrangian): normal pair C_n, Alfven pair C_A
    const T Bt1c = bd1 + b1, Bt2c = bd2 + b2, Bnc = bdn + bn;
    const T idm = Ar<T>::rcp(dm);
    const T tdm = dt * idm;
    const Frac<T> yn(tmin(T(1), Ar<T>::sqrtp(rho * (gam * pth + Bt1c * Bt1c + Bt2c * Bt2c)) * tdm));
    const Frac<T> yA(tmin(T(1), Ar<T>::sqrtp(rho) * tabs(Bnc) * tdm));
    // time-centring of the couplings left out of the two decoupled Riemann
    // problems: oblique-field terms and the variation of B_n along the pencil
    // (h*: half a step times the gradients d/dm; dB_d over the zone's faces,
    // dB'_n between the neighbours' centres)
    const T htm = T(0.5) * tdm;
    const T hbn = dt * (bnp - bnm) * Ar<T>::rcp(dmm + dmp + (dm + dm));
    const T hdn = htm * (bfn - bln), hd1 = htm * (bf1 - bl1), hd2 = htm * (bf2 - bl2);
    const T hBn = hdn + hbn;
    const T corrU = Bnc * hbn + bn * hdn;
    const T corrV1 = b1 * hBn + bd1 * hbn + bn * hd1;
    const T corrV2 = b2 * hBn + bd2 * hbn + bn * hd2;
    // (the oblique-field terms, in the gradients of u, v_t1 and v_t2, are in
    // the eigenvectors of the characteristic mode)
    const T e1 = v1 * hBn - un * hd1, e2 = v2 * hBn - un * hd2;
    const T hu = TRACE ? T(0) : htm * pc[1].D;
    const T corrB1 = rho * (e1 - Bt1c * hu);
    const T corrB2 = rho * (e2 - Bt2c * hu);
    const T hB = TRACE ? T(0) : htm * Bnc;
    const T corrP = rho * (Bt1c * (e1 + hB * pc[2].D) + Bt2c * (e2 + hB * pc[3].D));

    // Characteristic mode: the face states traced wave by wave.  The
    // reference is the zone's parabola averaged over the fast wave's domain
    // of dependence; the Alfven and slow waves moving into the face get their
    // own averages (difference projected on the left eigenvector, taken out
    // along the right one).  A traced state without positive density and
    // pressure falls back to the zone average.  The split multi-D terms are
    // added to u, v_t and B_t; the thermal pressure takes none (its
    // Lagrangian equation has no term in dB_n/dm: corrP is the magnetic-
    // pressure change B_t . corrB, which the corrected field carries into
    // the interface total pressure).  The right-face state stays in
    // registers, the left-face state goes to the zone on the left through
    // LDS (slots 0..6).
    T WLc[7];
    if constexpr (TRACE) {
        pc[0].set(W[0], edgeL[0], edgeR[0]);
#pragma unroll
        for (int k = 4; k < 7; ++k) pc[k].set(W[k], edgeL[k], edgeR[k]);
        Waves7<T> wz;
        wz.template init<Ar<T>>(rho, pth, gam, Bnc, Bt1c, Bt2c);
        const T sp = rho * tdm;
        const Frac<T> yf(tmin(T(1), wz.cf * sp)), ya(tmin(T(1), wz.ca * sp)), ys(tmin(T(1), wz.cs * sp));
        const T corr[7] = {T(0), corrU, corrV1, corrV2, corrB1, corrB2, T(0)};
        T WRc[7];
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            const T dir = side == 0 ? T(1) : T(-1);
            T ref[7], DA[7], DS[7];
#pragma unroll
            for (int k = 0; k < 7; ++k) {
                if (side == 0) {
                    ref[k] = pc[k].right(yf);
                    DA[k] = ref[k] - pc[k].right(ya);
                    DS[k] = ref[k] - pc[k].right(ys);
                } else {
                    ref[k] = pc[k].left(yf);
                    DA[k] = ref[k] - pc[k].left(ya);
                    DS[k] = ref[k] - pc[k].left(ys);
                }
            }
            T bfa, baa, bsa, bfs, bas, bss;
            wz.project(DA, dir, bfa, baa, bsa);
            wz.project(DS, dir, bfs, bas, bss);
            wz.add(ref, dir, T(0), wz.moves(wz.ca) ? -baa : T(0), wz.moves(wz.cs) ? -bss : T(0));
            const bool phys = ref[0] > T(0) && ref[6] > T(0);
            T *dst = side == 0 ? WLc : WRc;
#pragma unroll
            for (int k = 0; k < 7; ++k) dst[k] = (phys ? ref[k] : W[k]) + corr[k];
        }
        if (keeps) {
#pragma unroll
            for (int k = 0; k < 7; ++k) sA[k * S + t] = WRc[k];
        }
    }

    // interface states of this zone: L at its right face (i+1/2), R at its
    // left face (i-1/2); normal pair traced with y_n, Alfven pair with y_A.
    // The normal pair's state is (perturbation total pressure P~, u, 1 / C,
    // k / P): C = sqrt(rho (gamma p + B_t^2)) the Lagrangian sound speed, and
    // k = (ge + 1) / (2 ge) = 1/2 + rho P / (2 C^2) with ge = C^2 / (rho P).
    // The interface solve needs no other form of C, so one reciprocal square
    // root per side takes the place of a square root and two reciprocals.
    auto normal_state = [&](T r_, T u_, T p_, T q1, T q2, T g1, T g2, T Pd, T T1, T T2, T &Pt_, T &uu, T &iC, T &kP) {
        const T TT = T1 * T1 + T2 * T2;
        iC = Ar<T>::rsqrt(r_ * (gam * p_ + TT));
        // p + B_d . B' + B'^2 / 2 + the oblique term, at least half the
        // untraced total pressure
        Pt_ = (p_ + corrP) + q1 * (g1 + T(0.5) * q1) + q2 * (g2 + T(0.5) * q2);
        const T least = T(0.5) * (p_ + T(0.5) * TT) - Pd;
        if (Pt_ < least) Pt_ = least;
        kP = T(0.5) * (Ar<T>::rcp(Pt_ + Pd) + r_ * (iC * iC));
        uu = u_ + corrU;
    };
    const T PdR = T(0.5) * (bf1 * bf1 + bf2 * bf2);
    // The right-face (L) state is kept in registers, the left-face (R) state
    // goes to the zone on the left through LDS, variable by variable (few
    // parabolas are then live at a time).
    T LPt, Lu, LiC, LkP, Lr, Lv1, Lv2, Lb1, Lb2;
    T LrN, LT1, LT2;      // normal-pair density and total transverse field (guess features)
    if constexpr (!TRACE) {
        if (keeps) {
            sA[5 * S + t] = pc[2].left(yA) + corrV1;
            sA[6 * S + t] = pc[3].left(yA) + corrV2;
        }
        Lv1 = pc[2].right(yA) + corrV1;
        Lv2 = pc[3].right(yA) + corrV2;
        pc[4].set(W[4], edgeL[4], edgeR[4]);
        if (keeps) sA[7 * S + t] = pc[4].left(yA) + corrB1;
        Lb1 = pc[4].right(yA) + corrB1;
        const T q1l = pc[4].left(yn), q1r = pc[4].right(yn);
        pc[5].set(W[5], edgeL[5], edgeR[5]);
        if (keeps) sA[8 * S + t] = pc[5].left(yA) + corrB2;
        Lb2 = pc[5].right(yA) + corrB2;
        const T q2l = pc[5].left(yn), q2r = pc[5].right(yn);
        pc[0].set(W[0], edgeL[0], edgeR[0]);
        if (keeps) sA[4 * S + t] = Ar<T>::sqrtp(pc[0].left(yA));
        Lr = Ar<T>::sqrtp(pc[0].right(yA));
        const T rl = pc[0].left(yn);
        LrN = pc[0].right(yn);
        pc[6].set(W[6], edgeL[6], edgeR[6]);
        const T T1 = bl1 + q1l, T2 = bl2 + q2l;
        T Pt_, u_, iC, kP;
        normal_state(rl, pc[1].left(yn), pc[6].left(yn), q1l, q2l, bl1, bl2, T(0.5) * (bl1 * bl1 + bl2 * bl2), T1, T2,
                     Pt_, u_, iC, kP);
        if (keeps) {
            sA[0 * S + t] = Pt_;
            sA[1 * S + t] = u_;
            sA[2 * S + t] = iC;
            sA[3 * S + t] = kP;
            if (GUESS != kGuessPlain) {
                sA[16 * S + t] = rl;
                sA[17 * S + t] = T1;
                sA[18 * S + t] = T2;
            }
        }
        LT1 = bf1 + q1r;
        LT2 = bf2 + q2r;
        normal_state(LrN, pc[1].right(yn), pc[6].right(yn), q1r, q2r, bf1, bf2, PdR, LT1, LT2, LPt, Lu, LiC, LkP);
    }
    __syncthreads();

    // ------------------------------------------------------------ R4
    // face i+1/2 between this zone (L) and zone i+1 (R)
    // Learned guess: faces with a strong jump are compacted per workgroup and run
    // through the network 16 at a time on the matrix cores, the waves taking
    // tiles of 16 in turn (tiles of 64 left three of four waves waiting at the
    // barrier where a workgroup has a few such faces).  The list is in rows 9..15 of
    // buffer A (the edges, read in R3), seven words of two features each in
    // lane order, so that there is a place for every lane; the network's answer
    // takes row 9.  256x192x192 dipole, gates 0.1, one sweep, x / y / z: 997 /
    // 544 / 586 us as whole-pencil tiles with the list in buffer B, tiles of 64
    // and the features formed by every wave; 431 / 356 / 359 us as marches.
    // This pass comes before the solver's right states are
    // loaded, so that they do not occupy registers next to the network's; they
    // are read again from LDS below.
    bool lg_gate = false;                    // selected
    T lg_y = T(0), lg_Pbar = T(1);
    if constexpr (GUESS == kGuessLearned) {
        const int lane = tid & 63;
        unsigned int *F = reinterpret_cast<unsigned int *>(sA + 9 * S);
        auto column = [&](int n) -> int {                 // lane n's slot
            return MARCH ? march_slot(AX == 0, n, (int)(((float)n + 0.5f) * a.inv_div), P) : n;
        };
        int slot = 0;
        // (few waves have such a face: the others do not form the features)
        const T PL = LPt + PdR;
        lg_gate = face_ok && guess_selects(LrN, sA[16 * S + sp1], Lu, sA[1 * S + sp1], PL, sA[0 * S + sp1] + PdR,
                                           a.gate_p, a.gate_u);
        const unsigned long long bal = __ballot(lg_gate);
        if (bal) {
            int base = 0;
            if (lane == 0) base = (int)atomicAdd(&s_guess[0], (unsigned int)__popcll(bal));
            base = __shfl(base, 0);
            slot = column(lg_gate ? base + __popcll(bal & ((1ull << lane) - 1ull)) : 0);
            if (lg_gate) {
                const T Ls[7] = {LrN, Lu, Lv1, Lv2, LT1, LT2, PL};
                const T Rs[7] = {sA[16 * S + sp1], sA[1 * S + sp1],  sA[5 * S + sp1],      sA[6 * S + sp1],
                                 sA[17 * S + sp1], sA[18 * S + sp1], sA[0 * S + sp1] + PdR};
                T feat[14], cbar_;
                guess_features(Ls, Rs, feat, lg_Pbar, cbar_);
#pragma unroll
                for (int k = 0; k < 7; ++k) F[k * S + slot] = mlp::pack2(feat[2 * k], feat[2 * k + 1]);
            }
        }
        if (STATS) wave_add(&s_stat[35], lg_gate && g >= own_lo && g < gend);
        __syncthreads();
        const int nf = (int)s_guess[0], nw = (int)(blockDim.x >> 6);
#pragma unroll 1
        for (int b0 = (tid >> 6) * 16; b0 < nf; b0 += nw * 16) {
            // sample b0 + lane mod 16; features 4 (lane / 16) .. + 3
            const int n = b0 + (lane & 15), kq = lane >> 4;
            const int col = column(min(n, Suse - 1));
            const unsigned int f0 = F[2 * kq * S + col], f1 = kq < 3 ? F[(2 * kq + 1) * S + col] : 0u;
            const float y = mlp::forward_tile(f0, f1, a.mlp_frag, a.mlp_theta);
            if (kq == 0 && n < nf) sA[9 * S + col] = (T)y;
        }
        __syncthreads();
        if (lg_gate) lg_y = sA[9 * S + slot];
    }
    T Pst, ust, v1s, b1s, v2s, b2s;
    const T bns = T(0.5) * (bn + bnp);
    const T Bns = bfn + bns;
    if constexpr (TRACE) {
        // characteristic mode: the interface problem in its linearisation about
        // the mean of the two traced states; the face state is the left state
        // plus the waves of negative Lagrangian speed
        T WRc[7];
#pragma unroll
        for (int k = 0; k < 7; ++k) WRc[k] = face_ok ? sA[k * S + sp1] : WLc[k];
        Waves7<T> wf;
        wf.template init<Ar<T>>(T(0.5) * (WLc[0] + WRc[0]), T(0.5) * (WLc[6] + WRc[6]), gam, Bns,
                                bf1 + T(0.5) * (WLc[4] + WRc[4]), bf2 + T(0.5) * (WLc[5] + WRc[5]));
        T D[7];
#pragma unroll
        for (int k = 0; k < 7; ++k) D[k] = WRc[k] - WLc[k];
        T cfw, caw, csw;
        wf.project(D, T(-1), cfw, caw, csw);
        T Ws[7];
#pragma unroll
        for (int k = 0; k < 7; ++k) Ws[k] = WLc[k];
        wf.add(Ws, T(-1), wf.cf > T(0) ? cfw : T(0), wf.moves(wf.ca) ? caw : T(0), wf.moves(wf.cs) ? csw : T(0));
        ust = Ws[1];
        v1s = Ws[2];
        v2s = Ws[3];
        b1s = Ws[4];
        b2s = Ws[5];
        Pst = Ws[6] + bf1 * b1s + bf2 * b2s + T(0.5) * (b1s * b1s + b2s * b2s);
        if (STATS) {
            const bool counted = face_ok && g >= own_lo && g < gend;
            wave_add(&s_stat[0], counted);          // no iteration
            wave_add(&s_stat[32], cnt_floor);
            wave_add(&s_stat[34], cnt_bad);
        }
    } else {
    const T Rr = sA[4 * S + sp1], Rv1 = sA[5 * S + sp1], Rv2 = sA[6 * S + sp1];
    const T Rb1 = sA[7 * S + sp1], Rb2 = sA[8 * S + sp1];
    {
        const T RPt = sA[0 * S + sp1], Ru = sA[1 * S + sp1], RiC = sA[2 * S + sp1], RkP = sA[3 * S + sp1];
        const T Pd = PdR;
        const T Pfloor = T(1e-6) * (tmin(LPt, RPt) + Pd) - Pd;
        const T tol = a.tol;
        // The velocity mismatch u*_R - u*_L is formed from differences
        // ((u_R - u_L) + jumps / W) rather than as the difference of the two
        // star velocities, so that a large bulk velocity does not bury it in
        // rounding (same quantity; matters in single precision at high Mach).
        const T duRL = Ru - Lu;
        // linear guess P_L + C_L (P_R - P_L - C_R (u_R - u_L)) / (C_L + C_R)
        T P = LPt + ((RPt - LPt) * RiC - duRL) * Ar<T>::rcp(LiC + RiC);
        P = tmax(P, Pfloor);
        const T P0 = P;
        // Faces with a strong jump are selected for the learned guess.  Its
        // 14 inputs: both sides' (rho, u, v_t1, v_t2, B_t1, B_t2, P) of the
        // normal-pair problem, normalised by the pair means (velocities
        // relative to the mean, scaled by c = sqrt(P/rho); fields by
        // sqrt(P)).  Outputs: (P* - P0) / P and (u* - u0) / c.
        bool gate = false;
        T feat[14], Pbar = T(1), cbar = T(1);
        if (GUESS == kGuessHarvest) {
            const T Ls[7] = {LrN, Lu, Lv1, Lv2, LT1, LT2, LPt + Pd};
            const T Rs[7] = {sA[16 * S + sp1], Ru, Rv1, Rv2, sA[17 * S + sp1], sA[18 * S + sp1], RPt + Pd};
            guess_features(Ls, Rs, feat, Pbar, cbar);
            gate = face_ok && g >= own_lo && g < gend &&
                   guess_selects(Ls[0], Rs[0], Ls[1], Rs[1], Ls[6], Rs[6], a.gate_p, a.gate_u);
            if (STATS) wave_add(&s_stat[35], gate);
        }
        if (GUESS == kGuessLearned) {
            bool used = false;
            if (lg_gate) {
                const T Pg = P + lg_Pbar * lg_y;
                if (__builtin_isfinite(Pg) && Pg > Pfloor) {
                    P = Pg;
                    used = true;
                }
            }
            if (STATS) wave_add(&s_stat[36], lg_gate && !used && g >= own_lo && g < gend);
        }
        int it = 0;
        bool conv = true;
        // Shock impedances W_s = C_s sqrt(q_s), q_s = 1 + k_s (P - P_s) / P_s,
        // and Z_s = 2 W_s^3 / (W_s^2 + C_s^2), carried as s = 1/sqrt(q_s) and
        // g = 2/Z_s = (s + s^3) / C_s: two reciprocal square roots and one
        // reciprocal per iteration.  Then dP = -mis Z_L Z_R / (Z_L + Z_R) =
        // -2 mis / (g_L + g_R).
        T jL, gL, ig, dP, mis;
        for (;;) {
            const T aL = P - LPt, aR = P - RPt;
            const T sL = Ar<T>::rsqrt(T(1) + LkP * aL), sR = Ar<T>::rsqrt(T(1) + RkP * aR);
            const T wL = sL * LiC, wR = sR * RiC;
            jL = aL * wL;
            mis = (duRL + aR * wR) + jL;
            gL = wL + (sL * sL) * wL;
            ig = Ar<T>::rcp(gL + (wR + (sR * sR) * wR));
            dP = T(-2) * mis * ig;
            if (!face_ok || tabs(dP) <= tol * (P + Pd)) break;   // (faces in the ghosts do not iterate)
            if (it >= a.max_iter) { conv = false; break; }
            P = tmax(P + dP, Pfloor);
            ++it;
        }
        Pst = tmax(P + dP, Pfloor);
        ust = (Lu - jL) + mis * gL * ig;
        if constexpr (GUESS == kGuessHarvest) {
            // record the selected faces: inputs, targets and the solver's own
            // scalars (for checks against an independent solver)
            const int lane = tid & 63;
            const unsigned long long bal = __ballot(gate);
            if (bal && a.harvest) {
                unsigned long long base = 0;
                if (lane == 0) base = atomicAdd(a.harvest_count, (unsigned long long)__popcll(bal));
                base = __shfl(base, 0);
                const unsigned long long slot = base + (unsigned long long)__popcll(bal & ((1ull << lane) - 1ull));
                if (gate && slot < (unsigned long long)a.harvest_cap) {
                    float *rec = a.harvest + slot * mlp::kRecord;
                    const T LC = Ar<T>::rcp(LiC), RC = Ar<T>::rcp(RiC);
                    const T u0 = (LC * Lu + RC * Ru - (RPt - LPt)) * Ar<T>::rcp(LC + RC);
#pragma unroll
                    for (int k = 0; k < 14; ++k) rec[k] = (float)feat[k];
                    rec[14] = (float)((Pst - P0) * Ar<T>::rcp(Pbar));
                    rec[15] = (float)((ust - u0) * Ar<T>::rcp(cbar));
                    rec[16] = (float)LPt; rec[17] = (float)RPt; rec[18] = (float)Pd;
                    rec[19] = (float)Lu;  rec[20] = (float)Ru;
                    rec[21] = (float)LC;  rec[22] = (float)RC;
                    rec[23] = (float)(LkP * (LPt + Pd));  rec[24] = (float)(RkP * (RPt + Pd));
                    rec[25] = (float)P0;  rec[26] = (float)Pst; rec[27] = (float)ust;
                }
            }
        }
        if (STATS) {
            // owned faces: iteration histogram and non-converged count; zone
            // counters of R1 (after the first barrier)
            const bool counted = face_ok && g >= own_lo && g < gend;
            wave_hist(s_stat, counted, it < 31 ? it : 31);
            wave_add(&s_stat[33], counted && !conv);
            wave_add(&s_stat[32], cnt_floor);
            wave_add(&s_stat[34], cnt_bad);
        }
    }
    // transverse pair: linear Alfven problem, increment form from the left
    const T sig = tsgn(Bns);
    const T irs = Ar<T>::rcp(Lr + Rr);
    const T wR = Rr * irs, wL = Lr * irs, ws = sig * irs, wx = sig * Lr * wR;
    v1s = Lv1 + wR * (Rv1 - Lv1) + ws * (Rb1 - Lb1);
    b1s = Lb1 + wL * (Rb1 - Lb1) + wx * (Rv1 - Lv1);
    v2s = Lv2 + wR * (Rv2 - Lv2) + ws * (Rb2 - Lb2);
    b2s = Lb2 + wL * (Rb2 - Lb2) + wx * (Rv2 - Lv2);
    }
    // Lagrangian fluxes in dipole + deviation flux form
    const T nn = bns * (bfn + T(0.5) * bns);
    const T Fpi = Pst - nn;
    const T Fv1 = -(Bns * b1s + bns * bf1);
    const T Fv2 = -(Bns * b2s + bns * bf2);
    const T Fb1 = ust * bf1 - Bns * v1s;
    const T Fb2 = ust * bf2 - Bns * v2s;
    const T Fe = ust * (Pst + nn) - Bns * (ust * bns + v1s * b1s + v2s * b2s);
    const T delR = ust * dt;
    if (keeps) {
        sB[0 * S + t] = Fpi;
        sB[1 * S + t] = Fv1;
        sB[2 * S + t] = Fv2;
        sB[3 * S + t] = Fb1;
        sB[4 * S + t] = Fb2;
        sB[5 * S + t] = Fe;
        sB[6 * S + t] = delR;
    }
    if (leaves) {
        const int w = cslot(0);
        sB[0 * S + w] = Fpi;
        sB[1 * S + w] = Fv1;
        sB[2 * S + w] = Fv2;
        sB[3 * S + w] = Fb1;
        sB[4 * S + w] = Fb2;
        sB[5 * S + w] = Fe;
        sB[6 * S + w] = delR;
    }
    __syncthreads();

    // ------------------------------------------------------------ R5
    // Lagrangian update of the zone contents (faces i-1/2, i+1/2)
    const int fm1 = left(0);
    const T delL = sB[6 * S + fm1];
    T dC[7];
    dC[0] = T(0);
    dC[1] = -dt * (Fpi - sB[0 * S + fm1]);
    dC[2] = -dt * (Fv1 - sB[1 * S + fm1]);
    dC[3] = -dt * (Fv2 - sB[2 * S + fm1]);
    dC[4] = -dt * (Fb1 - sB[3 * S + fm1]);
    dC[5] = -dt * (Fb2 - sB[4 * S + fm1]);
    dC[6] = -dt * (Fe - sB[5 * S + fm1]);
    // remapped quantities per volume: rho, mn, m1, m2, b1, b2, E
    const T Qr[7] = {Q[0], Q[1], Q[2], Q[3], Q[5], Q[6], Q[7]};
    const T dd = delR - delL;
    const T dVL = dxi + dd;
    const T idVL = Ar<T>::rcp(dVL);
    T QL[7];
#pragma unroll
    for (int k = 0; k < 7; ++k) QL[k] = Qr[k] + (dC[k] - Qr[k] * dd) * idVL;
    if (keeps) {
#pragma unroll
        for (int k = 0; k < 7; ++k) sA[k * S + t] = QL[k];
        sA[7 * S + t] = dVL;
    }
    if (leaves) {
        const int w = cslot(1);
#pragma unroll
        for (int k = 0; k < 7; ++k) sA[k * S + w] = QL[k];
        sA[7 * S + w] = dVL;
    }
    __syncthreads();

    // ------------------------------------------------------------ R6
    // slopes shared through buffer B as in R2; edges to buffer A, slots 8..14
    T redgeR[7];
    {
        const int qm1 = left(1);
        const T vm = sA[7 * S + qm1], vp = sA[7 * S + sp1], vp2 = sA[7 * S + sp2];
        const Weights<T> w(vm, dVL, vp, vp2);
        T da0[7];
#pragma unroll
        for (int k = 0; k < 7; ++k) {
            const T dmv = QL[k] - sA[k * S + qm1], dpv = sA[k * S + sp1] - QL[k];
            da0[k] = limit_half(w.A * dpv + w.B * dmv, dmv, dpv);
            redgeR[k] = QL[k] + w.E0 * dpv + w.E3 * da0[k];
        }
        if (keeps) {
#pragma unroll
            for (int k = 0; k < 7; ++k) sB[k * S + t] = da0[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 7; ++k) redgeR[k] -= w.E2 * sB[k * S + sp1];
    }
    if (keeps) {
#pragma unroll
        for (int k = 0; k < 7; ++k) sA[(8 + k) * S + t] = redgeR[k];
    }
    if (leaves) {
        const int w = cslot(2);
#pragma unroll
        for (int k = 0; k < 7; ++k) sA[(8 + k) * S + w] = redgeR[k];
    }
    __syncthreads();

    // ------------------------------------------------------------ R7
    // donor-cell remap fluxes: this zone gives its right part across face
    // i+1/2 when delta > 0 and its left part across i-1/2 when delta < 0
    {
        const bool zone_ok = pen && i >= (first ? 6 : 0) && i <= M - 7;
        const bool wr = zone_ok && delR >= T(0);
        const bool wl = zone_ok && delL < T(0) && i >= 1;
        // (two registers a variable are held over the two directions, of which
        // most waves take one: left and right edge)
        T eL[7], eR[7];
        {
            T aL[7];
            const int e = left(2);
#pragma unroll
            for (int k = 0; k < 7; ++k) aL[k] = sA[(8 + k) * S + e];
            if (flat) {
#pragma unroll
                for (int k = 0; k < 7; ++k) {
                    aL[k] += fl * (QL[k] - aL[k]);
                    redgeR[k] += fl * (QL[k] - redgeR[k]);
                }
            }
#pragma unroll
            for (int k = 0; k < 7; ++k) {
                Para<T> rc;
                rc.set(QL[k], aL[k], redgeR[k]);
                eL[k] = rc.L;
                eR[k] = rc.R;
            }
        }
        if (wr) {
            const Frac<T> yR(delR * idVL);
#pragma unroll
            for (int k = 0; k < 7; ++k) {
                Para<T> rc;
                rc.edges(QL[k], eL[k], eR[k]);
                sB[k * S + t] = delR * rc.right(yR);
            }
        }
        if (wl) {
            const Frac<T> yL(-delL * idVL);
#pragma unroll
            for (int k = 0; k < 7; ++k) {
                Para<T> rc;
                rc.edges(QL[k], eL[k], eR[k]);
                sB[k * S + t - d] = delL * rc.left(yL);
            }
        }
    }
    // what the update reads from tables, requested ahead of the barrier
    const int gc = g < 0 ? 0 : (g < N ? g : N - 1);
    const T idx = load(a.rdx, gc), idc = load(a.rdc, gc);
    const T iwq = FUSE_CFL ? load(a.rdx_q, qq) : T(0), iwr = FUSE_CFL ? load(a.rdx_r, r) : T(0);
    __syncthreads();

    // ------------------------------------------------------------ R8
    T fr[7];
#pragma unroll
    for (int k = 0; k < 7; ++k) fr[k] = sB[k * S + t];
    if (leaves) {
        const int w = cslot(1);
#pragma unroll
        for (int k = 0; k < 7; ++k) sB[k * S + w] = fr[k];
    }
    if (interior) {
        const int rm1 = left(1);
        T out[8];
        T nw[7];
#pragma unroll
        for (int k = 0; k < 7; ++k) nw[k] = Qr[k] + (dC[k] + sB[k * S + rm1] - fr[k]) * idx;
        T nbn = bn, nb1 = nw[4], nb2 = nw[5];
        if (a.janhunen) {
            // -v div B' source, split: n-derivative of B'_n, pre-sweep velocity
            const T divn = dt * ((bnp - bnm) * idc);
            nbn -= un * divn;
            nb1 -= v1 * divn;
            nb2 -= v2 * divn;
        }
        out[0] = nw[0];
        out[1 + kn] = nw[1];
        out[1 + k1] = nw[2];
        out[1 + k2] = nw[3];
        out[4 + kn] = nbn;
        out[4 + k1] = nb1;
        out[4 + k2] = nb2;
        out[7] = nw[6];
        bool masked = false;
        if (a.has_inner) {
            T x, y, z;
            to_xyz<AX>(xci, c1, c2, x, y, z);
            if (x * x + y * y + z * z < a.r_inner2) {
                masked = true;
                // the inner state: rest, or the drift the ionosphere coupling set
                T vx = T(0), vy = T(0), vz = T(0);
                if (a.inner_v) {
                    int ix, iy, iz;
                    if (AX == 0) { ix = g; iy = j1; iz = j2; }
                    else if (AX == 1) { iy = g; iz = j1; ix = j2; }
                    else { iz = g; ix = j1; iy = j2; }
                    if (ix >= a.ib[0] && ix < a.ib[1] && iy >= a.ib[2] && iy < a.ib[3] && iz >= a.ib[4] &&
                        iz < a.ib[5]) {
                        const long long bi = a.ib[1] - a.ib[0], bj = a.ib[3] - a.ib[2];
                        const long long nb = bi * bj * (a.ib[5] - a.ib[4]);
                        const long long o = ((long long)(iz - a.ib[4]) * bj + (iy - a.ib[2])) * bi + (ix - a.ib[0]);
                        vx = (T)a.inner_v[o];
                        vy = (T)a.inner_v[nb + o];
                        vz = (T)a.inner_v[2 * nb + o];
                    }
                }
                out[0] = a.inner_rho;
                out[1] = a.inner_rho * vx;
                out[2] = a.inner_rho * vy;
                out[3] = a.inner_rho * vz;
                out[4] = out[5] = out[6] = T(0);
                out[7] = a.inner_E + T(0.5) * a.inner_rho * (vx * vx + vy * vy + vz * vz);
            }
        }
        const unsigned int o = base + (unsigned int)(g * (int)a.stride_n);
#pragma unroll
        for (int v = 0; v < 8; ++v) store(a.var[v], o, out[v]);
        if (FUSE_CFL && cfl_max && !masked) {
            // signal speed of the updated zone, for the next step's dt (the
            // maximum is reduced in FP64)
            const T r_ = out[0];
            const T ir = Ar<T>::rcp(r_);
            const T vn = nw[1] * ir, w1 = nw[2] * ir, w2 = nw[3] * ir;
            T p_ = (gam - T(1)) * (nw[6] - T(0.5) * ((nw[1] * vn + nw[2] * w1 + nw[3] * w2) +
                                                     (nbn * nbn + nb1 * nb1 + nb2 * nb2)));
            // fmax / fabs where they agree with the selects for every input
            // (a NaN p or discriminant gives the floor / zero either way);
            // the running maximum keeps its select, which passes a NaN on
            p_ = fmax_(p_, a.p_floor);
            // total field in the pencil frame (the background of R1)
            const T Bn = nbn + bdn, B1 = nb1 + bd1, B2 = nb2 + bd2;
            const T a2 = gam * p_ * ir;
            const T b2 = (Bn * Bn + B1 * B1 + B2 * B2) * ir;
            const T s2 = a2 + b2;
            const T q4 = T(4) * a2 * ir;
            // q is t1 for the x and z sweeps, t2 for the y sweep
            const T i1 = AX == 1 ? iwr : iwq, i2 = AX == 1 ? iwq : iwr;
            T sp = T(0);
            {
                T disc = fmax_(s2 * s2 - q4 * Bn * Bn, T(0));
                T cf = Ar<T>::sqrtp(T(0.5) * (s2 + Ar<T>::sqrt_(disc)));
                sp = tmax(sp, (fabs_(vn) + cf) * idx);
            }
            {
                T disc = fmax_(s2 * s2 - q4 * B1 * B1, T(0));
                T cf = Ar<T>::sqrtp(T(0.5) * (s2 + Ar<T>::sqrt_(disc)));
                sp = tmax(sp, (fabs_(w1) + cf) * i1);
            }
            {
                T disc = fmax_(s2 * s2 - q4 * B2 * B2, T(0));
                T cf = Ar<T>::sqrtp(T(0.5) * (s2 + Ar<T>::sqrt_(disc)));
                sp = tmax(sp, (fabs_(w2) + cf) * i2);
            }
            smax = smax > sp ? smax : sp;
        }
    }
    }
    if (STATS) {
        __syncthreads();
        const int w = threadIdx.x;
        if (w < kStatWords && s_stat[w] != 0u && args.stats)
            atomicAdd(&args.stats[stat_slot * kStatWords + w], (unsigned long long)s_stat[w]);
    }
    if (FUSE_CFL && cfl_max) {
        // wave max (all lanes active), workgroup max, one atomic per workgroup
        // (no target: a sweep that is not the last of its step in a launch
        // that runs several)
        for (int off = 32; off > 0; off >>= 1) {
            T o = __shfl_xor(smax, off);
            smax = o > smax ? o : smax;
        }
        if (__lane_id() == 0) s_red[threadIdx.x >> 6] = (double)smax;
        __syncthreads();
        if (threadIdx.x == 0) {
            double m = 0.0;
            const int nw = (blockDim.x + 63) >> 6;
            for (int w = 0; w < nw; ++w) m = s_red[w] > m ? s_red[w] : m;
            atomicMax(cfl_max, (unsigned long long)__double_as_longlong(m));
        }
    }
}

// Waves per SIMD that the register allocation of a sweep is held to: 6 (80
// registers) where the LDS of its workgroups (up to 512 lanes, or 768) admits
// them.  A wave's stages wait on LDS, barriers and loads more than half of
// their time, so resident waves decide: the ensemble sweep with 82 registers
// (two workgroups of 512 per CU instead of three) took 59.1 ms against 45.5 ms
// for four steps of 32 members.  A march's workgroups of 256 lanes leave room
// for 5 waves per SIMD in FP32 (88 registers, 95 in the fused form) and for 3
// in FP64 (168).
template <typename T>
constexpr int sweep_waves(int SM, int GUESS, bool TRACE, bool MARCH = false)
{
    if (GUESS == kGuessLearned) return 4;
    if (MARCH) return sizeof(T) == 4 ? (TRACE ? 4 : 5) : (TRACE ? 2 : 3);
    return sizeof(T) == 4 && GUESS == kGuessPlain && !TRACE && ((SM > 0 && SM <= 512) || SM == 768) ? 6 : 1;
}

// Maximum of the signal-speed slots (one wave, lane = slot; the bits of
// non-negative doubles order as unsigned integers, as for the atomics that
// filled them).
__device__ inline unsigned long long slot_max(const unsigned long long *slots, int lane)
{
    unsigned long long v = slots[lane * kCflStride];
    for (int off = 32; off > 0; off >>= 1) {
        unsigned long long o = __shfl_xor(v, off);
        v = o > v ? o : v;
    }
    return v;
}

// A value that all lanes hold, as a scalar.
__device__ inline float uniform(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
__device__ inline double uniform(double v)
{
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                            __builtin_amdgcn_readfirstlane(__double2loint(v)));
}

// Standalone sweep: one workgroup per tile.  The learned-guess form holds
// the network pass next to the sweep's registers; a budget of 4 waves per SIMD
// (128 registers, up to 15 values spilled in the fused march) was ~20 % faster
// than 132 registers and 3 waves.
template <int AX, typename T, bool STATS, bool FUSE_CFL, int SM, int GUESS = kGuessPlain, bool TRACE = false,
          bool MARCH = false>
__global__ void __launch_bounds__(SM > 0 ? SM : 1024)
    __attribute__((amdgpu_waves_per_eu(sweep_waves<T>(SM, GUESS, TRACE, MARCH)))) sweep_kernel(const SweepArgs<T> a)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    double *s_red = reinterpret_cast<double *>(smem_raw);
    unsigned int *s_stat = reinterpret_cast<unsigned int *>(smem_raw + 16 * sizeof(double));
    unsigned int *s_guess = s_stat + kStatWords;
    // XCD-aware tile order: consecutive workgroups go to different XCDs
    // round-robin, so workgroups b, b+8, b+16, ... (one XCD) take consecutive
    // tiles (q fastest, then r) and share L2 lines of neighbouring pencils.
    // The segments of a pencil group are either consecutive in this order
    // (seg_fast) or the grid is dealt out one segment band after another.
    const int b = blockIdx.x;
    const int slot = (b & 7) * a.tiles_per_xcd + (b >> 3);
    if (slot >= a.nslots * a.nseg) return;
    int seg, tile;
    if (a.seg_fast) { seg = slot % a.nseg; tile = slot / a.nseg; }
    else { seg = slot / a.nslots; tile = slot - seg * a.nslots; }
    const int r = tile / a.tiles_q;
    const int tq = tile - r * a.tiles_q;
    T dt;
    if (a.t_out) {
        double d = a.step;
        if (a.dt_slots) {
            // every wave on its own (all its lanes are active here)
            const double m = __longlong_as_double((long long)slot_max(a.dt_slots, (int)__lane_id()));
            d = m > 0.0 ? a.step / m : 0.0;
            if (b == 0 && threadIdx.x == 0) *a.dt_out = d;
        }
        if (b == 0 && threadIdx.x == 0) *a.t_out += d;
        dt = uniform(T(d));
    } else {
        dt = a.dt_dev ? T(*a.dt_dev) : a.dt;
    }
    if (a.clear_slots && b == 0 && threadIdx.x < kCflSlots) a.clear_slots[threadIdx.x * kCflStride] = 0ull;
    unsigned long long *cm = a.cfl_max ? a.cfl_max + (b % kCflSlots) * kCflStride : nullptr;
    if constexpr (MARCH) {
        // the arguments where the launch put them (the first bytes of the
        // kernel's argument segment), so that each chunk reads them from there
        typedef const __attribute__((address_space(4))) SweepArgs<T> kernarg_t;
        const kernarg_t &ka = *(kernarg_t *)__builtin_amdgcn_kernarg_segment_ptr();
        sweep_tile<AX, T, STATS, FUSE_CFL, SM, GUESS, TRACE, true>(ka, tq, r, seg, dt, cm, b % kStatSlots, smem_raw,
                                                                   s_red, s_stat, s_guess);
    } else {
        sweep_tile<AX, T, STATS, FUSE_CFL, SM, GUESS, TRACE>(a, tq, r, seg, dt, cm, b % kStatSlots, smem_raw, s_red,
                                                             s_stat, s_guess);
    }
}

// ---------------------------------------------------------------------------
// Batched ensemble sweep: one launch performs the same sweep (one axis) of
// every member of an ensemble of independent runs (different sizes, inflows
// and dt).  Every member's tiles are dealt out to the eight XCDs in equal
// shares of adjacent tiles, and an XCD takes the members one after the other:
// members' tiles differ in their work (a march of one chunk, or of six), so an
// even share of all tiles is not one of the work.  Each member's geometry, dt
// pointer, signal-speed slot and counters are in its own descriptor, so a
// member's arithmetic is exactly that of a single-run sweep with the same
// tiles (and segments: a segmented member reads one state and writes the
// other, as a single run does).  Successive sweeps are ordered by the launch boundaries: no
// workgroup waits on another.
template <typename T>
struct EnsembleSweepArgs {
    const SweepArgs<T> *desc;      // [members]: this axis's descriptor of each member
    const int *mo;                 // [members + 1]: first tile of each member in an XCD's share
    int members, per_xcd;          // per_xcd = mo[members]
};

// The largest m below members with mo[m] <= j (mo ascends from mo[0] = 0): 64
// members per load, one per lane, where a bisection would wait for as many
// loads as it takes steps.  All lanes of the wave must be active.
__device__ inline int member_of(const int *mo, int members, int j)
{
    const int lane = threadIdx.x & 63;
    int m = -1;
    for (int i = 0; i < members; i += 64) {
        const int k = min(i + lane, members - 1);
        m += __popcll(__ballot(i + lane < members && mo[k] <= j));
    }
    return m;
}

template <int AX, typename T, bool STATS, bool FUSE_CFL, int SM, bool MARCH = false>
__global__ void __launch_bounds__(SM) __attribute__((amdgpu_waves_per_eu(sweep_waves<T>(SM, kGuessPlain, false, MARCH))))
    ensemble_sweep_kernel(const EnsembleSweepArgs<T> e)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int b = blockIdx.x;
    const int j = b >> 3;
    const int lo = member_of(e.mo, e.members, j);
    const SweepArgs<T> &a = e.desc[lo];
    double *s_red = reinterpret_cast<double *>(smem_raw);
    unsigned int *s_stat = reinterpret_cast<unsigned int *>(smem_raw + 16 * sizeof(double));
    const int share = e.mo[lo + 1] - e.mo[lo];
    const int t = (b & 7) * share + (j - e.mo[lo]);
    if (t >= a.ntiles * a.nseg) return;
    int seg, tt;                                  // as in the single-run order
    if (a.seg_fast) { seg = t % a.nseg; tt = t / a.nseg; }
    else { seg = t / a.ntiles; tt = t - seg * a.ntiles; }
    const int tq = tt % a.tiles_q;
    const int r = tt / a.tiles_q;
    const T dt = a.dt_dev ? T(*a.dt_dev) : a.dt;
    unsigned long long *cm = a.cfl_max ? a.cfl_max + (b % kCflSlots) * kCflStride : nullptr;
    if constexpr (MARCH) {
        // (the descriptor as constant memory: each chunk reads it again, by
        // scalar loads)
        typedef const __attribute__((address_space(4))) SweepArgs<T> desc_t;
        const desc_t &da = *(desc_t *)&a;
        sweep_tile<AX, T, STATS, FUSE_CFL, SM, kGuessPlain, false, true>(da, tq, r, seg, dt, cm, b % kStatSlots, smem_raw,
                                                                         s_red, s_stat);
    } else {
        sweep_tile<AX, T, STATS, FUSE_CFL, SM>(a, tq, r, seg, dt, cm, b % kStatSlots, smem_raw, s_red, s_stat);
    }
}

}  // namespace ppmlr
