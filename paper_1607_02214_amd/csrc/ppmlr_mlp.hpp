// Small MLP that proposes the starting pressure of the interface Riemann
// solver's Newton iteration (the learned guess of the paper's batched /
// learned variants): 14 inputs (left and right primitive states, normalised
// by the pair means), two hidden layers of 64 with the tanh form of GELU
// (Hendrycks & Gimpel 2016), 2 outputs (star pressure and velocity as
// residuals on the plain linear guess).
//
// BF16 operands, FP32 accumulation, on the gfx950 matrix cores
// (v_mfma_f32_16x16x16_bf16).  Every product is computed transposed, with
// samples along the N (column) dimension:  Z^T = W^T H^T.  Then the FP32
// accumulator tile of one layer (lane l: column l%16, rows 4*(l/16)+i) has
// exactly the register layout of the B operand of the next layer (lane l:
// column l%16, k = 4*(l/16)+i), so activations never leave registers in the
// forward pass.  Weights are A-operand fragments (64 lanes x 4 BF16 per 16x16
// tile, 8 bytes per lane): packed in memory for the sweep, built from the
// parameters in LDS by the batch kernels.
//
// Parameter vector theta (FP32, 5250 values): W1[14][64], b1[64],
// W2[64][64], b2[64], W3[64][2], b3[2], row-major (input index first).
#pragma once
#include <hip/hip_runtime.h>

namespace ppmlr {
namespace mlp {

constexpr int kIn = 14, kH = 64, kOut = 2;
constexpr int kOffW1 = 0, kOffB1 = kIn * kH, kOffW2 = kOffB1 + kH, kOffB2 = kOffW2 + kH * kH;
constexpr int kOffW3 = kOffB2 + kH, kOffB3 = kOffW3 + kH * kOut, kNPar = kOffB3 + kOut;
static_assert(kNPar == 5250, "parameter count");

// packed fragment tiles (each 16x16 tile = 256 BF16)
constexpr int kTA1 = 0;            // W1^T: 4 (m) x 1 (k)   forward layer 1
constexpr int kTA2 = 4;            // W2^T: 4 x 4           forward layer 2
constexpr int kTA3 = 20;           // W3^T: 1 x 4           forward layer 3
constexpr int kTB3 = 24;           // W3  : 4 x 1           backward through layer 3
constexpr int kTB2 = 28;           // W2  : 4 x 4           backward through layer 2
constexpr int kTiles = 44;
constexpr int kFwdTiles = 24;      // the forward pass needs tiles [0, 24)
constexpr int kRecord = 28;        // floats per harvested interface record

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// FP32 -> BF16, round to nearest even (quiet NaN kept NaN)
__device__ __forceinline__ unsigned short f2bf(float f)
{
    unsigned int u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf2f(unsigned short h) { return __uint_as_float((unsigned int)h << 16); }

// two FP32 -> BF16 in one instruction (round to nearest even, as f2bf; a in the
// lower half)
__device__ __forceinline__ unsigned int pack2(float a, float b)
{
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    const f2 ab = {a, b};
    return __builtin_bit_cast(unsigned int, __builtin_convertvector(ab, b2));
}
__device__ __forceinline__ bf16x4 pack4(float a, float b, float c, float d)
{
    return __builtin_bit_cast(bf16x4, make_uint2(pack2(a, b), pack2(c, d)));
}

__device__ __forceinline__ f32x4 mfma(bf16x4 a, bf16x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// tanh-form GELU, written through the logistic function:
// x/2 (1 + tanh(u)) = x * sigma(2u),  u = sqrt(2/pi) (x + 0.044715 x^3)
constexpr float kGc = 0.7978845608028654f, kGa = 0.044715f;
__device__ __forceinline__ float gelu(float x)
{
    const float u = kGc * (x + kGa * x * x * x);
    const float s = __builtin_amdgcn_rcpf(1.0f + __expf(-2.0f * u));
    return x * s;
}
// derivative: sigma(2u) + x * 2 sigma (1 - sigma) * du/dx
__device__ __forceinline__ float gelu_grad(float x)
{
    const float u = kGc * (x + kGa * x * x * x);
    const float s = __builtin_amdgcn_rcpf(1.0f + __expf(-2.0f * u));
    return s + x * 2.0f * s * (1.0f - s) * kGc * (1.0f + 3.0f * kGa * x * x);
}

// Value of fragment element (tile t, lane l, item i) of the packed set; t0: t or
// a smaller tile of the same matrix and direction.  th: theta, or a copy
// whose W1 and W2 have rows of LD values.
template <int LD = kH>
__device__ __forceinline__ float frag_value(const float *th, int t0, int t, int l, int i)
{
    constexpr int oW2 = kIn * LD + kH, oW3 = oW2 + kH * LD + kH;
    const int r = l & 15, kk = 4 * (l >> 4) + i;
    if (t0 < kTA2) {                       // W1^T: m = hidden, k = input feature
        const int m = t * 16 + r, k = kk;
        return k < kIn ? th[k * LD + m] : 0.0f;
    }
    if (t0 < kTA3) {                       // W2^T: m = out hidden, k = in hidden
        const int u = t - kTA2, m = (u >> 2) * 16 + r, k = (u & 3) * 16 + kk;
        return th[oW2 + k * LD + m];
    }
    if (t0 < kTB3) {                       // W3^T: m = output, k = hidden
        const int m = r, k = (t - kTA3) * 16 + kk;
        return m < kOut ? th[oW3 + k * kOut + m] : 0.0f;
    }
    if (t0 < kTB2) {                       // W3: m = hidden, k = output
        const int m = (t - kTB3) * 16 + r, k = kk;
        return k < kOut ? th[oW3 + m * kOut + k] : 0.0f;
    }
    {                                      // W2: m = in hidden, k = out hidden
        const int u = t - kTB2, m = (u >> 2) * 16 + r, k = (u & 3) * 16 + kk;
        return th[oW2 + m * LD + k];
    }
}

// Pack theta into BF16 fragments: frag[(t * 64 + l) * 4 + i].
__global__ void pack_kernel(const float *__restrict__ theta, unsigned short *__restrict__ frag, int tiles)
{
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= tiles * 256) return;
    const int t = idx >> 8, l = (idx >> 2) & 63, i = idx & 3;
    frag[idx] = f2bf(frag_value(theta, t, t, l, i));
}

__device__ __forceinline__ bf16x4 load_frag(const unsigned short *frag, int t, int lane)
{
    return *reinterpret_cast<const bf16x4 *>(frag + ((size_t)t * 64 + lane) * 4);
}

// Forward pass of one wave over 16 samples.  f0, f1: BF16 features 4q .. 4q + 3
// (q = lane / 16; columns 14, 15 zero) of sample lane mod 16, the lower one in
// the lower half.  Returns output 0 (the pressure) of that sample in lanes
// 0..15.  Must be called by all 64 lanes of the wave.  Only one tile's
// activations are live (this runs inside the sweep, next to the solver's own
// registers); the weight fragments are re-read per tile from the L2-resident
// packed buffer.
__device__ __forceinline__ float forward_tile(unsigned int f0, unsigned int f1, const unsigned short *frag,
                                              const float *__restrict__ theta)
{
    const int lane = threadIdx.x & 63;
    const int q = lane >> 4;
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    // keeps the weight loads inside the caller's loop (not hoisted into registers)
    asm volatile("" ::: "memory");
    const bf16x4 xb = __builtin_bit_cast(bf16x4, make_uint2(f0, f1));
    // layer 1: Z1^T[64 x 16] = W1^T[64 x 16] X^T[16 x 16]
    bf16x4 h1[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
        const f32x4 z = mfma(load_frag(frag, kTA1 + mt, lane), xb, zero);
        const float *b1 = theta + kOffB1 + mt * 16 + 4 * q;
        h1[mt] = pack4(gelu(z[0] + b1[0]), gelu(z[1] + b1[1]), gelu(z[2] + b1[2]), gelu(z[3] + b1[3]));
    }
    // layer 2: Z2^T = W2^T H1^T (weight loads kept per output tile, so
    // that at most four fragments are in flight)
    bf16x4 h2[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
        asm volatile("" ::: "memory");
        f32x4 acc = zero;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) acc = mfma(load_frag(frag, kTA2 + mt * 4 + kt, lane), h1[kt], acc);
        const float *b2 = theta + kOffB2 + mt * 16 + 4 * q;
        h2[mt] = pack4(gelu(acc[0] + b2[0]), gelu(acc[1] + b2[1]), gelu(acc[2] + b2[2]), gelu(acc[3] + b2[3]));
    }
    // layer 3: O^T[16 x 16] = W3^T[16 x 64] H2^T (rows 0, 1 valid)
    f32x4 o = zero;
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) o = mfma(load_frag(frag, kTA3 + kt, lane), h2[kt], o);
    return o[0] + theta[kOffB3];
}

// The parameters staged in LDS by a workgroup of 256: coalesced loads, rows of
// W1 and W2 of 65 values, so that a fragment's column is spread over the banks.
constexpr int kLdW = kH + 1;
constexpr int kStage = kNPar + kIn + kH;
constexpr int kStB1 = kIn * kLdW, kStB2 = kStB1 + kH + kH * kLdW, kStB3 = kStB2 + kH + kH * kOut;
__device__ __forceinline__ void stage_theta(const float *__restrict__ theta, float *stage)
{
#pragma unroll
    for (int k = 0; k < (kNPar + 255) / 256; ++k) {
        const int p = k * 256 + (int)threadIdx.x;
        const int row = p < kOffB1 ? p / kH : (p < kOffW2 ? kIn : (p < kOffB2 ? kIn + (p - kOffW2) / kH : kIn + kH));
        if (p < kNPar) stage[p + row * (kLdW - kH)] = theta[p];
    }
}

// Fragment of tile t of the packed set for this lane, from the staged
// parameters (t0: see frag_value).
__device__ __forceinline__ bf16x4 stage_frag(const float *stage, int t0, int t, int lane)
{
    return pack4(frag_value<kLdW>(stage, t0, t, lane, 0), frag_value<kLdW>(stage, t0, t, lane, 1),
                 frag_value<kLdW>(stage, t0, t, lane, 2), frag_value<kLdW>(stage, t0, t, lane, 3));
}

// Features of sample s for this lane as B operand (k = 4q .. 4q + 3; features
// 14, 15 are zero).  VEC: rows on 16-byte boundaries.
template <bool VEC>
__device__ __forceinline__ bf16x4 load_x(const float *__restrict__ X, int ldx, long long s, int q)
{
    const float *x = X + s * ldx + 4 * q;
    float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (VEC && q < 3) {
        const float4 w = *reinterpret_cast<const float4 *>(x);
        v[0] = w.x; v[1] = w.y; v[2] = w.z; v[3] = w.w;
    } else if (VEC) {
        const float2 w = *reinterpret_cast<const float2 *>(x);
        v[0] = w.x; v[1] = w.y;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (4 * q + i < kIn) v[i] = x[i];
    }
    return pack4(v[0], v[1], v[2], v[3]);
}

// Forward over n samples.  A wave keeps the whole network in registers (24
// fragments and the biases, ~80 registers, built once from theta staged in LDS)
// and takes tiles of 16 samples in turn, the next tile's features requested
// ahead; the samples do not go through LDS.  What bounds it is the GELU of 128 hidden units a sample
// (10 vector instructions, two of them transcendental): the matrix products
// take a quarter of that and the records 112 MB.  1 M records with rows of 28
// floats: 170 us as one wave per 64 samples with the weights re-read per tile
// (and a launch to pack them), 68 us now.
template <bool VEC>
__global__ void __launch_bounds__(256) forward_kernel(const float *__restrict__ X, int ldx, int n,
                                                      const float *__restrict__ theta, float *__restrict__ Y, int ldy)
{
    const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    const int tiles = (int)(((long long)n + 15) / 16), nw = (int)gridDim.x * 4;
    int tile = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6);
    __shared__ float stage[kStage];
    auto sample = [&](int t) { const long long s = (long long)t * 16 + r; return s < n ? s : (long long)n - 1; };
    bf16x4 xb = load_x<VEC>(X, ldx, sample(tile), q);
    bf16x4 w1[4], w2[16], w3[4];
    f32x4 b1[4], b2[4];
    stage_theta(theta, stage);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        w1[t] = stage_frag(stage, kTA1, kTA1 + t, lane);
        w3[t] = stage_frag(stage, kTA3, kTA3 + t, lane);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            b1[t][i] = stage[kStB1 + t * 16 + 4 * q + i];
            b2[t][i] = stage[kStB2 + t * 16 + 4 * q + i];
        }
    }
#pragma unroll
    for (int t = 0; t < 16; ++t) w2[t] = stage_frag(stage, kTA2, kTA2 + t, lane);
    const float b30 = stage[kStB3], b31 = stage[kStB3 + 1];
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    for (; tile < tiles; tile += nw) {
        const bf16x4 x0 = xb;
        if (tile + nw < tiles) xb = load_x<VEC>(X, ldx, sample(tile + nw), q);
        bf16x4 h1[4], h2[4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            const f32x4 z = mfma(w1[mt], x0, zero);
            h1[mt] = pack4(gelu(z[0] + b1[mt][0]), gelu(z[1] + b1[mt][1]), gelu(z[2] + b1[mt][2]),
                           gelu(z[3] + b1[mt][3]));
        }
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            f32x4 z = zero;
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) z = mfma(w2[mt * 4 + kt], h1[kt], z);
            h2[mt] = pack4(gelu(z[0] + b2[mt][0]), gelu(z[1] + b2[mt][1]), gelu(z[2] + b2[mt][2]),
                           gelu(z[3] + b2[mt][3]));
        }
        f32x4 o = zero;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) o = mfma(w3[kt], h2[kt], o);
        const long long s = (long long)tile * 16 + r;
        if (q == 0 && s < n) {
            Y[s * ldy + 0] = o[0] + b30;
            Y[s * ldy + 1] = o[1] + b31;
        }
    }
}

// Sum over the 16 lanes of a row (every lane gets it), in registers.
__device__ __forceinline__ float row_sum(float v)
{
#define PPMLR_ROR(n) v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + n, 0xf, 0xf, true))
    PPMLR_ROR(8);
    PPMLR_ROR(4);
    PPMLR_ROR(2);
    PPMLR_ROR(1);
#undef PPMLR_ROR
    return v;
}

// Loss and gradient of L = (1 / 2n) sum (o - y)^2.  A workgroup of four waves
// packs the parameters into LDS fragments, then every wave takes tiles of 16
// samples: forward and backward as matrix products that hand their result
// tiles on in registers, the weight gradients as contractions over the
// tile's samples (operands transposed through the wave's own part of LDS),
// accumulated in registers over the wave's tiles.  At the end the four waves'
// gradients are added in a fixed order and the workgroup writes one partial
// gradient, in theta order, and its partial loss to part[kNPar].  The
// backward pass uses BF16 operands / FP32 accumulation; the GELU derivatives
// are rounded to BF16.
// Tiles of 16 samples a wave put a batch of 4096 on 256 waves.  A tile itself
// takes 4 us; the rest is the chain around it, so the parameters come to LDS by
// coalesced loads (gathered from memory as fragments: 6.5 us), with rows of 65
// that spread their columns over the banks, and the gradients are added as
// they lie in the registers, 16 bytes a lane, by all threads (in theta order,
// one wave at a time, value by value: 8 us).  Batch of 4096: 22 us before,
// 9.9 us now; a training step 25.6 and 14.3 us.
constexpr int kGradWave = (16 + 64 * 4 + 16) * 16;                 // BF16 values of a wave's transposed operands
constexpr size_t kGradLds = (size_t)kTiles * 512 + 4 * (size_t)kGradWave * 2;
static_assert(kStage * 4 <= 4 * kGradWave * 2, "the parameters are staged where the operands go");
constexpr int kSumRegs = 12;                                       // registers (x 4) of a wave added at a time
constexpr size_t kSumBias = (size_t)4 * kSumRegs * 1024;           // after them: both biases' and the scalars
static_assert(kSumBias + 4 * (2 * kH + 4) * 4 <= kGradLds, "the reduction reuses the operands' LDS");

template <bool VEC>
__global__ void __launch_bounds__(256) grad_kernel(const float *__restrict__ X, int ldx, const float *__restrict__ Yt,
                                                   int ldy, int n, const float *__restrict__ theta,
                                                   float *__restrict__ partials)
{
    __shared__ __align__(16) unsigned char lds[kGradLds];
    unsigned short *frag = reinterpret_cast<unsigned short *>(lds);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, q = lane >> 4;
    unsigned short *XT = frag + kTiles * 256 + wave * kGradWave;    // [feature][sample]
    unsigned short *H1T = XT + 16 * 16, *H2T = H1T + 64 * 16;       // [hidden][sample]
    unsigned short *D2T = H2T + 64 * 16, *D1T = D2T + 64 * 16;      // dZ2^T, dZ1^T
    unsigned short *DOT = D1T + 64 * 16;                            // dO^T, rows >= 2 zero
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    const int tiles = (n + 15) / 16;
    int tile = (int)blockIdx.x * 4 + wave;
    // the first tile's samples
    auto sample = [&](int t) -> long long { return min((long long)t * 16 + r, (long long)n - 1); };
    bf16x4 xn = load_x<VEC>(X, ldx, sample(tile), q);
    float y0 = Yt[sample(tile) * ldy], y1 = Yt[sample(tile) * ldy + 1];
    float *stage = reinterpret_cast<float *>(frag + kTiles * 256);
    stage_theta(theta, stage);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kTiles; k += 4) {                           // (four tiles of one matrix)
        const int t = k + wave;
        *reinterpret_cast<bf16x4 *>(frag + (t * 64 + lane) * 4) = stage_frag(stage, k, t, lane);
    }
    f32x4 b1[4], b2[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            b1[t][i] = stage[kStB1 + t * 16 + 4 * q + i];
            b2[t][i] = stage[kStB2 + t * 16 + 4 * q + i];
        }
    const float b30 = stage[kStB3], b31 = stage[kStB3 + 1];
    __syncthreads();                                                // (the operands go where the stage was)
    auto weights = [&](int t) { return *reinterpret_cast<const bf16x4 *>(frag + (t * 64 + lane) * 4); };
    auto put = [&](unsigned short *M, int row0, const bf16x4 &v) {  // rows row0 + 4q .. + 3 of sample r
#pragma unroll
        for (int i = 0; i < 4; ++i) M[(row0 + 4 * q + i) * 16 + r] = (unsigned short)v[i];
    };
    auto get = [&](const unsigned short *M, int row0) {             // row row0 + r, samples 4q .. 4q + 3
        return *reinterpret_cast<const bf16x4 *>(M + (row0 + r) * 16 + 4 * q);
    };
    f32x4 gw1[4], gw2[16], gw3[4], gb1[4], gb2[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) { gw1[t] = gw3[t] = gb1[t] = gb2[t] = zero; }
#pragma unroll
    for (int t = 0; t < 16; ++t) gw2[t] = zero;
    float sq = 0.0f, gb30 = 0.0f, gb31 = 0.0f;
    const float inv_n = 1.0f / (float)n;
    for (; tile < tiles; tile += (int)gridDim.x * 4) {
        const bool in = (long long)tile * 16 + r < n;
        bf16x4 x = xn;
        const float t0 = y0, t1 = y1;
        if (!in) x = bf16x4{0, 0, 0, 0};
        const int next = tile + (int)gridDim.x * 4;
        if (next < tiles) {
            xn = load_x<VEC>(X, ldx, sample(next), q);
            y0 = Yt[sample(next) * ldy];
            y1 = Yt[sample(next) * ldy + 1];
        }
        put(XT, 0, x);
        // ---- forward, keeping the activations and the GELU derivatives
        bf16x4 h1[4], h2[4], g1[4], g2[4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            f32x4 z = mfma(weights(kTA1 + mt), x, zero);
#pragma unroll
            for (int i = 0; i < 4; ++i) z[i] += b1[mt][i];
            g1[mt] = pack4(gelu_grad(z[0]), gelu_grad(z[1]), gelu_grad(z[2]), gelu_grad(z[3]));
            h1[mt] = pack4(gelu(z[0]), gelu(z[1]), gelu(z[2]), gelu(z[3]));
            put(H1T, mt * 16, h1[mt]);
        }
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            f32x4 z = zero;
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) z = mfma(weights(kTA2 + mt * 4 + kt), h1[kt], z);
#pragma unroll
            for (int i = 0; i < 4; ++i) z[i] += b2[mt][i];
            g2[mt] = pack4(gelu_grad(z[0]), gelu_grad(z[1]), gelu_grad(z[2]), gelu_grad(z[3]));
            h2[mt] = pack4(gelu(z[0]), gelu(z[1]), gelu(z[2]), gelu(z[3]));
            put(H2T, mt * 16, h2[mt]);
        }
        f32x4 o = zero;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) o = mfma(weights(kTA3 + kt), h2[kt], o);
        // ---- output error dO = (o - y) / n (rows 0, 1 of the output tile), loss
        float d0 = 0.0f, d1 = 0.0f;
        if (q == 0 && in) {
            const float e0 = o[0] + b30 - t0, e1 = o[1] + b31 - t1;
            sq += e0 * e0;
            sq += e1 * e1;
            d0 = e0 * inv_n;
            d1 = e1 * inv_n;
        }
        gb30 += d0;
        gb31 += d1;
        const bf16x4 dO = pack4(d0, d1, 0.0f, 0.0f);
        put(DOT, 0, dO);
        // ---- through layer 3: dH2^T = W3 dO^T, dZ2 = dH2 gelu'(Z2)
        bf16x4 d2[4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            f32x4 g = mfma(weights(kTB3 + mt), dO, zero);
#pragma unroll
            for (int i = 0; i < 4; ++i) g[i] *= bf2f((unsigned short)g2[mt][i]);
            gb2[mt] += g;
            d2[mt] = pack4(g[0], g[1], g[2], g[3]);
            put(D2T, mt * 16, d2[mt]);
        }
        // ---- through layer 2: dH1^T = W2 dZ2^T, dZ1 = dH1 gelu'(Z1)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
            f32x4 g = zero;
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) g = mfma(weights(kTB2 + mt * 4 + kt), d2[kt], g);
#pragma unroll
            for (int i = 0; i < 4; ++i) g[i] *= bf2f((unsigned short)g1[mt][i]);
            gb1[mt] += g;
            put(D1T, mt * 16, pack4(g[0], g[1], g[2], g[3]));
        }
        __builtin_amdgcn_wave_barrier();                            // (a wave's LDS accesses stay in order)
        // ---- weight gradients: contractions over the 16 samples
        const bf16x4 dot = get(DOT, 0), xt = get(XT, 0);
        bf16x4 d2t[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            d2t[t] = get(D2T, t * 16);
            gw3[t] = mfma(get(H2T, t * 16), dot, gw3[t]);           // dW3[hid][o] = sum_s H2[s][hid] dO[s][o]
            gw1[t] = mfma(xt, get(D1T, t * 16), gw1[t]);            // dW1[f][h] = sum_s X[s][f] dZ1[s][h]
        }
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {                            // dW2[h1][h2] = sum_s H1[s][h1] dZ2[s][h2]
            const bf16x4 h = get(H1T, mt * 16);
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) gw2[mt * 4 + nt] = mfma(h, d2t[nt], gw2[mt * 4 + nt]);
        }
        __builtin_amdgcn_wave_barrier();
    }
    // ---- the waves' gradients: sums over the lanes where a lane holds a part
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            gb1[t][i] = row_sum(gb1[t][i]);
            gb2[t][i] = row_sum(gb2[t][i]);
        }
    gb30 = row_sum(gb30);
    gb31 = row_sum(gb31);
    sq = row_sum(sq);
    // every wave's registers into LDS as they are, kSumRegs of the 24 at a time,
    // then four threads' share each: (wave 0 + wave 2) + (wave 1 + wave 3)
    float *part = partials + (size_t)blockIdx.x * (kNPar + 1);
    f32x4 *raw = reinterpret_cast<f32x4 *>(lds);
    float *small = reinterpret_cast<float *>(lds + kSumBias);       // [wave][b1 64, b2 64, b3 2, loss]
    auto sum4 = [](auto a, auto b, auto c, auto d) { return (a + c) + (b + d); };
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kSumRegs; ++k) {
            const int j = half * kSumRegs + k;                      // gw2 0..15, gw1, gw3
            raw[(wave * kSumRegs + k) * 64 + lane] = j < 16 ? gw2[j] : (j < 20 ? gw1[j - 16] : gw3[j - 20]);
        }
        if (half == 0) {
            float *sm = small + wave * (2 * kH + 4);
            if (r == 0) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    *reinterpret_cast<f32x4 *>(sm + t * 16 + 4 * q) = gb1[t];
                    *reinterpret_cast<f32x4 *>(sm + kH + t * 16 + 4 * q) = gb2[t];
                }
            }
            if (lane == 0) { sm[2 * kH] = gb30; sm[2 * kH + 1] = gb31; sm[2 * kH + 2] = sq; }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kSumRegs; k += 4) {
            const f32x4 *x = raw + (k + wave) * 64 + lane;
            const f32x4 v = sum4(x[0], x[kSumRegs * 64], x[2 * kSumRegs * 64], x[3 * kSumRegs * 64]);
            const int j0 = half * kSumRegs + k, j = j0 + wave;      // (four registers of one matrix)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (j0 < 16) part[kOffW2 + ((j >> 2) * 16 + 4 * q + i) * kH + (j & 3) * 16 + r] = v[i];
                else if (j0 < 20) { if (4 * q + i < kIn) part[kOffW1 + (4 * q + i) * kH + (j - 16) * 16 + r] = v[i]; }
                else if (r < kOut) part[kOffW3 + ((j - 20) * 16 + 4 * q + i) * kOut + r] = v[i];
            }
        }
        if (half == 0 && threadIdx.x < 2 * kH + 3) {
            constexpr int w = 2 * kH + 4;
            const int k = threadIdx.x;
            const float v = sum4(small[k], small[w + k], small[2 * w + k], small[3 * w + k]);
            if (k < kH) part[kOffB1 + k] = v;
            else if (k < 2 * kH) part[kOffB2 + k - kH] = v;
            else if (k < 2 * kH + 2) part[kOffB3 + k - 2 * kH] = v;
            else part[kNPar] = 0.5f * v * inv_n;
        }
    }
}

// Sum the per-workgroup partials in a fixed order: 64 parameters per workgroup,
// four threads each (consecutive quarters of the partials, added in LDS).
// grad (may be null) receives the gradient, loss (may be null) the loss; with
// adam != 0 the bias-corrected Adam step (Kingma & Ba 2015; c1, c2 = 1 - beta^t)
// is applied to theta in place.  One thread per parameter over all 64 partials
// of a batch of 4096 was 21 workgroups waiting on 64 loads each (16.9 us; now
// 4.2 us).
__global__ void __launch_bounds__(256) reduce_adam_kernel(const float *__restrict__ partials, int nblk, float *grad,
                                                          float *loss, float *theta, float *m, float *v, int adam,
                                                          float c1, float c2, float lr, float b1, float b2, float eps)
{
    __shared__ float part[4][64];
    const int j = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int p = blockIdx.x * 64 + j;
    const int per = (nblk + 3) / 4, lo = w * per, hi = min(nblk, lo + per);
    float g = 0.0f;
    if (p <= kNPar) {
#pragma unroll 16
        for (int b = lo; b < hi; ++b) g += partials[(size_t)b * (kNPar + 1) + p];
    }
    part[w][j] = g;
    __syncthreads();
    if (w != 0 || p > kNPar) return;
    g = ((part[0][j] + part[1][j]) + part[2][j]) + part[3][j];
    if (p == kNPar) {
        if (loss) *loss = g;
        return;
    }
    if (grad) grad[p] = g;
    if (adam) {
        const float mm = b1 * m[p] + (1.0f - b1) * g;
        const float vv = b2 * v[p] + (1.0f - b2) * g * g;
        m[p] = mm;
        v[p] = vv;
        theta[p] -= lr * (mm / c1) / (sqrtf(vv / c2) + eps);
    }
}

}  // namespace mlp
}  // namespace ppmlr
