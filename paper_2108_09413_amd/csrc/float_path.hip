// Kernels of the two floating-point comparison systems of the paper's evaluation (section
// "Experiments": FloatRS-quant, FloatRS-fp): continuous Gaussian noise on the image, then either
// rounding back onto the pixel grid (the int8 network follows) or the fp32 network, whose
// convolutions run here as implicit GEMMs on the bfloat16 MFMA with exactly split operands.
#include <hip/hip_runtime.h>

#include <string>

#include "conv_device.h"
#include "isr_internal.h"
#include "nearest_root.h"
#include "noise_device.h"

namespace isr {

namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// The binary32 standard-normal sampler.  Every step is one IEEE operation (+, -, *, /, sqrt,
// rounded once, never contracted into a fused multiply-add), so a draw is the same bit pattern
// on any conforming machine:
//   Box-Muller on two 32-bit words (wa, wb): u = ((wa >> 8) + 1) / 2^24 in (0, 1],
//   v = (wb >> 8) / 2^24 in [0, 1);  z_a = sqrt(-2 ln u) cos(2 pi v), z_b = sqrt(-2 ln u) sin(2 pi v);
//   ln by range reduction to [sqrt(1/2), sqrt(2)] and the atanh series, cos / sin by octant and the
//   Taylor polynomials on [0, pi/4).

// -ln(n / 2^24), n in [1, 2^24].
__device__ __forceinline__ float neg_log_u24(uint32_t n) {
#pragma clang fp contract(off)
    const float f = (float)n;                                  // exact
    const uint32_t bits = __float_as_uint(f);
    int E = (int)(bits >> 23) - 127;                           // n = m 2^E, m in [1, 2)
    float m = __uint_as_float((bits & 0x7FFFFFu) | 0x3F800000u);
    if (m > 1.41421354f) { m = m * 0.5f; E += 1; }
    const float k = (float)(24 - E);
    const float s = __fdiv_rn(m - 1.0f, m + 1.0f);             // ln m = 2 atanh(s)
    const float s2 = s * s;
    float p = 0.222222224f;
    p = p * s2; p = p + 0.285714298f;
    p = p * s2; p = p + 0.400000006f;
    p = p * s2; p = p + 0.666666687f;
    p = p * s2; p = p + 2.0f;
    const float lnm = s * p;
    const float a = k * 0.693145752f;                          // ln 2 = hi + lo; k * hi is exact
    const float b = k * 1.42860677e-06f;
    const float d = a - lnm;
    return d + b;
}

// cos and sin of 2 pi t / 2^24, t in [0, 2^24).
__device__ __forceinline__ void cos_sin_turn24(uint32_t t, float &co, float &si) {
#pragma clang fp contract(off)
    const float phi = (float)(t & 0x1FFFFFu) * 3.74507039e-07f;              // (pi/4) / 2^21
    const float x2 = phi * phi;
    float c = -2.755732e-07f;
    c = c * x2; c = c + 2.48015876e-05f;
    c = c * x2; c = c - 0.00138888892f;
    c = c * x2; c = c + 0.0416666679f;
    c = c * x2; c = c - 0.5f;
    c = c * x2; c = c + 1.0f;
    float s = 2.75573188e-06f;
    s = s * x2; s = s - 0.000198412701f;
    s = s * x2; s = s + 0.00833333377f;
    s = s * x2; s = s - 0.166666672f;
    s = s * x2; s = s + 1.0f;
    s = s * phi;
    float d = c - s, e = c + s;
    d = d * 0.707106769f;
    e = e * 0.707106769f;
    // odd octants: the angle pi/4 on, (d, e); then quarter turns: (p, q), (-q, p), (-p, -q), (q, -p).  By selection and sign
    // bits: as a switch every wave went through all eight cases.
    const float p = t & (1u << 21) ? d : c, q = t & (1u << 21) ? e : s;
    const bool quarter = t & (1u << 22);
    co = __uint_as_float(__float_as_uint(quarter ? q : p) ^ (((t << 8) ^ (t << 9)) & 0x80000000u));
    si = __uint_as_float(__float_as_uint(quarter ? p : q) ^ ((t << 8) & 0x80000000u));
}

// The root instruction is off by at most one unit, in a sixth of the draws.  With the binary64 root, rounded once more, a certification of
// ResNet-20 on rounded noise (10 100 copies) took 606.6 us, with this 600.9.
__device__ __forceinline__ float sqrt_rn(float x) { return nearest_root(x, __builtin_amdgcn_sqrtf(x)); }

__device__ __forceinline__ void box_muller(uint32_t wa, uint32_t wb, float &za, float &zb) {
#pragma clang fp contract(off)
    const float l = neg_log_u24((wa >> 8) + 1u);
    const float r = sqrt_rn(2.0f * l);
    float c, s;
    cos_sin_turn24(wb >> 8, c, s);
    za = r * c;
    zb = r * s;
}

// One thread per four horizontally adjacent pixels of one copy: per channel one Philox call gives
// the four draws of logical elements (c*H + y)*W + 4 x4 .. + 3.
__global__ __launch_bounds__(256) void float_noise_kernel(const FloatNoiseParams p) {
#pragma clang fp contract(off)
    const int W4 = p.W >> 2;
    const long groups_per_sample = (long)p.H * W4;
    const long total = groups_per_sample * p.count;
    for (long g = (long)blockIdx.x * 256 + threadIdx.x; g < total; g += (long)gridDim.x * 256) {
        const uint32_t s_local = (uint32_t)(g / groups_per_sample);
        const int rem = (int)(g - (long)s_local * groups_per_sample);
        const int y = rem / W4, x4 = rem - y * W4;
        float v[3][4];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[c][j] = p.quant ? 128.0f : p.center;   // absent channels: code 0 / real value 0
            if (c < p.C) {
                const uint32_t pix = (uint32_t)((c * p.H + y) * p.W + x4 * 4);
                uint32_t w[4];
                philox4x32_10(pix >> 2, p.sample_begin + s_local, p.image, 8u + p.phase, p.key0, p.key1, w);
                float z[4];
                box_muller(w[0], w[1], z[0], z[1]);
                box_muller(w[2], w[3], z[2], z[3]);
                const uint32_t px4 = *(const uint32_t *)(p.x + pix);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float sz = p.sigma * z[j];
                    v[c][j] = (float)((px4 >> (8 * j)) & 0xFF) + sz;
                }
            }
        }
        const long o = (long)s_local * groups_per_sample + rem;
        if (p.quant) {
            int packed[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                uint32_t word = 0;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    float r = rintf(v[c][j]);
                    r = r < 0.0f ? 0.0f : (r > 255.0f ? 255.0f : r);
                    word |= (uint32_t)(((int)r - 128) & 0xFF) << (8 * c);
                }
                packed[j] = (int)word;
            }
            *(v4i *)((int8_t *)p.out + o * 16) = v4i{packed[0], packed[1], packed[2], packed[3]};
        } else {
            float *dst = (float *)p.out + o * 16;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                *(v4f *)(dst + 4 * j) = v4f{v[0][j] - p.center, v[1][j] - p.center, v[2][j] - p.center, 0.0f};
        }
    }
}

// ---------------------------------------------------------------------------
// fp32 convolution: implicit GEMM on v_mfma_f32_32x32x16_bf16 with exact operands.  A = weights (rows = output channels),
// B = im2col pixels (columns), K = (tap, channel) in steps of 32.
//
// The weights are the int8 codes of the quantized network: whole numbers of at most 8 bits, exact in bfloat16.  An fp32
// activation is the exact sum of three bfloat16 numbers, x = x1 + x2 + x3, each the leading 8 bits of what the ones before
// leave (24 = 8 + 8 + 8).  So x w = x1 w + x2 w + x3 w with every product of 16 bits and fp32 accumulation, at a third of the
// bfloat16 rate (2500 / 3 = 833 TFLOP/s nominal) instead of the fp32 one (157).
//
// How the matrix unit adds (measured bit for bit): 8 products at a time, each cut towards zero at 2^-24 of the largest of
// their powers of two; the accumulator cut there as well, downwards; their sum rounded to nearest fp32.  One rounding per 8
// products and part, where the fp32 instruction rounds after every product, so a sum is closer to the exact one (0.72 of
// the error).  But where the accumulator is smaller than a product it loses bits downwards, and sums are too low by
// 3e-9 .. 3e-8 of their size on average: nothing in one layer, but a residual stream collected it over its blocks
// (ResNet-110: 5.3e-7 on the logits, nine tenths of it the same in every copy).  Therefore every other channel is
// computed with its sign reversed, and the channels change roles from block to block (float_api.cpp): the shares cancel.
//
// Both operands go from global memory straight into LDS, two steps deep: the weights as bfloat16 rows of 64 bytes, the
// pixels as fp32 rows of 128 bytes (4 bytes an element to read where three stored parts would be 6); 16-byte chunks
// swizzled on the global side (conv_device.h).  Out-of-image taps come from a page of zeros.  Each of the four waves owns all BM channels of its own
// 32 NT pixels, so a pixel fragment is split in registers by one wave only: 5.5 instructions an element, for MT MFMAs of
// 32 cycles per 8 of them.
//
// ResNet-50 at 224 x 224, 668 copies: 58 -> 26.8 ms for all layers by these products, 96 -> 213 TFLOP/s on 128-channel tiles; 18.6 ms
// with the fused and the 3x3 kernels below.
// Error of the logits against binary64 (2-norm), fp32 instruction -> this kernel: tiny net 3.5e-7 -> 3.3e-7, ResNet-20
// 2.0e-7 -> 1.55e-7, ResNet-110 3.1e-7 -> 2.5e-7, ResNet-50 at 96 to 224 pixels 8.1 .. 9.5e-7 -> 4.9 .. 5.8e-7; with the sums that
// fpatch_kernel, fpatch16_kernel and fstem_pool_kernel keep apart 3.3e-7, 1.45e-7, 2.1e-7 and 4.8 .. 5.4e-7.
//
// FLAT: 1x1 stride-1 layers; else TABLE: K chunks of 4 channels looked up in ktab (a tap changes inside a step), else a
// step lies inside one tap (Cin a multiple of 32) and its tap is counted along, all taps of 32 channels before the next 32.  PAIR: a 1x1 layer of any stride whose residual is
// another one's result that nothing else reads (the first block of a stage: closing convolution and projection).  The kernel
// computes that one first and keeps it in registers, with the same operations on the same numbers; three stages, because such
// layers have few steps (two: 1407 / 1086 / 729 / 605 us).  668 copies, two kernels -> one, at 56 / 28 / 14 / 7 pixels: 1881 -> 919,
// 1220 -> 771, 866 -> 646, 665 -> 562 us.

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
enum FAddress { F_FLAT, F_TAP, F_TABLE, F_PAIR };

// the three bfloat16 parts of 8 floats, 8 to a register quadruple
__device__ __forceinline__ void split_bf16(const v4f &lo, const v4f &hi, v4i (&part)[3]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float a = i < 2 ? lo[2 * i] : hi[2 * i - 4], b = i < 2 ? lo[2 * i + 1] : hi[2 * i - 3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            part[k][i] = (int)__builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);   // both upper halves
            if (k < 2) {
                a = a - __uint_as_float(__float_as_uint(a) & 0xFFFF0000u);   // exact
                b = b - __uint_as_float(__float_as_uint(b) & 0xFFFF0000u);
            }
        }
    }
}

// Epilogue of a tile of 32 MT channels by 32 NT pixels a wave: with the weight rows in MFMA row order a lane holds 16 consecutive
// channels of one pixel.  Bias and scale come from LDS (`bs`, a stage that the last step did not use), the residual is read three groups
// of 16 channels ahead: a load waits for the stores issued before it, and with bias, scale and residual loaded where they are used
// each of the 8 MT stores of a wave was waited for in turn (64 -> 256 with residual, 668 copies of 56 x 56: 1285 -> 1140 us).
// PAIR: the residual is in `other`.  FULL: every pixel and channel of the tile exists.
template <bool FULL, bool RES, bool PAIR, int MT, int NT, class Other>
__device__ __forceinline__ void fconv_finish(const FConvParams &p, const v16f (&acc)[MT][NT], const Other &other, const float *bs, long px, int ch0, int lane) {
    constexpr int BM = 32 * MT, U = NT * MT, AHEAD = 3;
    const int half = lane >> 5, l32 = lane & 31;
    const float lo = p.relu ? 0.0f : -INFINITY, add_lo = p.add_relu ? 0.0f : -INFINITY;
    long at[NT];
    bool ok[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const long P = px + j * 32 + l32;
        ok[j] = FULL || P < p.npix;
        at[j] = (ok[j] ? P : 0) * p.Cout_p + ch0 + 16 * half;
    }
    // Cout_p is a multiple of 16: the run of a lane is stored whole or not at all
    auto there = [&](int u) { return FULL || (ok[u / MT] && ch0 + (u % MT) * 32 + 16 * half < p.Cout_p); };
    constexpr bool LOADED = RES && !PAIR;
    v4f r[LOADED ? AHEAD + 1 : 1][4];
    auto fetch = [&](int u) {
        const float *src = p.res + (there(u) ? at[u / MT] + (u % MT) * 32 : 0);
#pragma unroll
        for (int g = 0; g < 4; ++g) r[LOADED ? u % (AHEAD + 1) : 0][g] = *(const v4f *)(src + 4 * g);
    };
    if constexpr (LOADED)
#pragma unroll
        for (int u = 0; u < AHEAD && u < U; ++u) fetch(u);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = u % MT, j = u / MT, ch = i * 32 + 16 * half;
        if constexpr (LOADED)
            if (u + AHEAD < U) fetch(u + AHEAD);
        __builtin_amdgcn_sched_barrier(0);
        v4f t[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const v4f bias = *(const v4f *)(bs + ch + 4 * g), scale = *(const v4f *)(bs + BM + ch + 4 * g);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                t[g][e] = fmaxf((acc[i][j][4 * g + e] + bias[e]) * scale[e], lo);
                if constexpr (LOADED) t[g][e] = fmaxf(p.ma * t[g][e] + p.mb * r[u % (AHEAD + 1)][g][e], add_lo);
                else if constexpr (RES) t[g][e] = fmaxf(p.ma * t[g][e] + p.mb * other[i][j][4 * g + e], add_lo);
            }
        }
        if (there(u))
#pragma unroll
            for (int g = 0; g < 4; ++g) *(v4f *)(p.out + at[j] + i * 32 + 4 * g) = t[g];
    }
}
template <bool PAIR, int MT, int NT, class Other>
__device__ __forceinline__ void fconv_finish_tile(const FConvParams &p, const v16f (&acc)[MT][NT], const Other &other, const float *bs, long px0, int ch0,
                                                  int wave, int lane, int waves) {
    const bool full = px0 + waves * 32 * NT <= p.npix && ch0 + 32 * MT <= p.Cout_p;
    const long px = px0 + wave * NT * 32;
    if (PAIR || p.res) {
        if (full) fconv_finish<true, true, PAIR>(p, acc, other, bs, px, ch0, lane);
        else fconv_finish<false, true, PAIR>(p, acc, other, bs, px, ch0, lane);
    } else {
        if (full) fconv_finish<true, false, PAIR>(p, acc, other, bs, px, ch0, lane);
        else fconv_finish<false, false, PAIR>(p, acc, other, bs, px, ch0, lane);
    }
}

// of 4 floats, 4 to a pair
__device__ __forceinline__ void split_bf16_4(const v4f &v, uint2 (&part)[3]) {
    float x[4] = {v[0], v[1], v[2], v[3]};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        part[k].x = __builtin_amdgcn_perm(__float_as_uint(x[1]), __float_as_uint(x[0]), 0x07060302u);
        part[k].y = __builtin_amdgcn_perm(__float_as_uint(x[3]), __float_as_uint(x[2]), 0x07060302u);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (k < 2) x[e] = x[e] - __uint_as_float(__float_as_uint(x[e]) & 0xFFFF0000u);   // exact
    }
}

template <int MT, int NT, int ADDR>
__global__ __launch_bounds__(256, 2) void fconv_kernel(const FConvParams p) {
    constexpr int BM = 32 * MT, BN = 128 * NT;
    constexpr int ASTAGE = BM * 64, STAGE = ASTAGE + BN * 128;   // bytes
    constexpr int NA = (BM + 63) / 64, NB = BN / 32;             // direct-to-LDS loads per lane and step
    constexpr bool PAIR = ADDR == F_PAIR;
    constexpr int NST = PAIR ? 3 : 2;                            // stages; the steps after the current one are on their way to the others
    __shared__ __attribute__((aligned(256))) int8_t lds[NST * STAGE];
    __shared__ __attribute__((aligned(16))) float consts[PAIR ? 4 * BM : 1];                  // PAIR: bias, scale of the other layer, then of this one

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int mtiles = p.Cout_pp / BM;
    // Workgroup ids are dealt round-robin over the 8 XCDs (each with its own L2): renumber them so that an XCD
    // works on a contiguous run of tiles, in which the channel tiles of one pixel tile are neighbours and
    // share that pixel tile through the XCD's L2.
    const long nb = gridDim.x, per = nb >> 3, rem = nb & 7;
    const long xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const long bid = xcd * per + (xcd < rem ? xcd : rem) + slot;   // XCD x owns per (+1 for x < rem) consecutive ids
    const int ch0 = (int)(bid % mtiles) * BM;
    const long px0 = (bid / mtiles) * BN;
    const uint32_t lds0 = lds_address(lds);

    // The lane's place in a step: of the pixels, 16-byte chunk `bc` (4 channels) of rows tid / 8 + 32 j; of the weights,
    // chunk `ac` (8 channels) of rows tid / 4 + 64 j.  LDS position (row, c) holds chunk c ^ swz(row), the same for all
    // rows of a lane.
    const int brow = tid >> 3, bc = (tid & 7) ^ swz<8>(brow);
    const int arow = tid >> 2, ac = (tid & 3) ^ swz<4>(arow);
    const uint8_t *wsrc = (const uint8_t *)p.w + ((size_t)(ch0 + arow) * 64 + ac * 16);
    const uint8_t *in = (const uint8_t *)p.in;
    uint32_t boff[NB];          // byte offset of tap (0, 0) of the lane's pixel (of the pixel itself: FLAT), wrapping below 0
    uint32_t boff2[ADDR == F_PAIR ? NB : 1];
    int iy0[NB], ix0[NB];
    const int hw_o = p.Ho * p.Wo;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const long P = px0 + brow + 32 * j;
        const int n = (int)(P < p.npix ? P : p.npix - 1);      // pixels past the end repeat the last one; never stored
        if constexpr (ADDR == F_FLAT) {
            boff[j] = (uint32_t)n * (uint32_t)(p.Cin_p * 4) + (uint32_t)(bc * 16);
        } else if constexpr (ADDR == F_PAIR) {
            const int b = n / hw_o, r = n - b * hw_o, oy = r / p.Wo, ox = r - oy * p.Wo;
            boff[j] = (uint32_t)((b * p.H + oy * p.stride) * p.W + ox * p.stride) * (uint32_t)(p.Cin_p * 4) + (uint32_t)(bc * 16);
            boff2[j] = (uint32_t)((b * p.H2 + oy * p.stride2) * p.W2 + ox * p.stride2) * (uint32_t)(p.Cin2_p * 4) + (uint32_t)(bc * 16);
        } else {
            const int b = n / hw_o, r = n - b * hw_o, oy = r / p.Wo, ox = r - oy * p.Wo;
            const int y = oy * p.stride - p.pad, x = ox * p.stride - p.pad;
            iy0[j] = y;
            ix0[j] = x;
            boff[j] = (uint32_t)(((b * p.H + y) * p.W + x) * p.Cin_p * 4) + (ADDR == F_TAP ? (uint32_t)(bc * 16) : 0u);
        }
    }
    const int nsteps = p.Kq >> 3;
    int dy = 0, dx = 0, c0 = 0;                 // F_TAP: tap and first channel of the next step to fetch
    int entry = ADDR == F_TABLE ? p.ktab[bc] : 0;   // F_TABLE: the lane's quad of the next step to fetch
    auto issue = [&](int step, int buf) {
        const uint32_t a = lds0 + buf * STAGE + wave * 1024, b = lds0 + buf * STAGE + ASTAGE + wave * 1024;
#pragma unroll
        for (int j = 0; j < NA; ++j)
            if (BM >= 64 || wave < 2)
                ISR_GLOBAL_TO_LDS16_AT(wsrc + (size_t)(ADDR == F_TAP ? (dy * p.k + dx) * (p.Cin_p >> 5) + (c0 >> 5) : step) * p.Cout_pp * 64 + j * 4096, a + j * 4096);
        if constexpr (ADDR == F_FLAT) {
#pragma unroll
            for (int j = 0; j < NB; ++j) ISR_GLOBAL_TO_LDS16_AT(in + (boff[j] + (uint32_t)step * 128u), b + j * 4096);
        } else {
            bool real = true;
            uint32_t toff;
            if constexpr (ADDR == F_TAP) {
                toff = (uint32_t)(((dy * p.W + dx) * p.Cin_p + c0) * 4);
            } else {
                const int e = entry;
                if (step + 1 < nsteps) entry = p.ktab[(step + 1) * 8 + bc];
                dy = e >> 24; dx = (e >> 16) & 0xFF;
                toff = (uint32_t)(((dy * p.W + dx) * p.Cin_p + (e & 0xFFFF)) * 4);
                real = e >= 0;
            }
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const bool ok = (int)real & (int)((unsigned)(iy0[j] + dy) < (unsigned)p.H) & (int)((unsigned)(ix0[j] + dx) < (unsigned)p.W);
                const uint8_t *src = in + (boff[j] + toff);
                ISR_GLOBAL_TO_LDS16_AT(ok ? src : (const uint8_t *)p.zeros, b + j * 4096);
            }
            if constexpr (ADDR == F_TAP) {
                if (++dx == p.k) { dx = 0; if (++dy == p.k) { dy = 0; c0 += 32; } }
            }
        }
    };

    // one constant of the epilogue per thread: bias [BM], scale [BM]
    static_assert(2 * BM <= 256 && 8 * BM <= STAGE, "one constant a thread, into one stage");
    float bias_or_scale = 0.0f;
    if (tid < 2 * BM) {
        const int ch = ch0 + (tid < BM ? tid : tid - BM);
        bias_or_scale = (tid < BM ? p.bias : p.scale)[ch];
        if constexpr (PAIR) {
            consts[tid] = (tid < BM ? p.bias2 : p.scale2)[ch];
            consts[2 * BM + tid] = bias_or_scale;
        }
    }

    v16f acc[MT][NT];
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
    };
    clear();
    auto multiply = [&](int buf) {
        const int8_t *A = lds + buf * STAGE, *B = A + ASTAGE;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            v4i af[MT];
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                const int r = i * 32 + l32;
                af[i] = *(const v4i *)(A + r * 64 + (((2 * ks + half) ^ swz<4>(r)) << 4));
            }
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                const int r = (wave * NT + j) * 32 + l32, c = 4 * ks + 2 * half;
                const v4f x0 = *(const v4f *)(B + r * 128 + ((c ^ swz<8>(r)) << 4)), x1 = *(const v4f *)(B + r * 128 + (((c + 1) ^ swz<8>(r)) << 4));
                v4i part[3];
                split_bf16(x0, x1, part);
#pragma unroll
                for (int k = 2; k >= 0; --k)    // the small parts first
#pragma unroll
                    for (int i = 0; i < MT; ++i)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, af[i]), __builtin_bit_cast(v8bf, part[k]),
                                                                             acc[i][j], 0, 0, 0);
            }
        }
    };

    v16f other[PAIR ? MT : 1][PAIR ? NT : 1];   // PAIR: the residual
    const float *bs = consts + 2 * BM;          // bias, scale
    if constexpr (!PAIR) {
        issue(0, 0);
        for (int step = 0; step < nsteps; ++step) {
            wait_vmcnt<0>();
            lds_barrier();   // every wave's loads of this step landed; every wave is done reading the other buffer
            if (step + 1 < nsteps) issue(step + 1, (step + 1) & 1);
            multiply(step & 1);
        }
        float *idle = (float *)(lds + (nsteps & 1) * STAGE);   // the stage that the last step did not use
        if (tid < 2 * BM) idle[tid] = bias_or_scale;
        lds_barrier();
        bs = idle;
    } else {
        // the steps of both layers are one sequence; these layers have few, and wait for memory with one of them ahead
        const uint8_t *wsrc2 = (const uint8_t *)p.w2 + ((size_t)(ch0 + arow) * 64 + ac * 16), *in2 = (const uint8_t *)p.in2;
        const int steps2 = p.Cin2_p >> 5, all = steps2 + nsteps;
        auto fetch = [&](int s, int buf) {
            const uint32_t a = lds0 + buf * STAGE + wave * 1024, b = lds0 + buf * STAGE + ASTAGE + wave * 1024;
            const bool own = s >= steps2;
            const int step = own ? s - steps2 : s;
            const uint8_t *w = (own ? wsrc : wsrc2) + (size_t)step * p.Cout_pp * 64, *x = (own ? in : in2) + step * 128;
#pragma unroll
            for (int j = 0; j < NA; ++j) ISR_GLOBAL_TO_LDS16_AT(w + j * 4096, a + j * 4096);
#pragma unroll
            for (int j = 0; j < NB; ++j) ISR_GLOBAL_TO_LDS16_AT(x + (own ? boff[j] : boff2[j]), b + j * 4096);
        };
        fetch(0, 0);
        fetch(1, 1);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the constants are stored
        int buf = 0;
        for (int s = 0; s < all; ++s) {
            if (s + 1 < all) wait_vmcnt<NA + NB>();   // only the next step's loads may be in flight
            else wait_vmcnt<0>();
            lds_barrier();
            if (s + 2 < all) fetch(s + 2, buf == 0 ? 2 : buf - 1);
            multiply(buf);
            buf = buf == 2 ? 0 : buf + 1;
            if (s + 1 == steps2) {
                const float lo = p.relu2 ? 0.0f : -INFINITY;
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int j = 0; j < NT; ++j)
#pragma unroll
                        for (int g = 0; g < 4; ++g) {
                            const int ch = i * 32 + 16 * half + 4 * g;
                            const v4f bias = *(const v4f *)(consts + ch), scale = *(const v4f *)(consts + BM + ch);
#pragma unroll
                            for (int e = 0; e < 4; ++e) other[i][j][4 * g + e] = fmaxf((acc[i][j][4 * g + e] + bias[e]) * scale[e], lo);
                        }
                clear();
            }
        }
    }

    fconv_finish_tile<PAIR>(p, acc, other, bs, px0, ch0, wave, lane, 4);
}

// Workgroups of fpatch_kernel a CU: as many as LDS has room for, where registers allow (left to itself the compiler takes a few more than
// three or four of them leave: 256 copies of the fp32 ResNet-50 at 96 x 96 2206 instead of 2072 us).
template <int MT, int NL>
constexpr int fpatch_workgroups() {
    constexpr int fit = 160 * 1024 / (3 * 32 * MT * 64 + 3 * (32 * NL + 1) * 64);
    return MT == 4 || fit < 2 ? 2 : MT == 2 && fit > 3 ? 3 : fit > 4 ? 4 : fit;
}

// 3x3 layers of stride 1 with a border of one pixel: the nine taps of 128 consecutive pixels lie in one run of 130 + 2 W pixels.  The
// workgroup splits 32 channels of that run once into three planes of bfloat16 in LDS, from which all nine taps read their
// operands; tap by tap through fconv_kernel every pixel was fetched and split nine times, 44 instructions for 3 MT matrix instructions,
// which left the matrix unit idle for half of the time.  Taps outside the image read a row of zeros.  The weights
// of a tap come through three stages, two steps ahead; the next channels of the run are fetched into registers during the second to
// ninth tap.  Products are added in the order of fconv_kernel.  Where registers allow (maps of at most 31 pixels a row), the two small
// parts of the pixels have a sum of their own, whose roundings are too small to count: 12 us of 333 at 14 x 14 for up to a fifth
// of the error of the logits.  668 copies of ResNet-50's layers of 64 channels at
// 56 x 56, 128 at 28 x 28, 256 at 14 x 14, 512 at 7 x 7, tap by tap -> from the run: 600 -> 450, 464 -> 374, 410 -> 345, 387 -> 331 us
// (0.21 ms at the nominal rate of the matrix unit); 16 copies at 56 x 56: 27 -> 21 us.
template <int MT, int NL>   // NL: rows of 32 pixels of the run, 130 + 2 W <= 32 NL
__global__ __launch_bounds__(256, (fpatch_workgroups<MT, NL>())) void fpatch_kernel(const FConvParams p) {
    constexpr int BM = 32 * MT, BN = 128, NST = 3, ASTAGE = BM * 64, NA = (BM + 63) / 64, ZERO = 32 * NL, PLANE = (32 * NL + 1) * 64;
    __shared__ __attribute__((aligned(256))) int8_t wt[NST * ASTAGE];
    __shared__ __attribute__((aligned(256))) int8_t run[3 * PLANE];
    static_assert(sizeof(wt) + sizeof(run) <= 80 * 1024 && 2 * BM <= 256 && 8 * BM <= ASTAGE, "two workgroups a CU; the constants fit a stage");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int mtiles = p.Cout_pp / BM;
    const long nb = gridDim.x, per = nb >> 3, rem = nb & 7, xcd = blockIdx.x & 7;
    const long bid = xcd * per + (xcd < rem ? xcd : rem) + (blockIdx.x >> 3);   // as fconv_kernel
    const int ch0 = (int)(bid % mtiles) * BM;
    const int px0 = (int)(bid / mtiles) * BN;
    const uint32_t lds0 = lds_address(wt) + wave * 1024;
    const int nblk = p.Cin_p >> 5, arow = tid >> 2, ac = (tid & 3) ^ swz<4>(arow);
    const uint32_t wlane = (uint32_t)((ch0 + arow) * 64 + ac * 16);

    int ft = 0, fb = 0, fbuf = 0;   // tap, block of 32 channels and stage of the next weights to fetch
    auto weights = [&]() {
        if (fb >= nblk) return;
        const uint8_t *w = (const uint8_t *)p.w + (size_t)(ft * nblk + fb) * p.Cout_pp * 64;
#pragma unroll
        for (int j = 0; j < NA; ++j)
            if (BM >= 64 || wave < 2) ISR_GLOBAL_TO_LDS16_AT(w + (wlane + (uint32_t)(j * 4096)), lds0 + fbuf * ASTAGE + j * 4096);
        fbuf = fbuf == NST - 1 ? 0 : fbuf + 1;
        if (++ft == 9) { ft = 0; ++fb; }
    };
    // a thread's four channels of NL pixels of the run; pixels outside the tensor are never read from LDS
    const int rrow = tid >> 3, rc = tid & 7;
    v4f next[NL];
    auto fetch = [&](int blk) {
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            int n = px0 - p.W - 1 + rrow + 32 * j;
            n = n < 0 ? 0 : (n < p.npix ? n : p.npix - 1);
            next[j] = *(const v4f *)((const uint8_t *)p.in + ((uint32_t)n * (uint32_t)(p.Cin_p * 4) + (uint32_t)(blk * 128 + rc * 16)));
        }
    };
    auto store = [&]() {
        int8_t *dst = run + rrow * 64 + (((rc >> 1) ^ swz<4>(rrow)) << 4) + (rc & 1) * 8;
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            uint2 part[3];
            split_bf16_4(next[j], part);
#pragma unroll
            for (int k = 0; k < 3; ++k) *(uint2 *)(dst + k * PLANE + j * 2048) = part[k];
        }
    };
    float bias_or_scale = 0.0f;
    if (tid < 2 * BM) bias_or_scale = (tid < BM ? p.bias : p.scale)[ch0 + (tid < BM ? tid : tid - BM)];
    fetch(0);
    if (tid < 12) *(v4i *)(run + (tid >> 2) * PLANE + ZERO * 64 + (tid & 3) * 16) = v4i{0, 0, 0, 0};

    // the lane's pixel: which taps are inside the image
    const int P = px0 + wave * 32 + l32, n = P < p.npix ? P : p.npix - 1;
    const int x = n % p.W, y = n / p.W % p.H;
    const int centre = wave * 32 + l32 + p.W + 1;
    constexpr bool TWO = NL <= 6;
    v16f acc[MT][1], small[TWO ? MT : 1];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            acc[i][0][e] = 0.0f;
            if (TWO) small[TWO ? i : 0][e] = 0.0f;
        }

    store();
    weights();
    weights();
    int buf = 0;
    auto block = [&](int blk, auto not_last) {
        constexpr bool more = decltype(not_last)::value;
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            // what may be left of what this thread has issued since this step's weights: those of the next step, and the run's channels,
            // fetched in step 0
            if (tap == 8 && !more) wait_vmcnt<0>();
            else if ((tap == 1 || tap == 2) && more) wait_vmcnt<NA + NL>();
            else wait_vmcnt<NA>();
            lds_barrier();   // the run is stored (tap 0); every wave is done with the step before
            __builtin_amdgcn_sched_barrier(0);
            weights();
            if (tap == 0 && more) {
                asm volatile("" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
                fetch(blk + 1);
                asm volatile("" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
            }
            const int dy = tap / 3 - 1, dx = tap % 3 - 1;
            const bool ok = (unsigned)(y + dy) < (unsigned)p.H && (unsigned)(x + dx) < (unsigned)p.W;
            const int row = ok ? centre + dy * p.W + dx : ZERO;
            const int at = row * 64 + ((half ^ swz<4>(row)) << 4);
            const int8_t *A = wt + buf * ASTAGE;
            // The reads of the second half are issued before the last products of the first: they are complete at the next barrier
            // without a wait there (13 layers of one copy's fp32 ResNet-50, where nothing hides it, 325 -> 300 us).
            v4i af[2][MT], part[2][3];
            auto read = [&](int ks) {
#pragma unroll
                for (int k = 2; k >= 0; --k) part[ks][k] = *(const v4i *)(run + k * PLANE + (at ^ (32 * ks)));
#pragma unroll
                for (int i = 0; i < MT; ++i) {
                    const int r = i * 32 + l32;
                    af[ks][i] = *(const v4i *)(A + r * 64 + (((2 * ks + half) ^ swz<4>(r)) << 4));
                }
            };
            read(0);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int k = 2; k >= 0; --k) {
                    if (ks == 0 && k == 0) {
                        __builtin_amdgcn_sched_barrier(0);
                        read(1);
                        __builtin_amdgcn_sched_barrier(0);
                    }
#pragma unroll
                    for (int i = 0; i < MT; ++i) {
                        v16f &sum = TWO && k ? small[TWO ? i : 0] : acc[i][0];
                        sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, af[ks][i]), __builtin_bit_cast(v8bf, part[ks][k]), sum, 0, 0, 0);
                    }
                }
            buf = buf == NST - 1 ? 0 : buf + 1;
        }
        if (more) {
            lds_barrier();   // every wave has read the run
            store();
        }
    };
    for (int blk = 0; blk + 1 < nblk; ++blk) block(blk, std::true_type{});
    block(nblk - 1, std::false_type{});
    if constexpr (TWO)
#pragma unroll
        for (int i = 0; i < MT; ++i) acc[i][0] += small[i];
    lds_barrier();   // every wave has read its last step, whose stage may be the one that follows
    float *bs = (float *)wt;
    if (tid < 2 * BM) bs[tid] = bias_or_scale;
    lds_barrier();
    fconv_finish_tile<false>(p, acc, 0, bs, px0, ch0, wave, lane, 4);
}

// The same for inputs of an odd multiple of 16 channels (fpatch_kernel's steps are of 32): the run of 256 pixels, 16 channels of it, and the
// weights of all nine taps fit LDS together, so that the taps follow one another without a barrier.  Rows of LDS are 32 bytes, the two
// chunks of every other group of eight rows exchanged, which keeps the rows that are read together in different banks.  Through the table
// these layers were half of the fp32 nets on 32 x 32 images: largest launches of ResNet-110 on 1024 copies 421 -> 250 us, its
// certification at n = 10 000 45.9 -> 32.8 ms (three workgroups a CU; 35.1 with two), ResNet-20's at 20 000 17.1 -> 12.7.  Of few copies
// as well: certifications of ResNet-20 with 1 + 4, 1 + 100, 1 + 1000 copies 395 -> 325, 457 -> 367, 1189 -> 820 us, ResNet-110 with 1 + 4
// 1935 -> 1510.
template <int MT, int NL>   // 258 + 2 W <= 32 NL
__global__ __launch_bounds__(256, MT == 1 ? 3 : 2) void fpatch16_kernel(const FConvParams p) {
    constexpr int BM = 32 * MT, NT = 2, BN = 128 * NT, ROWS = 32 * NL, ZERO = ROWS, PLANE = (ROWS + 1) * 32, TAP = BM * 32;
    constexpr int NX = (4 * ROWS + 255) / 256, NW = (18 * BM + 255) / 256;   // chunks of pixels, of weights a thread
    __shared__ __attribute__((aligned(256))) int8_t wt[9 * TAP];
    __shared__ __attribute__((aligned(256))) int8_t run[3 * PLANE];
    __shared__ __attribute__((aligned(16))) float bs[2 * BM];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int mtiles = p.Cout_pp / BM;
    const long nb = gridDim.x, per = nb >> 3, rem = nb & 7, xcd = blockIdx.x & 7;
    const long bid = xcd * per + (xcd < rem ? xcd : rem) + (blockIdx.x >> 3);   // as fconv_kernel
    const int ch0 = (int)(bid % mtiles) * BM;
    const int px0 = (int)(bid / mtiles) * BN;
    const int nblk = p.Cin_p >> 4;
    auto place = [](int row, int chunk) { return row * 32 + ((chunk ^ (row >> 3 & 1)) << 4); };

    if (tid < 2 * BM) bs[tid] = (tid < BM ? p.bias : p.scale)[ch0 + (tid < BM ? tid : tid - BM)];
    if (tid < 6) *(v4i *)(run + (tid >> 1) * PLANE + ZERO * 32 + (tid & 1) * 16) = v4i{0, 0, 0, 0};
    int x[NT], y[NT], centre[NT];
    v16f acc[MT][NT], small[MT][NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int r = (wave * NT + j) * 32 + l32, n = px0 + r < p.npix ? px0 + r : p.npix - 1;
        x[j] = n % p.W;
        y[j] = n / p.W % p.H;
        centre[j] = r + p.W + 1;
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = small[i][j][e] = 0.0f;
    }
    for (int blk = 0; blk < nblk; ++blk) {
        v4f px[NX];
        v4i wv[NW];
#pragma unroll
        for (int j = 0; j < NX; ++j) {
            int n = px0 - p.W - 1 + ((tid + 256 * j) >> 2);
            n = n < 0 ? 0 : (n < p.npix ? n : p.npix - 1);
            px[j] = *(const v4f *)((const uint8_t *)p.in + ((uint32_t)n * (uint32_t)(p.Cin_p * 4) + (uint32_t)(blk * 64 + (tid & 3) * 16)));
        }
#pragma unroll
        for (int j = 0; j < NW; ++j) {
            int i = tid + 256 * j;
            if (i >= 18 * BM) i = 18 * BM - 1;
            const int row = (i >> 1) % BM, k16 = (i >> 1) / BM * nblk + blk;
            wv[j] = *(const v4i *)((const uint8_t *)p.w + ((size_t)(k16 >> 1) * p.Cout_pp + ch0 + row) * 64 + (k16 & 1) * 32 + (i & 1) * 16);
        }
        if (blk > 0) __syncthreads();   // every wave has read what this one replaces
#pragma unroll
        for (int j = 0; j < NX; ++j) {
            const int row = (tid + 256 * j) >> 2, c = tid & 3;
            uint2 part[3];
            split_bf16_4(px[j], part);
            if (row < ROWS)
#pragma unroll
                for (int k = 0; k < 3; ++k) *(uint2 *)(run + k * PLANE + place(row, c >> 1) + (c & 1) * 8) = part[k];
        }
#pragma unroll
        for (int j = 0; j < NW; ++j) {
            const int i = tid + 256 * j, row = (i >> 1) % BM;
            if (i < 18 * BM) *(v4i *)(wt + (i >> 1) / BM * TAP + place(row, i & 1)) = wv[j];
        }
        __syncthreads();
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            const int dy = tap / 3 - 1, dx = tap % 3 - 1;
            v4i af[MT], part[NT][3];
#pragma unroll
            for (int i = 0; i < MT; ++i) af[i] = *(const v4i *)(wt + tap * TAP + place(i * 32 + l32, half));
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                const bool ok = (unsigned)(y[j] + dy) < (unsigned)p.H && (unsigned)(x[j] + dx) < (unsigned)p.W;
                const int at = place(ok ? centre[j] + dy * p.W + dx : ZERO, half);
#pragma unroll
                for (int k = 0; k < 3; ++k) part[j][k] = *(const v4i *)(run + k * PLANE + at);
            }
#pragma unroll
            for (int k = 2; k >= 0; --k)
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int i = 0; i < MT; ++i) {
                        v16f &sum = k ? small[i][j] : acc[i][j];
                        sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, af[i]), __builtin_bit_cast(v8bf, part[j][k]), sum, 0, 0, 0);
                    }
        }
    }
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] += small[i][j];
    fconv_finish_tile<false>(p, acc, 0, bs, px0, ch0, wave, lane, 4);
}

// First layer (7x7, stride 2, border 3, 4 stored channels in, 64 out) with the 3x3 / 2 max pooling that alone reads it.  The layer's
// result is four times the pooled one, and writing it and reading it back took as long as all its products should; here it
// never leaves the registers.  A workgroup makes 4 pooled rows x 31 pooled columns: the 23 x 136 pixels that this takes are split
// once into three planes of bfloat16 in LDS; a wave computes 32 channels of 2 pooled rows, row of the layer by row, the 32
// even columns 2 px and the 32 odd ones 2 px - 1 of a row as one fragment each, with its weights in registers.  The right
// neighbour of a pooled pixel is the next lane's odd column.  A fragment's operand is two pixels (16 bytes) of one kernel row, eight
// taps of which the last has zero weights; the pairs of pixels of a row of LDS lie by parity, so that lanes, two pairs apart, read
// neighbouring places.  Eight taps of a row are four groups of products to add instead of three and a half, and each rounds; the small
// parts of the pixels, two thirds of the products, therefore have a sum of their own, whose roundings are too small to count.  224 x 224, the two / this one: 668 copies
// 1272 + 581 -> 800 us, 96 copies 188 + 84 -> 124, 16 copies 44 + 16 -> 27 (42, 7 and 2 us less with one sum).  Bound by the reads of the planes (3 KB for two
// matrix instructions a wave) and the products themselves (five rows for four).
constexpr int FS_ROWS = 2, FS_BAND = 4, FS_COLS = 31, FS_IN = 4 * FS_BAND + 7, FS_HALF = 34, FS_PITCH = 2 * FS_HALF * 16;
__global__ __launch_bounds__(256, 2) void fstem_pool_kernel(const FConvParams p, const int Hp, const int Wp, float *const out) {
    constexpr int PLANE = FS_IN * FS_PITCH;
    __shared__ __attribute__((aligned(256))) int8_t img[3 * PLANE];
    __shared__ __attribute__((aligned(16))) float consts[128];   // bias, scale
    static_assert(sizeof(img) + sizeof(consts) <= 80 * 1024, "two workgroups a CU");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int bands = (Hp + FS_BAND - 1) / FS_BAND, strips = (Wp + FS_COLS - 1) / FS_COLS;
    const int strip = blockIdx.x % strips, band = blockIdx.x / strips % bands, b = blockIdx.x / (strips * bands);
    const int py0 = band * FS_BAND, px0 = strip * FS_COLS;
    const float *in = p.in + (size_t)b * p.H * p.W * 4;

    const int mf = wave & 1, group = wave >> 1;
    v4i af[14];   // [kernel row][half of its eight taps]
#pragma unroll
    for (int s = 0; s < 14; ++s) af[s] = *(const v4i *)((const uint8_t *)p.w + ((s >> 1) * 64 + mf * 32 + l32) * 64 + (2 * (s & 1) + half) * 16);
    if (tid < 128) consts[tid] = tid < 64 ? p.bias[tid] : p.scale[tid - 64];
    // input pixel (4 py0 - 5 + r, 4 px0 - 5 + x) -> row r, pair x / 2; zeros outside the image
    constexpr int PIX = FS_IN * 4 * FS_HALF, PER = (PIX + 255) / 256;
    v4f v4[PER];
    auto place = [&](int j, int &r, int &x) {
        const int i = tid + 256 * j;
        r = i / (4 * FS_HALF);
        x = i % (4 * FS_HALF);
        return i < PIX;
    };
    auto inside = [&](int r, int x) { return (unsigned)(4 * py0 - 5 + r) < (unsigned)p.H && (unsigned)(4 * px0 - 5 + x) < (unsigned)p.W; };
#pragma unroll
    for (int j = 0; j < PER; ++j) {   // all on their way before the first is waited for
        int r, x;
        place(j, r, x);
        v4[j] = *(const v4f *)(in + (inside(r, x) ? (4 * py0 - 5 + r) * p.W + 4 * px0 - 5 + x : 0) * 4);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        int r, x;
        if (!place(j, r, x)) break;
        const bool ok = inside(r, x);
#pragma unroll
        for (int e = 0; e < 4; ++e) v4[j][e] = ok ? v4[j][e] : 0.0f;
        uint2 part[3];
        split_bf16_4(v4[j], part);
        const int q = x >> 1;
#pragma unroll
        for (int k = 0; k < 3; ++k) *(uint2 *)(img + k * PLANE + r * FS_PITCH + ((q & 1) * FS_HALF + (q >> 1)) * 16 + (x & 1) * 8) = part[k];
    }
    lds_barrier();

    const int py = py0 + group * FS_ROWS, px = px0 + l32;
    if (py >= Hp) return;
    // pairs of the odd column: 2 l + 2 ks + half, of the even one: one further
    const int8_t *odd = img + 4 * group * FS_ROWS * FS_PITCH + (half * FS_HALF + l32) * 16;
    const int8_t *even = img + 4 * group * FS_ROWS * FS_PITCH + (half ? l32 + 1 : FS_HALF + l32) * 16;
    const bool odd_ok = 2 * px - 1 >= 0 && 2 * px - 1 < p.Wo, store = l32 < FS_COLS && px < Wp;
    const int c0 = mf * 32 + 16 * half;
    const float lo = p.relu ? 0.0f : -INFINITY;
    float v[16];
#pragma unroll
    for (int i = 0; i < 2 * FS_ROWS + 1; ++i) {
        const int cy = 2 * py - 1 + i;
        float h[16];
        if ((unsigned)cy < (unsigned)p.Ho) {
            v16f ae, ao, se, so;   // sums of the leading parts, of the two small ones
#pragma unroll
            for (int e = 0; e < 16; ++e) ae[e] = ao[e] = se[e] = so[e] = 0.0f;
#pragma unroll
            for (int s = 0; s < 14; ++s) {
                const int at = (2 * i + (s >> 1)) * FS_PITCH + (s & 1) * 16;
#pragma unroll
                for (int k = 2; k >= 0; --k) {
                    const v4i xe = *(const v4i *)(even + k * PLANE + at), xo = *(const v4i *)(odd + k * PLANE + at);
                    v16f &e = k ? se : ae, &o = k ? so : ao;
                    e = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, af[s]), __builtin_bit_cast(v8bf, xe), e, 0, 0, 0);
                    o = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, af[s]), __builtin_bit_cast(v8bf, xo), o, 0, 0, 0);
                }
            }
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const v4f bias = *(const v4f *)(consts + c0 + 4 * g), scale = *(const v4f *)(consts + 64 + c0 + 4 * g);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float te = fmaxf(((ae[4 * g + e] + se[4 * g + e]) + bias[e]) * scale[e], lo);
                    const float to = odd_ok ? fmaxf(((ao[4 * g + e] + so[4 * g + e]) + bias[e]) * scale[e], lo) : -INFINITY;
                    // wave_shl:1 reads the next lane (the last one, which has none, makes no pixel)
                    const float right = __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(to), 0x130, 0xf, 0xf, true));
                    h[4 * g + e] = fmaxf(fmaxf(te, to), right);
                }
            }
        } else {
#pragma unroll
            for (int e = 0; e < 16; ++e) h[e] = -INFINITY;
        }
        // pooled row j takes rows 2 j, 2 j + 1, 2 j + 2 of these
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = i == 0 ? h[e] : fmaxf(v[e], h[e]);
        if (i > 0 && (i & 1) == 0) {
            const int y = py + i / 2 - 1;
            if (store && y < Hp)
#pragma unroll
                for (int g = 0; g < 4; ++g) *(v4f *)(out + (((size_t)b * Hp + y) * Wp + px) * 64 + c0 + 4 * g) = v4f{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = h[e];
        }
    }
}

// A closing 1x1 layer with its residual add, and the 1x1 layer that reads the sum, in one kernel.  Both are bound by memory, by
// nothing but the sum where channels are few, and the second one reads back what the first has just written; here a workgroup takes
// 32 NW pixels through both.  Its steps are of two kinds, each with weights and one tile of pixels by 32 channels in a stage of
// LDS: a step of the first layer (128 channels at a time, kept in registers), or 32 channels of the residual, which are added, stored,
// split in registers and multiplied with 32 columns of the second layer's weights.  So that a lane's sums are the operand that
// it would read from memory, row r of a first layer's fragment is the channel whose stored row has bits 2 and 4 of r exchanged.
// Every sum is taken in the order of the separate kernels: the results are the same to the bit.  The fp32 ResNet-50 on 668 copies:
// 38.2 us a copy with neither pairs nor this, 34.6 with pairs, 31.1 with both (each pair of layers: fexpand_wanted).
//
// Three stages.  Loads and stores end in order, so a step waits until only what was issued after its loads is left: the loads of
// the next step and the stores of the two steps before.  Pixels past the end repeat the last one and store the same values to
// the same place, so that the number of stores is always the same; tests/test_kernel_listing.py counts them in the machine code.
//
// PAIR: the residual is another 1x1 layer's result, as F_PAIR: its steps come before the first layer's, its sums stay in registers.
struct FExpandParams {
    const float *in, *res;       // [B][H][W][Cin], [npix][C]
    float *sum, *out;            // [npix][C], [npix][Cout]
    const uint16_t *w1, *w2;     // as FConvParams::w
    const float *bias1, *scale1, *bias2, *scale2;
    int32_t npix, Cin, C, relu1, add_relu, relu2;
    float ma, mb;
    const float *in0;            // PAIR: [B][H0][W0][Cin0]
    const uint16_t *w0;
    const float *bias0, *scale0;
    int32_t Cin0, relu0, Ho, Wo, H, W, stride, H0, W0, stride0;
};
template <int MT2, int NW, bool PAIR>
struct FExpandShape {
    static constexpr int MAXC = 128 * MT2 < 512 ? 512 : 128 * MT2;                                    // channels of the sum whose constants fit
    static constexpr int BN = 32 * NW, ASLOT = (MT2 > 4 ? MT2 : 4) * 2048, STAGE = ASLOT + BN * 128;
    static constexpr int LDS = 3 * STAGE + (PAIR ? 4 : 2) * MAXC * 4;
};
template <int MT2, int NW, bool PAIR>
__global__ __launch_bounds__(64 * NW, 2) void fexpand_kernel(const FExpandParams p) {
    typedef FExpandShape<MT2, NW, PAIR> Shape;
    constexpr int NT = 64 * NW, MT1 = 4, COUT = 32 * MT2, NST = 3, STAGE = Shape::STAGE, ASLOT = Shape::ASLOT;
    constexpr int NA1 = MT1 * 2048 / (NT * 16), NA2 = MT2 * 2048 / (NT * 16), NB = 4;   // direct-to-LDS loads per lane and step
    constexpr int L1 = NA1 + NB, L2 = NA2 + (PAIR ? 0 : NB), ST = 4;                    // loads of a step, stores of a step of the second kind
    constexpr int G1 = PAIR ? 2 : 4, G2 = PAIR || MT2 < 4 ? 2 : 4;                      // weight fragments at a time: registers are short
    static_assert(NA1 >= 1 && NA2 >= 1 && MT1 == 4, "whole loads; the waits below");
    __shared__ __attribute__((aligned(256))) int8_t lds[NST * STAGE];
    __shared__ __attribute__((aligned(16))) float c1[(PAIR ? 4 : 2) * Shape::MAXC];     // bias, scale; PAIR: those of the other layer behind them
    static_assert(sizeof(lds) + sizeof(c1) == Shape::LDS && 2 * COUT <= NT && 8 * COUT <= STAGE, "one constant of the second layer a thread, into one stage");

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const long nb = gridDim.x, per = nb >> 3, rem = nb & 7, xcd = blockIdx.x & 7;   // neighbouring tiles on one XCD, as above
    const long px0 = (xcd * per + (xcd < rem ? xcd : rem) + (blockIdx.x >> 3)) * Shape::BN;
    const uint32_t lds0 = lds_address(lds) + wave * 1024;

    const int brow = tid >> 3, bc = (tid & 7) ^ swz<8>(brow);
    const int arow = tid >> 2, ac = (tid & 3) ^ swz<4>(arow);
    const uint32_t wlane = (uint32_t)(arow * 64 + ac * 16);
    uint32_t row[NB], row0[PAIR ? NB : 1];   // the lane's pixels in the first layer's input; PAIR: how far from there in the other one's
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const long P = px0 + brow + NT / 8 * j;
        const int n = (int)(P < p.npix ? P : p.npix - 1);
        row[j] = (uint32_t)n;
        if constexpr (PAIR) {
            const int hw = p.Ho * p.Wo, b = n / hw, r = n - b * hw, oy = r / p.Wo, ox = r - oy * p.Wo;
            row[j] = (uint32_t)((b * p.H + oy * p.stride) * p.W + ox * p.stride);
            row0[j] = (uint32_t)((b * p.H0 + oy * p.stride0) * p.W0 + ox * p.stride0) - row[j];
        }
    }
    for (int i = tid; i < 2 * p.C; i += NT) {
        c1[i] = i < p.C ? p.bias1[i] : p.scale1[i - p.C];
        if constexpr (PAIR) c1[2 * p.C + i] = i < p.C ? p.bias0[i] : p.scale0[i - p.C];
    }
    float constant2 = 0.0f;
    if (tid < 2 * COUT) constant2 = tid < COUT ? p.bias2[tid] : p.scale2[tid - COUT];

    const int steps0 = PAIR ? p.Cin0 >> 5 : 0, steps1 = steps0 + (p.Cin >> 5), chunks = p.C >> 7;   // steps of the first kind: the other layer's, all
    int fc = 0, fs = 0, fbuf = 0;   // chunk, step in the chunk and stage of the next step to fetch
    auto fetch = [&]() {
        if (fc >= chunks) return;
        const uint32_t a = lds0 + fbuf * STAGE, b = a + ASLOT;
        const bool first = fs < steps1, own = fs >= steps0;
        const int step = own ? fs - steps0 : fs, block = fc * MT1 + fs - steps1;
        const uint8_t *w = (const uint8_t *)(first ? (own ? p.w1 : p.w0) : p.w2) + (first ? (size_t)(step * p.C + fc * 128) * 64 : (size_t)block * (COUT * 64));
        const uint8_t *x = (const uint8_t *)(first ? (own ? p.in : p.in0) : p.res) + (first ? step : block) * 128;
        const uint32_t stride = (uint32_t)(first ? (own ? p.Cin : p.Cin0) : p.C) * 4u, other = own ? 0u : 0xFFFFFFFFu;
#pragma unroll
        for (int j = 0; j < (NA1 > NA2 ? NA1 : NA2); ++j)
            if (j < (first ? NA1 : NA2)) ISR_GLOBAL_TO_LDS16_AT(w + (wlane + (uint32_t)(j * (NT * 16))), a + j * (NT * 16));
        if (first || !PAIR)
#pragma unroll
            for (int j = 0; j < NB; ++j) ISR_GLOBAL_TO_LDS16_AT(x + ((row[j] + (PAIR ? row0[PAIR ? j : 0] & other : 0u)) * stride + (uint32_t)(bc * 16)), b + j * (NT * 16));
        fbuf = fbuf == NST - 1 ? 0 : fbuf + 1;
        if (++fs == steps1 + MT1) { fs = 0; ++fc; }
    };

    v16f acc[MT1], acc2[MT2], res[PAIR ? MT1 : 1];
#pragma unroll
    for (int i = 0; i < MT2; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc2[i][e] = 0.0f;
    const long P = px0 + wave * 32 + l32, pix = P < p.npix ? P : p.npix - 1;
    const uint32_t sum = ((uint32_t)pix * (uint32_t)p.C + (uint32_t)(8 * half)) * 4u;   // bytes
    const int row1 = (l32 & 0x0B) | (l32 & 4) << 2 | (l32 & 16) >> 2;
    const float lo1 = p.relu1 ? 0.0f : -INFINITY, add_lo = p.add_relu ? 0.0f : -INFINITY, ma = p.ma, mb = p.mb;
    // the wave's 8 channels of K step ks of its pixels in a stage
    auto operand = [&](const int8_t *B, int ks, v4f &x0, v4f &x1) {
        const int r = wave * 32 + l32, c = 4 * ks + 2 * half;
        x0 = *(const v4f *)(B + r * 128 + ((c ^ swz<8>(r)) << 4));
        x1 = *(const v4f *)(B + r * 128 + (((c + 1) ^ swz<8>(r)) << 4));
    };
    auto weights = [&](const int8_t *A, int i, int r, int ks) { return *(const v4i *)(A + (i * 32 + r) * 64 + (((2 * ks + half) ^ swz<4>(r)) << 4)); };
    auto begin = [&]() {   // after the wait for this wave's loads of the step
        lds_barrier();
        __builtin_amdgcn_sched_barrier(0);
        fetch();
    };

    fetch();
    fetch();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the constants are stored
    int buf = 0;
    for (int c = 0; c < chunks; ++c) {
#pragma unroll
        for (int i = 0; i < MT1; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][e] = 0.0f;
        for (int s = 0; s < steps1; ++s) {
            if (s + 1 < steps1) {   // the step after is of the first kind; before steps 0 and 1 come two and one that store
                if (c == 0 || s >= 2) wait_vmcnt<L1>();
                else if (s == 0) wait_vmcnt<L1 + 2 * ST>();
                else wait_vmcnt<L1 + ST>();
            } else {
                if (c == 0 || s >= 2) wait_vmcnt<L2>();
                else wait_vmcnt<L2 + ST>();
            }
            begin();
            const int8_t *A = lds + buf * STAGE, *B = A + ASLOT;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                v4f x0, x1;
                operand(B, ks, x0, x1);
                v4i part[3];
                split_bf16(x0, x1, part);
#pragma unroll
                for (int m = 0; m < MT1; m += G1) {
                    v4i af[G1];
#pragma unroll
                    for (int q = 0; q < G1; ++q) af[q] = weights(A, m + q, row1, ks);
#pragma unroll
                    for (int k = 2; k >= 0; --k)
#pragma unroll
                        for (int q = 0; q < G1; ++q)
                            acc[m + q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, af[q]), __builtin_bit_cast(v8bf, part[k]), acc[m + q], 0, 0, 0);
                }
            }
            buf = buf == NST - 1 ? 0 : buf + 1;
            if (PAIR && s + 1 == steps0) {
                const float *bias = c1 + 2 * p.C + c * 128 + 8 * half, *scale = bias + p.C;
                const float lo = p.relu0 ? 0.0f : -INFINITY;
#pragma unroll
                for (int i = 0; i < MT1; ++i)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int ch = i * 32 + 16 * (g >> 1) + 4 * (g & 1);
                        const v4f b = *(const v4f *)(bias + ch), sc = *(const v4f *)(scale + ch);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            res[PAIR ? i : 0][4 * g + e] = fmaxf((acc[i][4 * g + e] + b[e]) * sc[e], lo);
                            acc[i][4 * g + e] = 0.0f;
                        }
                    }
            }
        }
#pragma unroll
        for (int i = 0; i < MT1; ++i) {
            if (i == 0) wait_vmcnt<L2>();
            else if (i == 1) wait_vmcnt<L2 + ST>();
            else if (i + 1 < MT1) wait_vmcnt<L2 + 2 * ST>();
            else if (c + 1 < chunks) wait_vmcnt<L1 + 2 * ST>();
            else wait_vmcnt<2 * ST>();
            begin();
            const int8_t *A = lds + buf * STAGE, *B = A + ASLOT;
            const float *bias = c1 + c * 128 + i * 32 + 8 * half, *scale = bias + p.C;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                v4f r[2], y[2];
                if constexpr (!PAIR) operand(B, ks, r[0], r[1]);
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    const v4f b = *(const v4f *)(bias + 16 * ks + 4 * g), sc = *(const v4f *)(scale + 16 * ks + 4 * g);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float t = fmaxf((acc[i][8 * ks + 4 * g + e] + b[e]) * sc[e], lo1);
                        y[g][e] = fmaxf(ma * t + mb * (PAIR ? res[PAIR ? i : 0][8 * ks + 4 * g + e] : r[g][e]), add_lo);
                    }
                    *(v4f *)((uint8_t *)(p.sum + c * 128 + i * 32 + 16 * ks + 4 * g) + sum) = y[g];
                }
                v4i part[3];
                split_bf16(y[0], y[1], part);
#pragma unroll
                for (int m = 0; m < MT2; m += G2) {
                    v4i af[G2];
#pragma unroll
                    for (int q = 0; q < G2; ++q) af[q] = weights(A, m + q, l32, ks);
#pragma unroll
                    for (int k = 2; k >= 0; --k)
#pragma unroll
                        for (int q = 0; q < G2; ++q)
                            acc2[m + q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, af[q]), __builtin_bit_cast(v8bf, part[k]), acc2[m + q], 0, 0, 0);
                }
            }
            asm volatile("" ::: "memory");           // the stores stay in their step: the waits count them
            __builtin_amdgcn_sched_barrier(0);
            buf = buf == NST - 1 ? 0 : buf + 1;
        }
    }
    lds_barrier();   // every wave has read its last step, nothing is on its way: the first stage takes the second layer's constants
    float *c2 = (float *)lds;
    if (tid < 2 * COUT) c2[tid] = constant2;
    lds_barrier();
    const float lo2 = p.relu2 ? 0.0f : -INFINITY;
    float *const out = p.out + pix * COUT + 16 * half;
#pragma unroll
    for (int i = 0; i < MT2; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const v4f b = *(const v4f *)(c2 + i * 32 + 16 * half + 4 * g), sc = *(const v4f *)(c2 + COUT + i * 32 + 16 * half + 4 * g);
            v4f t;
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] = fmaxf((acc2[i][4 * g + e] + b[e]) * sc[e], lo2);
            *(v4f *)(out + i * 32 + 4 * g) = t;
        }
}

__global__ __launch_bounds__(256) void fadd_kernel(const FAddParams p) {
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < p.n4; i += (long)gridDim.x * 256) {
        const v4f a = ((const v4f *)p.a)[i], b = ((const v4f *)p.b)[i];
        v4f o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            o[e] = p.ma * a[e] + p.mb * b[e];
            if (p.relu) o[e] = fmaxf(o[e], 0.0f);
        }
        ((v4f *)p.out)[i] = o;
    }
}

// One thread per (copy, output pixel, 4 channels): max over the in-bounds taps.
__global__ __launch_bounds__(256) void fmaxpool_kernel(const FPoolParams p) {
    const int c4n = p.Cp >> 2;
    const long total = (long)p.B * p.Ho * p.Wo * c4n;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long)gridDim.x * 256) {
        const int c4 = (int)(i % c4n);
        long r = i / c4n;
        const int ox = (int)(r % p.Wo);
        r /= p.Wo;
        const int oy = (int)(r % p.Ho), b = (int)(r / p.Ho);
        v4f best = {0.f, 0.f, 0.f, 0.f};
        bool any = false;
        for (int ky = 0; ky < p.k; ++ky) {
            const int iy = oy * p.stride - p.pad + ky;
            if (iy < 0 || iy >= p.H) continue;
            for (int kx = 0; kx < p.k; ++kx) {
                const int ix = ox * p.stride - p.pad + kx;
                if (ix < 0 || ix >= p.W) continue;
                const v4f q = *(const v4f *)(p.in + (((long)b * p.H + iy) * p.W + ix) * p.Cp + 4 * c4);
                if (!any) best = q;
                else
#pragma unroll
                    for (int e = 0; e < 4; ++e) best[e] = fmaxf(best[e], q[e]);
                any = true;
            }
        }
        *(v4f *)(p.out + (((long)b * p.Ho + oy) * p.Wo + ox) * p.Cp + 4 * c4) = best;
    }
}

// One thread per (copy, 4 channels): scale * sum over the H x W positions.
__global__ __launch_bounds__(256) void fgap_kernel(const FGapParams p) {
    const int c4n = p.Cp >> 2;
    const long total = (long)p.B * c4n;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long)gridDim.x * 256) {
        const int c4 = (int)(i % c4n);
        const long b = i / c4n;
        v4f s = {0.f, 0.f, 0.f, 0.f};
        const float *src = p.in + b * p.HW * p.Cp + 4 * c4;
        for (int j = 0; j < p.HW; ++j) {
            const v4f q = *(const v4f *)(src + (long)j * p.Cp);
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] += q[e];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] *= p.scale;
        *(v4f *)(p.out + b * p.Cp + 4 * c4) = s;
    }
}

// One wave per copy: the class with the largest logit (lowest index among equals) and its vote.
__global__ __launch_bounds__(64) void fvote_kernel(const FVoteParams p) {
    const int b = blockIdx.x, lane = threadIdx.x;
    const float *lg = p.logits + (long)b * p.stride;
    float best = 0.f;
    int arg = 0x7FFFFFFF;
    for (int c = lane; c < p.classes; c += 64) {
        const float v = lg[c];
        if (arg == 0x7FFFFFFF || v > best) { best = v; arg = c; }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const float ob = __shfl_xor(best, off);
        const int oa = __shfl_xor(arg, off);
        if (oa != 0x7FFFFFFF && (arg == 0x7FFFFFFF || ob > best || (ob == best && oa < arg))) { best = ob; arg = oa; }
    }
    if (lane == 0) {
        if (p.argmax) p.argmax[b] = arg;
        if (p.counts) atomicAdd(p.counts + arg, 1u);
    }
}

long grid_for(long items, long cap = 256L * 32) {
    long blocks = (items + 255) / 256;
    return blocks < 1 ? 1 : (blocks > cap ? cap : blocks);
}

}  // namespace

hipError_t launch_float_noise(const FloatNoiseParams &p, hipStream_t st) {
    if (p.count == 0) return hipSuccess;
    if (p.C < 1 || p.C > 3 || (p.W & 3) != 0 || !(p.sigma >= 0.0f)) return hipErrorInvalidValue;
    const long total = (long)p.H * (p.W >> 2) * p.count;
    set_kernel_name(p.quant ? "float_noise_kernel (rounded)" : "float_noise_kernel");
    hipLaunchKernelGGL(float_noise_kernel, dim3((unsigned)grid_for(total)), dim3(256), 0, st, p);
    return hipGetLastError();
}

int fconv_tile_m(int cout_p) { return cout_p <= 32 ? 32 : (cout_p <= 64 ? 64 : 128); }

template <int MT, int NT>
static hipError_t launch_fconv_tile(const FConvParams &p, hipStream_t st) {
    const long blocks = (((long)p.npix + 128 * NT - 1) / (128 * NT)) * (p.Cout_pp / (32 * MT));
    if (blocks > 0x7FFFFFFFL) return hipErrorInvalidValue;
    static const std::string name = "fconv_kernel<" + std::to_string(32 * MT) + " x " + std::to_string(128 * NT) + ">";
    set_kernel_name(name.c_str());
    const dim3 grid((unsigned)blocks), block(256);
    if (p.k == 1 && p.stride == 1 && p.pad == 0 && p.Cin_p % 32 == 0) hipLaunchKernelGGL((fconv_kernel<MT, NT, F_FLAT>), grid, block, 0, st, p);
    else if (p.Cin_p % 32 == 0) hipLaunchKernelGGL((fconv_kernel<MT, NT, F_TAP>), grid, block, 0, st, p);
    else hipLaunchKernelGGL((fconv_kernel<MT, NT, F_TABLE>), grid, block, 0, st, p);
    return hipGetLastError();
}

// Two 1x1 layers of one kernel (F_PAIR): the same output tensor, channels in whole steps, stored channels in whole tiles' runs.
bool fconv_pair_supported(const FConvParams &p, const FConvParams &q) {
    return p.k == 1 && q.k == 1 && p.pad == 0 && q.pad == 0 && p.Cin_p % 32 == 0 && q.Cin_p % 32 == 0 && p.Cout_p == q.Cout_p && p.Cout_pp == q.Cout_pp &&
           p.Ho == q.Ho && p.Wo == q.Wo && p.Cout_pp % 128 == 0;
}

// The one kernel has one tile, of 128 pixels by 128 channels; the two take smaller ones where the pixels are few.  It pays from as many
// tiles as half of the CUs.  fp32 ResNet-50, us of a run of 1, 4, 8, 16, 32, 64 copies:
//   always paired            896   940  1031  1282  1685  2551
//   from 96 tiles            869   920  1021  1284  1685  2553
//   from 192                 869   921  1020  1280  1685  2552
//   from 384                 869   925  1026  1290  1700  2560
//   never                    871   925  1027  1304  1739  2629
bool fconv_pair_wanted(const FConvParams &p) { return ((long)p.npix + 127) / 128 * (p.Cout_pp / 128) >= 128; }

static hipError_t launch_fconv_pair(const FConvParams &p, hipStream_t st) {
    if (p.k != 1 || p.pad != 0 || p.Cin_p % 32 || p.Cin2_p <= 0 || p.Cin2_p % 32 || p.Cout_pp % 128 || !p.w2 || !p.bias2 || !p.scale2 || p.stride < 1 ||
        p.stride2 < 1 || (p.Ho - 1) * p.stride >= p.H || (p.Wo - 1) * p.stride >= p.W || (p.Ho - 1) * p.stride2 >= p.H2 || (p.Wo - 1) * p.stride2 >= p.W2 ||
        (long)p.npix / ((long)p.Ho * p.Wo) * p.H2 * p.W2 * p.Cin2_p >= (1L << 30))
        return hipErrorInvalidValue;
    const long blocks = (((long)p.npix + 127) / 128) * (p.Cout_pp / 128);
    if (blocks > 0x7FFFFFFFL) return hipErrorInvalidValue;
    set_kernel_name("fconv_kernel<128 x 128, pair>");
    hipLaunchKernelGGL((fconv_kernel<4, 1, F_PAIR>), dim3((unsigned)blocks), dim3(256), 0, st, p);
    return hipGetLastError();
}

template <int MT>
static hipError_t launch_fpatch(const FConvParams &p, hipStream_t st) {
    const long blocks = (((long)p.npix + 127) / 128) * (p.Cout_pp / (32 * MT));
    if (blocks > 0x7FFFFFFFL || 130 + 2 * p.W > 256) return hipErrorInvalidValue;
    static const std::string name = "fpatch_kernel<" + std::to_string(32 * MT) + ">";
    set_kernel_name(name.c_str());
    const dim3 grid((unsigned)blocks), block(256);
    if (130 + 2 * p.W <= 160) hipLaunchKernelGGL((fpatch_kernel<MT, 5>), grid, block, 0, st, p);
    else if (130 + 2 * p.W <= 192) hipLaunchKernelGGL((fpatch_kernel<MT, 6>), grid, block, 0, st, p);
    else hipLaunchKernelGGL((fpatch_kernel<MT, 8>), grid, block, 0, st, p);
    return hipGetLastError();
}

template <int MT>
static hipError_t launch_fpatch16(const FConvParams &p, hipStream_t st) {
    const long blocks = (((long)p.npix + 255) / 256) * (p.Cout_pp / (32 * MT));
    if (blocks > 0x7FFFFFFFL || 258 + 2 * p.W > 352) return hipErrorInvalidValue;
    static const std::string name = "fpatch16_kernel<" + std::to_string(32 * MT) + ">";
    set_kernel_name(name.c_str());
    const dim3 grid((unsigned)blocks), block(256);
    if (258 + 2 * p.W <= 288) hipLaunchKernelGGL((fpatch16_kernel<MT, 9>), grid, block, 0, st, p);
    else hipLaunchKernelGGL((fpatch16_kernel<MT, 11>), grid, block, 0, st, p);
    return hipGetLastError();
}

hipError_t launch_fconv(const FConvParams &p, hipStream_t st) {
    if (p.npix <= 0) return hipSuccess;
    const int bm = fconv_tile_m(p.Cout_p);
    // 32-bit byte offsets inside the input tensor
    if (p.Kq <= 0 || (p.Kq & 7) || p.Cout_pp % bm != 0 || p.Cout_p > p.Cout_pp || (p.Cout_p & 15) || (p.Cin_p & 3) || !p.zeros ||
        (long)p.npix / ((long)p.Ho * p.Wo) * p.H * p.W * p.Cin_p >= (1L << 30))
        return hipErrorInvalidValue;
    if (p.in2) return launch_fconv_pair(p, st);
    // The largest tile (fewest bytes into LDS and fewest splits per multiply) that still gives every CU its two
    // workgroups; launches with few pixels take smaller ones.
    auto tiles = [&](int m, int n) { return (((long)p.npix + n - 1) / n) * (p.Cout_pp / m); };
    constexpr long FULL = 512;
    if (p.k == 3 && p.stride == 1 && p.pad == 1 && p.Cin_p % 32 == 0 && p.W <= 63 && p.Ho == p.H && p.Wo == p.W) {
        if (bm == 128 && tiles(128, 128) >= FULL) return launch_fpatch<4>(p, st);
        if (bm >= 64 && tiles(64, 128) >= FULL) return launch_fpatch<2>(p, st);
        return launch_fpatch<1>(p, st);
    }
    if (p.k == 3 && p.stride == 1 && p.pad == 1 && p.Cin_p % 32 == 16 && p.W <= 47 && p.Ho == p.H && p.Wo == p.W)
        return bm == 32 ? launch_fpatch16<1>(p, st) : launch_fpatch16<2>(p, st);
    if (bm == 128) {
        if (tiles(128, 256) >= FULL) return launch_fconv_tile<4, 2>(p, st);
        if (tiles(128, 128) >= FULL) return launch_fconv_tile<4, 1>(p, st);
    }
    if (bm >= 64) {
        if (tiles(64, 256) >= FULL) return launch_fconv_tile<2, 2>(p, st);
        if (tiles(64, 128) >= FULL) return launch_fconv_tile<2, 1>(p, st);
    }
    return tiles(32, 256) >= FULL ? launch_fconv_tile<1, 2>(p, st) : launch_fconv_tile<1, 1>(p, st);
}

// The first layer closes a block of whole 128-channel tiles (its add with a stored residual, or a paired layer), the second reads its sum.
bool fexpand_supported(const FConvParams &p, const FConvParams &q) {
    const bool one = p.k == 1 && p.pad == 0 && (p.stride == 1 || p.w2) && q.k == 1 && q.stride == 1 && q.pad == 0;
    const int cout = q.Cout_p;
    return one && p.Ho == q.Ho && p.Wo == q.Wo && p.Cin_p % 32 == 0 && p.Cin_p + (p.w2 ? p.Cin2_p : 0) >= 64 && p.Cin2_p % 32 == 0 && p.Cout_p == p.Cout_pp &&
           p.Cout_p % 128 == 0 && q.Cin_p == p.Cout_p && q.Cout_pp == cout && (cout == 64 || cout == 128 || (cout == 256 && !p.w2)) &&
           p.Cout_p <= (cout == 256 ? 1024 : 512);
}

template <int MT2, int NW, bool PAIR>
static hipError_t launch_fexpand_tile(const FExpandParams &p, hipStream_t st) {
    static_assert(FExpandShape<MT2, NW, PAIR>::LDS <= 160 * 1024 / (NW == 4 ? 2 : 1), "eight waves on a CU");
    static const std::string name = "fexpand_kernel<" + std::to_string(32 * MT2) + (PAIR ? ", pair>" : ">");
    set_kernel_name(name.c_str());
    hipLaunchKernelGGL((fexpand_kernel<MT2, NW, PAIR>), dim3((unsigned)(((long)p.npix + 32 * NW - 1) / (32 * NW))), dim3(64 * NW), 0, st, p);
    return hipGetLastError();
}

// Whether two layers that fexpand_supported takes run in one kernel, for this number of pixels.  A workgroup goes through all channels,
// so time goes by whole rounds: of 32768 pixels with four waves (one workgroup for each CU; the second one on a CU takes nearly as
// long again) and 65536 with eight.  One kernel where what a round leaves idle is less than what it gains.  us, one kernel / two, of
// ResNet-50's layers at 16, 32, 64, 96, 160, 668 copies:
//   56 x 56 pixels, 256 -> 64      28 /  49    63 /  83   111 / 175   168 / 268   266 / 424   1053 / 1623
//   28 x 28, 512 -> 128            42 /  31    46 /  60    76 / 100   112 / 141   155 / 231    608 /  933
//   28 x 28, 512 -> 256            67 /  40    74 /  67    87 / 120   171 / 178   203 / 273    785 / 1042
//   14 x 14, 1024 -> 256          157 /  33   158 /  46   165 /  81   165 / 105   176 / 151    459 /  581
//   pair, 56 x 56, 256 -> 64       34 /  47    62 /  82   111 / 145   153 / 240   244 / 389    999 / 1424
//   pair, 28 x 28, 512 -> 128      75 /  40    79 /  72   100 / 120   179 / 164   222 / 263    916 / 1013
bool fexpand_wanted(const FConvParams &e, const FConvParams &r) {
    const bool wide = r.Cout_p == 256;
    const long npix = e.npix, round = wide ? 65536 : 32768, rounds = (npix + round - 1) / round;
    const int gain = wide ? 133 : e.w2 ? (r.Cout_p == 64 ? 140 : 110) : 150;   // per cent
    return rounds * round * 100 <= npix * gain && npix * e.Cout_p < (1L << 30);
}

hipError_t launch_fexpand(const FConvParams &e, const FConvParams &r, hipStream_t st) {
    const long images = e.npix > 0 ? (long)e.npix / ((long)e.Ho * e.Wo) : 0;
    auto fits = [](long elements) { return elements < (1L << 30); };   // 32-bit byte offsets inside the tensors
    if (!fexpand_supported(e, r) || e.npix <= 0 || !e.in || !e.out || !r.out || r.in2 || r.res || !e.in2 != !e.w2 || !e.in2 == !e.res || !fits((long)e.npix * e.Cout_p) ||
        !fits(images * e.H * e.W * e.Cin_p) || e.stride < 1 || (e.Ho - 1) * e.stride >= e.H || (e.Wo - 1) * e.stride >= e.W ||
        (e.in2 && (!e.bias2 || !e.scale2 || e.Cin2_p <= 0 || e.stride2 < 1 || (e.Ho - 1) * e.stride2 >= e.H2 || (e.Wo - 1) * e.stride2 >= e.W2 ||
                   !fits(images * e.H2 * e.W2 * e.Cin2_p))))
        return hipErrorInvalidValue;
    const FExpandParams p{e.in, e.res, e.out, r.out, e.w, r.w, e.bias, e.scale, r.bias, r.scale, e.npix, e.Cin_p, e.Cout_p, e.relu, e.add_relu, r.relu, e.ma, e.mb,
                          e.in2, e.w2, e.bias2, e.scale2, e.Cin2_p, e.relu2, e.Ho, e.Wo, e.H, e.W, e.stride, e.H2, e.W2, e.stride2};
    if (e.in2) return r.Cout_p == 64 ? launch_fexpand_tile<2, 4, true>(p, st) : launch_fexpand_tile<4, 4, true>(p, st);
    if (r.Cout_p == 64) return launch_fexpand_tile<2, 4, false>(p, st);
    if (r.Cout_p == 128) return launch_fexpand_tile<4, 4, false>(p, st);
    return launch_fexpand_tile<8, 8, false>(p, st);
}

bool fstem_pool_supported(const FConvParams &p, const FPoolParams &q) {
    return p.k == 7 && p.stride == 2 && p.pad == 3 && p.Cin_p == 4 && p.Cout_p == 64 && p.Cout_pp == 64 && q.k == 3 && q.stride == 2 && q.pad == 1 && q.Cp == 64 &&
           q.H == p.Ho && q.W == p.Wo && p.Ho == (p.H - 1) / 2 + 1 && p.Wo == (p.W - 1) / 2 + 1 && q.Ho == (q.H - 1) / 2 + 1 && q.Wo == (q.W - 1) / 2 + 1;
}

hipError_t launch_fstem_pool(const FConvParams &p, const FPoolParams &q, hipStream_t st) {
    if (!fstem_pool_supported(p, q) || !p.in || !q.out || p.res || p.in2 || q.B <= 0) return hipErrorInvalidValue;
    const long blocks = (long)((q.Ho + FS_BAND - 1) / FS_BAND) * ((q.Wo + FS_COLS - 1) / FS_COLS) * q.B;
    if (blocks > 0x7FFFFFFFL) return hipErrorInvalidValue;
    set_kernel_name("fstem_pool_kernel");
    hipLaunchKernelGGL(fstem_pool_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p, q.Ho, q.Wo, q.out);
    return hipGetLastError();
}

hipError_t launch_fadd(const FAddParams &p, hipStream_t st) {
    if (p.n4 <= 0) return hipSuccess;
    set_kernel_name("fadd_kernel");
    hipLaunchKernelGGL(fadd_kernel, dim3((unsigned)grid_for(p.n4)), dim3(256), 0, st, p);
    return hipGetLastError();
}

hipError_t launch_fmaxpool(const FPoolParams &p, hipStream_t st) {
    if (p.B <= 0) return hipSuccess;
    if (p.Cp & 3) return hipErrorInvalidValue;
    set_kernel_name("fmaxpool_kernel");
    hipLaunchKernelGGL(fmaxpool_kernel, dim3((unsigned)grid_for((long)p.B * p.Ho * p.Wo * (p.Cp >> 2))), dim3(256), 0, st, p);
    return hipGetLastError();
}

hipError_t launch_fgap(const FGapParams &p, hipStream_t st) {
    if (p.B <= 0) return hipSuccess;
    if (p.Cp & 3) return hipErrorInvalidValue;
    set_kernel_name("fgap_kernel");
    hipLaunchKernelGGL(fgap_kernel, dim3((unsigned)grid_for((long)p.B * (p.Cp >> 2))), dim3(256), 0, st, p);
    return hipGetLastError();
}

hipError_t launch_fvote(const FVoteParams &p, hipStream_t st) {
    if (p.B <= 0) return hipSuccess;
    if (p.classes < 1) return hipErrorInvalidValue;
    set_kernel_name("fvote_kernel");
    hipLaunchKernelGGL(fvote_kernel, dim3((unsigned)p.B), dim3(64), 0, st, p);
    return hipGetLastError();
}

}  // namespace isr
