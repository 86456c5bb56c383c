// The device sampler of the noise stage, shared by the kernels that draw noisy pixels:
//   x + delta, delta ~ discrete Gaussian (Def. 3.3), saturated to [0,255], recentred to int8.
// Randomness: Philox4x32-10 keyed by the seed; counter (p >> 2, sample, image, 2*phase + half)
// with p the logical [C][H][W] pixel index; word p & 3; half 0 supplies the high 32 bits of the
// uniform 64-bit u, half 1 the low 32 bits.  The low half is generated only when the high word
// ties with a threshold.
#ifndef ISR_NOISE_DEVICE_H
#define ISR_NOISE_DEVICE_H

#include "isr_internal.h"

namespace isr {

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) { return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96); }

__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t out[4]) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        uint64_t p0 = (uint64_t)0xD2511F53u * c0;   // one 32x32->64 multiply gives both halves
        uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
        c0 = r == 0 ? (uint32_t)(p1 >> 32) ^ c1 ^ k0   // scalar where image and sample are uniform
                    : xor3((uint32_t)(p1 >> 32), c1, k0);
        c1 = (uint32_t)p1;
        c2 = xor3((uint32_t)(p0 >> 32), c3, k1);
        c3 = (uint32_t)p0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// The draw of a high word u that the guide word does not decide: x = u or ~u meets threshold `base`, or lies below all buckets
// (thresholds 0 .. base there).  Binary search for the first high word not below x, then the low words.
__device__ __noinline__ int noise_draw_slow(const uint32_t *thi, const uint32_t *tlo, const NoiseSampler &s, uint32_t u, uint32_t base,
                                            uint32_t grp, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t key0, uint32_t key1, int word) {
    const bool right = (int)u < 0;
    const uint32_t x = right ? ~u : u;
    uint32_t a = (float)x <= s.lo ? 0 : base, e = base + 1;
    if (e > s.reach) e = s.reach;
    while (a < e) {
        const uint32_t mid = (a + e) >> 1;
        if (thi[mid] < x) a = mid + 1; else e = mid;
    }
    if (a < s.reach && thi[a] == x) {
        uint32_t lo4[4];
        philox4x32_10(grp, c1, c2, c3 + 1, key0, key1, lo4);
        uint32_t ulo = lo4[0];
        if (word == 1) ulo = lo4[1];
        if (word == 2) ulo = lo4[2];
        if (word == 3) ulo = lo4[3];
        if (right) ulo = ~ulo;
        // left of the centre a threshold equal to u counts, the mirrored one of the right does not
        while (a < s.reach && thi[a] == x && (right ? tlo[a] < ulo : tlo[a] <= ulo)) ++a;
    }
    const int d = (int)a - (int)s.reach;
    return right ? -d : d;
}

// The four draws of the Philox block of counter (grp, c1, c2, c3).  A draw is one LDS read and about a dozen instructions: the
// difference of its guide word and its own mantissa bits tells by the sign on which side of the bucket's threshold it lies,
// and by a small value that this is open.
__device__ __forceinline__ void noise_draw4(const uint32_t *guide, const NoiseSampler &s, const uint32_t *thi, const uint32_t *tlo,
                                            uint32_t grp, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t key0, uint32_t key1, int (&d)[4]) {
    uint32_t u[4], t[4], e[4];
    philox4x32_10(grp, c1, c2, c3, key0, key1, u);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int right = (int)u[j] >> 31;
        const uint32_t bits = __float_as_uint(__builtin_amdgcn_fmed3f((float)(u[j] ^ (uint32_t)right), s.lo, s.hi));
        e[j] = *(const uint32_t *)((const uint8_t *)guide + ((bits >> s.shift) & s.mask));
        t[j] = e[j] - (bits << s.key_shift);
        const int m = (int)(e[j] & NOISE_DRAW_MASK) + ((int)t[j] >> 31);   // |draw|
        d[j] = right - (m ^ right);
    }
    if (min(min(t[0], t[1]), min(t[2], t[3])) <= NOISE_DRAW_MASK) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (t[j] <= NOISE_DRAW_MASK)
                d[j] = noise_draw_slow(thi, tlo, s, u[j], s.reach - (e[j] & NOISE_DRAW_MASK), grp, c1, c2, c3, key0, key1, j);
    }
}

struct NoiseLds {
    uint32_t guide[NOISE_GUIDE_MAX];
};

// A workgroup of NT threads stages a table into LDS: the loads, and later the stores (followed by a barrier at the caller).
template <int NT>
struct NoiseStage {
    static constexpr int N = NOISE_GUIDE_MAX / 4, LOADS = (N + NT - 1) / NT;
    uint4 v[LOADS];
};
template <int NT = 256>
__device__ __forceinline__ NoiseStage<NT> fetch_noise_table(const DeviceNoiseTable *tab, int tid) {
    typedef NoiseStage<NT> Stage;
    const uint4 *src = (const uint4 *)tab->guide;
    Stage s;
#pragma unroll
    for (int j = 0; j < Stage::LOADS; ++j) s.v[j] = src[tid + j * NT < Stage::N ? tid + j * NT : 0];
    return s;
}
template <int NT = 256>
__device__ __forceinline__ void store_noise_table(NoiseLds &t, const NoiseStage<NT> &s, int tid) {
    typedef NoiseStage<NT> Stage;
#pragma unroll
    for (int j = 0; j < Stage::LOADS; ++j)
        if (tid + j * NT < Stage::N) ((uint4 *)t.guide)[tid + j * NT] = s.v[j];
}

// Channel values of four horizontally adjacent noisy pixels, not yet saturated: x + delta of logical elements pix .. pix + 3; 128
// where the image lacks the channel, so that it holds 0 after the recentring.
__device__ __forceinline__ void noisy_sums(const NoiseLds &t, const NoiseSampler &s, const DeviceNoiseTable *tab, const uint8_t *xim, bool there,
                                           uint32_t pix, uint32_t sample, uint32_t image_id, uint32_t phase, uint32_t key0, uint32_t key1, int (&v)[4]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = 128;
    if (there) {
        const uint32_t px4 = *(const uint32_t *)(xim + pix);   // pix is a multiple of 4
        noise_draw4(t.guide, s, tab->hi, tab->lo, pix >> 2, sample, image_id, phase * 2u, key0, key1, v);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] += (int)((px4 >> (8 * j)) & 0xFF);
    }
}
// the same as int8 codes: clamp(x + delta, 0, 255) - 128
__device__ __forceinline__ void noisy_values(const NoiseLds &t, const NoiseSampler &s, const DeviceNoiseTable *tab, const uint8_t *xim, bool there,
                                             uint32_t pix, uint32_t sample, uint32_t image_id, uint32_t phase, uint32_t key0, uint32_t key1, int (&v)[4]) {
    noisy_sums(t, s, tab, xim, there, pix, sample, image_id, phase, key0, key1, v);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = min(max(v[j], 0), 255) - 128;
}

// Four horizontally adjacent noisy pixels (x4 * 4 .. x4 * 4 + 3 of row y) of one copy as NHWC4 words:
// byte c of word j = clamp(x[c][y][4 x4 + j] + delta, 0, 255) - 128, byte 3 = 0.
__device__ __forceinline__ void noisy_quad(const NoiseLds &t, const NoiseSampler &s, const DeviceNoiseTable *tab, const uint8_t *xim, int C, int H,
                                           int W, int y, int x4, uint32_t sample, uint32_t image_id, uint32_t phase, uint32_t key0,
                                           uint32_t key1, uint32_t packed[4]) {
    int v[3][4];
#pragma unroll
    for (int c = 0; c < 3; ++c)
        noisy_sums(t, s, tab, xim, c < C, (uint32_t)((c * H + y) * W + x4 * 4), sample, image_id, phase, key0, key1, v[c]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {   // saturation of two 16-bit values to bytes at once
        uint32_t lo = __builtin_amdgcn_perm((uint32_t)v[1][j], (uint32_t)v[0][j], 0x05040100u), hi = (uint32_t)v[2][j];
        asm("v_sat_pk_u8_i16 %0, %1" : "=v"(lo) : "v"(lo));
        asm("v_sat_pk_u8_i16 %0, %1" : "=v"(hi) : "v"(hi));
        packed[j] = ((hi << 16) | lo) ^ 0x00808080u;
    }
}

__device__ __forceinline__ SlotUse resolve_noise_source(const NoiseSource &s, long copy, const uint8_t *&xim,
                                                        const DeviceNoiseTable *&tab, uint32_t &image_id) {
    const SlotUse use = slot_use(s.slots, (uint64_t)copy);
    xim = s.x; tab = s.table; image_id = s.image;
    if (s.items) {
        const NoiseItem it = s.items[use.pair];
        xim = s.x + (size_t)it.image * s.C * s.H * s.W;
        tab = s.table + it.table_slot;
        image_id = it.image_id;
    }
    return use;
}

}  // namespace isr

#endif
