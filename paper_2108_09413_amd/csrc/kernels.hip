// Memory-bound stages of the Monte-Carlo loop: noise injection, residual add,
// pooling, the FC + argmax + vote tally.
#include "noise_device.h"

namespace isr {

typedef int v4i __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// Noise: x + delta, delta ~ discrete Gaussian (Def. 3.3), saturated to [0,255],
// recentred to int8, written as NHWC4 (4th channel 0).
//
// Randomness: Philox4x32-10 keyed by the seed; counter (p >> 2, sample, image,
// 2*phase + half) with p the logical [C][H][W] pixel index; word p & 3; half 0
// supplies the high 32 bits of the uniform 64-bit u, half 1 the low 32 bits.
// The low half is generated only when the high word ties with a threshold.

__global__ __launch_bounds__(256) void noise_kernel(const NoiseParams p) {
    __shared__ __attribute__((aligned(16))) NoiseLds t;
    // what this workgroup draws: one image, one table, a range of sample indices, a range of output copies
    const uint8_t *xim = p.x;
    const DeviceNoiseTable *tab = p.table;
    uint32_t image_id = p.image, sample_begin = p.sample_begin, count = p.count;
    long out_copy0 = 0;
    if (p.items) {   // batch mode: grid row = item; its slots that fall into this chunk
        const uint64_t item = (uint64_t)p.item_first + blockIdx.y;
        const uint64_t first = item * p.n_per_item, last = first + p.n_per_item, chunk_end = p.slot_begin + p.count;
        const uint64_t lo = first > p.slot_begin ? first : p.slot_begin, hi = last < chunk_end ? last : chunk_end;
        if (hi <= lo) return;   // uniform over the workgroup
        const NoiseItem it = p.items[item];
        xim = p.x + (size_t)it.image * p.C * p.H * p.W;
        tab = p.table + it.table_slot;
        image_id = it.image_id;
        sample_begin = (uint32_t)(lo - first);
        count = (uint32_t)(hi - lo);
        out_copy0 = (long)(lo - p.slot_begin);
    }
    store_noise_table(t, fetch_noise_table(tab, threadIdx.x), threadIdx.x);
    const NoiseSampler smp = tab->s;
    __syncthreads();

    const int W4 = p.W >> 2;
    const long groups_per_sample = (long)p.H * W4;
    const long total = groups_per_sample * count;
    for (long g = (long)blockIdx.x * 256 + threadIdx.x; g < total; g += (long)gridDim.x * 256) {
        const uint32_t s_local = (uint32_t)(g / groups_per_sample);
        const int rem = (int)(g - (long)s_local * groups_per_sample);
        const int y = rem / W4, x4 = rem - y * W4;
        const uint32_t sample = sample_begin + s_local;
        uint32_t packed[4];
        noisy_quad(t, smp, tab, xim, p.C, p.H, p.W, y, x4, sample, image_id, p.phase, p.key0, p.key1, packed);
        v4i o = {(int)packed[0], (int)packed[1], (int)packed[2], (int)packed[3]};
        *(v4i *)(p.out + ((out_copy0 + s_local) * groups_per_sample + rem) * 16) = o;
    }
}

hipError_t launch_noise(const NoiseParams &p, hipStream_t st) {
    if (p.count == 0) return hipSuccess;
    if (p.C < 1 || p.C > 3 || (p.W & 3) != 0) return hipErrorInvalidValue;
    unsigned rows = 1;
    uint32_t per_row = p.count;
    if (p.items) {
        if (p.n_per_item == 0 || p.item_count == 0 || p.item_count > 65535) return hipErrorInvalidValue;
        rows = p.item_count;
        if (p.n_per_item < per_row) per_row = p.n_per_item;
    }
    long total = (long)p.H * (p.W >> 2) * per_row;
    long blocks = (total + 255) / 256;
    const long cap = rows >= 4 ? 256 : 256 * 4;   // the table is staged into LDS once per workgroup
    if (blocks > cap) blocks = cap;
    set_kernel_name("noise_kernel");
    hipLaunchKernelGGL(noise_kernel, dim3((unsigned)blocks, rows), dim3(256), 0, st, p);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Noise bank: the discrete-Gaussian draws themselves (no image, no saturation), int16, for
// noise that is sampled ahead of training and stored.  Same generator and counter layout as
// above with the tensor index in the sample word, the bank id in the image word and phase 2.  The guide table (15 KB up
// to sigma 169, 57 KB at sigma 1024) is staged into LDS, except for small banks (launch_noise_bank); the thresholds stay in memory,
// for the few draws that it leaves open.
//
// Bound by the issue of the generator's and the sampler's integer arithmetic.  A draw is one LDS read and seven instructions up to
// its word t, two and a half from there on: the guide word (bank_guide) has |draw| left of its bucket's threshold on top of the
// threshold's 16 lowest float bits, so subtracting the draw's own bits borrows one where x lies behind the threshold and
// leaves zeros below where that is open; sign and packing go by halves of a register.  84 instructions per four draws instead of
// 113 with noise_draw4, which keeps to guides of half the size up to sigma 86: there is less to stage for workgroups that draw
// few pixels a thread (a net's first kernel on 32 x 32 images got 1 % slower with the words used here).
// WHOLE: tensors of whole waves (d a multiple of 256).  A wave's draws then lie in one tensor, and what depends on the tensor
// alone -- a quarter of the first two rounds of the generator, indices, addresses -- is scalar arithmetic.
// 50 000 x 3072 draws, calls in a row: 130 -> 108 us at sigma 32; one call alone 149 -> 121 at sigma 256, 148 -> 129 at 1000.

typedef short v2s __attribute__((ext_vector_type(2)));
__device__ __forceinline__ v2s upper_halves(uint32_t a, uint32_t b) { return __builtin_bit_cast(v2s, __builtin_amdgcn_perm(b, a, 0x07060302u)); }

// The four draws of the Philox block of counter (grp, c1, c2, c3), two to a register.
__device__ __forceinline__ void bank_draw4(const uint32_t *guide, const NoiseSampler &s, const uint32_t *thi, const uint32_t *tlo,
                                           uint32_t grp, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t key0, uint32_t key1, v2s (&d)[2]) {
    uint32_t u[4], t[4];
    philox4x32_10(grp, c1, c2, c3, key0, key1, u);
    auto bits_of = [&](int j) { return __float_as_uint(__builtin_amdgcn_fmed3f((float)(u[j] ^ (uint32_t)((int)u[j] >> 31)), s.lo, s.hi)); };
    auto word = [&](uint32_t bits) { return *(const uint32_t *)((const uint8_t *)guide + ((bits >> s.shift) & s.mask)); };
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t bits = bits_of(j);
        t[j] = word(bits) - (bits & 0xFFFF);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {   // with m = |draw| and r = -1 right of the centre, 0 left of it: r - (m ^ r)
        const v2s r = upper_halves(u[2 * j], u[2 * j + 1]) >> 15;
        d[j] = r - (upper_halves(t[2 * j], t[2 * j + 1]) ^ r);
    }
    const uint16_t low[4] = {(uint16_t)t[0], (uint16_t)t[1], (uint16_t)t[2], (uint16_t)t[3]};
    if (min(min(low[0], low[1]), min(low[2], low[3])) == 0) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (low[j] == 0)
                d[j >> 1][j & 1] = (short)noise_draw_slow(thi, tlo, s, u[j], s.reach - (word(bits_of(j)) >> 16), grp, c1, c2, c3, key0, key1, j);
    }
}

// WORDS == 0: the guide stays in memory (launch_noise_bank).
template <int WORDS, int THREADS, bool WHOLE>
__global__ __launch_bounds__(THREADS) void noise_bank_kernel(const NoiseBankParams p) {
    __shared__ __attribute__((aligned(16))) uint32_t staged[WORDS ? WORDS : 4];
    const uint32_t *const guide = WORDS ? staged : p.guide;
    if constexpr (WORDS != 0) {
        for (uint32_t i = threadIdx.x; i < p.guide_words / 4; i += THREADS) ((uint4 *)staged)[i] = ((const uint4 *)p.guide)[i];
        __syncthreads();
    }
    const uint32_t groups_per_tensor = p.d >> 2;
    auto draw = [&](uint32_t grp, uint32_t t) {
        v2s d[2];
        bank_draw4(guide, p.s, p.thi, p.tlo, grp, p.first + t, p.bank, 4u, p.key0, p.key1, d);
        return make_uint2(__builtin_bit_cast(uint32_t, d[0]), __builtin_bit_cast(uint32_t, d[1]));
    };
    if constexpr (WHOLE) {
        const uint32_t lane = threadIdx.x & 63, runs = groups_per_tensor >> 6;   // of 64 groups, one per wave and step
        const uint64_t total = (uint64_t)runs * p.count, step = (uint64_t)gridDim.x * (THREADS / 64);
        const uint32_t dt = (uint32_t)(step / runs), dr = (uint32_t)(step % runs);
        uint64_t q = (uint64_t)blockIdx.x * (THREADS / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        uint32_t t = (uint32_t)(q / runs), r = (uint32_t)(q - (uint64_t)t * runs);
        for (; q < total; q += step) {
            ((uint2 *)p.out + q * 64)[lane] = draw(r * 64 + lane, t);
            t += dt;
            r += dr;
            if (r >= runs) { r -= runs; ++t; }
        }
    } else {
        const uint64_t total = (uint64_t)groups_per_tensor * p.count, step = (uint64_t)gridDim.x * THREADS;
        const uint32_t dt = (uint32_t)(step / groups_per_tensor), dg = (uint32_t)(step % groups_per_tensor);
        uint64_t g = (uint64_t)blockIdx.x * THREADS;
        uint32_t t = (uint32_t)((g + threadIdx.x) / groups_per_tensor), grp = (uint32_t)(g + threadIdx.x - (uint64_t)t * groups_per_tensor);
        for (; g < total; g += step) {   // uniform
            const uint2 w = draw(grp, t);
            if (threadIdx.x < total - g) ((uint2 *)p.out + g)[threadIdx.x] = w;
            t += dt;
            grp += dg;
            if (grp >= groups_per_tensor) { grp -= groups_per_tensor; ++t; }
        }
    }
}

template <int WORDS, int THREADS>
static hipError_t launch_noise_bank_guide(const NoiseBankParams &p, hipStream_t st) {
    const uint64_t total = (uint64_t)(p.d >> 2) * p.count;
    uint64_t blocks = (total + THREADS - 1) / THREADS;
    if (blocks > 256 * (2048 / THREADS)) blocks = 256 * (2048 / THREADS);   // a full chip
    set_kernel_name("noise_bank_kernel");
    const dim3 grid((unsigned)blocks), block(THREADS);
    if (p.d % 256 == 0) hipLaunchKernelGGL((noise_bank_kernel<WORDS, THREADS, true>), grid, block, 0, st, p);
    else hipLaunchKernelGGL((noise_bank_kernel<WORDS, THREADS, false>), grid, block, 0, st, p);
    return hipGetLastError();
}

hipError_t launch_noise_bank(const NoiseBankParams &p, hipStream_t st) {
    if (p.count == 0) return hipSuccess;
    if (p.d == 0 || (p.d & 3) != 0 || p.s.reach < 1 || p.s.reach > 16384 || !p.thi || !p.tlo || !p.guide || !p.out) return hipErrorInvalidValue;
    if (p.guide_words * 4 <= (p.s.mask >> 1) || p.guide_words > 14336 || (p.guide_words & 3)) return hipErrorInvalidValue;   // the index's leading exponent bit is set for the largest x
    // Small banks: the guide is not staged.  A workgroup would wait for all of it to make one step, which reads a few lines of its upper
    // octaves.  From the second step of a thread on, with the large guides from half a step, those reads cost more.  us of a call, not
    // staged / staged:
    //   groups      40 k            130 k           237 k           521 k           768 k           1536 k
    //   sigma 32    16.42 / 16.70                   17.41 / 17.65   18.70 / 19.13   19.74 / 19.65   23.25 / 22.30
    //   sigma 300   16.51 / 17.15   16.98 / 17.40   17.57 / 17.71   19.08 / 18.94   20.28 / 19.70   24.04 / 22.25
    //   sigma 900   17.87 / 18.70   18.70 / 19.22   19.48 / 19.68   21.18 / 21.13   22.63 / 21.97   27.19 / 24.97
    if ((uint64_t)(p.d >> 2) * p.count <= 256 * (p.guide_words <= 3840 ? 2048 : 512)) return launch_noise_bank_guide<0, 256>(p, st);
    // the waves of a workgroup share a guide: large ones where eight workgroups' guides would not fit a CU
    if (p.guide_words <= 3840) return launch_noise_bank_guide<3840, 256>(p, st);
    if (p.guide_words <= 7680) return launch_noise_bank_guide<7680, 1024>(p, st);
    return launch_noise_bank_guide<14336, 1024>(p, st);
}

// ---------------------------------------------------------------------------
// Residual add of two int8 tensors with requantisation:
//   out = clamp(z_o + RHA((qa - za) Ma + (qb - zb) Mb, shift), relu ? z_o : -128, 127)

__device__ __forceinline__ int rha64(long v, int s) {
    if (s == 0) return (int)v;
    long half = 1L << (s - 1);
    return (int)(v >= 0 ? (v + half) >> s : -((-v + half) >> s));
}

__global__ __launch_bounds__(256) void add_kernel(const AddParams p) {
    const int lo = p.relu ? p.zo : -128;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < p.n16; i += (long)gridDim.x * 256) {
        v4i va = *(const v4i *)(p.a + i * 16), vb = *(const v4i *)(p.b + i * 16), vo;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            uint32_t packed = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                int qa = (int)(int8_t)((uint32_t)va[d] >> (8 * e));
                int qb = (int)(int8_t)((uint32_t)vb[d] >> (8 * e));
                long v = (long)(qa - p.za) * p.Ma + (long)(qb - p.zb) * p.Mb;
                int r = p.zo + rha64(v, p.sh);
                r = r < lo ? lo : (r > 127 ? 127 : r);
                packed |= (uint32_t)(r & 0xFF) << (8 * e);
            }
            vo[d] = (int)packed;
        }
        *(v4i *)(p.out + i * 16) = vo;
    }
}

hipError_t launch_add(const AddParams &p, hipStream_t st) {
    if (p.n16 <= 0) return hipSuccess;
    long blocks = (p.n16 + 255) / 256;
    if (blocks > 256 * 32) blocks = 256 * 32;
    set_kernel_name("add_kernel");
    hipLaunchKernelGGL(add_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Max pooling over in-bounds taps, NHWC, 16 channels per thread.

__global__ __launch_bounds__(256) void maxpool_kernel(const PoolParams p) {
    const int c16 = p.Cp >> 4;
    const long total = (long)p.B * p.Ho * p.Wo * c16;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long)gridDim.x * 256) {
        int cg = (int)(i % c16);
        long pix = i / c16;
        int ox = (int)(pix % p.Wo);
        long t = pix / p.Wo;
        int oy = (int)(t % p.Ho);
        long b = t / p.Ho;
        int best[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) best[e] = -128;
        for (int ky = 0; ky < p.k; ++ky) {
            int iy = oy * p.stride - p.pad + ky;
            if ((unsigned)iy >= (unsigned)p.H) continue;
            for (int kx = 0; kx < p.k; ++kx) {
                int ix = ox * p.stride - p.pad + kx;
                if ((unsigned)ix >= (unsigned)p.W) continue;
                v4i v = *(const v4i *)(p.in + ((b * p.H + iy) * p.W + ix) * p.Cp + cg * 16);
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    int q = (int)(int8_t)((uint32_t)v[e >> 2] >> (8 * (e & 3)));
                    best[e] = q > best[e] ? q : best[e];
                }
            }
        }
        v4i o;
#pragma unroll
        for (int d = 0; d < 4; ++d)
            o[d] = (int)((uint32_t)(best[4 * d] & 0xFF) | ((uint32_t)(best[4 * d + 1] & 0xFF) << 8) |
                         ((uint32_t)(best[4 * d + 2] & 0xFF) << 16) | ((uint32_t)best[4 * d + 3] << 24));
        *(v4i *)(p.out + pix * p.Cp + cg * 16) = o;
    }
}

hipError_t launch_maxpool(const PoolParams &p, hipStream_t st) {
    long total = (long)p.B * p.Ho * p.Wo * (p.Cp >> 4);
    if (total <= 0) return hipSuccess;
    long blocks = (total + 255) / 256;
    if (blocks > 256 * 32) blocks = 256 * 32;
    set_kernel_name("maxpool_kernel");
    hipLaunchKernelGGL(maxpool_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Global average pooling: S = sum over H*W of (q - z_in), requantised like a
// convolution output with a scalar (M0, shift); 4 channels per thread.

__global__ __launch_bounds__(256) void gap_kernel(const GapParams p) {
    const int c4 = p.Cp >> 2;
    const long total = (long)p.B * c4;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long)gridDim.x * 256) {
        int cg = (int)(i % c4);
        long b = i / c4;
        const int8_t *src = p.in + b * p.HW * p.Cp + cg * 4;
        int s[4] = {0, 0, 0, 0};
        // eight loads in flight: one at a time a launch of 100 copies of 7 x 7 x 2048 took 14.5 us
        for (int t0 = 0; t0 < p.HW; t0 += 8) {
            int v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = t0 + j < p.HW ? *(const int *)(src + (long)(t0 + j) * p.Cp) : 0;
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) s[e] = __builtin_amdgcn_sdot4(v[j], 1 << (8 * e), s[e], false);
        }
        uint32_t packed = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            long v = (long)(s[e] - p.HW * p.zp_in) * p.M0;
            int r = p.zp_out + rha64(v, 31 + p.sh);
            r = r < -128 ? -128 : (r > 127 ? 127 : r);
            packed |= (uint32_t)(r & 0xFF) << (8 * e);
        }
        *(uint32_t *)(p.out + b * p.Cp + cg * 4) = packed;
    }
}

hipError_t launch_gap(const GapParams &p, hipStream_t st) {
    long total = (long)p.B * (p.Cp >> 2);
    if (total <= 0) return hipSuccess;
    long blocks = (total + 255) / 256;
    if (blocks > 256 * 32) blocks = 256 * 32;
    set_kernel_name("gap_kernel");
    hipLaunchKernelGGL(gap_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// FC logits (int32, no requantisation), wavefront argmax (lowest index among
// maxima) and vote histogram: one wave per sample, LDS histogram per block,
// one global atomic per class per block.

constexpr int FC_MAX_CLASSES = 1024;

__global__ __launch_bounds__(256) void fc_vote_kernel(const FcParams p) {
    __shared__ uint32_t hist[2 * FC_MAX_CLASSES];   // single pair: the workgroup's votes of the two phases
    for (int i = threadIdx.x; i < 2 * p.classes; i += 256) hist[i] = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (long s = (long)blockIdx.x * 4 + wave; s < p.B; s += (long)gridDim.x * 4) {
        const int8_t *a = p.in + s * p.Kp;
        int best = INT32_MIN, best_idx = 0x7FFFFFFF;
        for (int c = lane; c < p.classes; c += 64) {
            // weights are stored [K / 16][classes_p][16]: the 64 classes of a pass read 1 KiB contiguous
            const int8_t *w = p.w + (long)c * 16;
            int acc = p.bias[c];
#pragma unroll 4
            for (int k = 0; k < p.Kp; k += 16) {
                v4i va = *(const v4i *)(a + k), vw = *(const v4i *)(w + (long)(k >> 4) * p.classes_p * 16);
#pragma unroll
                for (int d = 0; d < 4; ++d) acc = __builtin_amdgcn_sdot4(va[d], vw[d], acc, false);
            }
            if (p.logits) p.logits[s * p.classes + c] = acc;
            if (acc > best) { best = acc; best_idx = c; }   // ascending c keeps the lowest index
        }
        // wave reduction: larger logit wins, then the lower class index
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            int ob = __shfl_xor(best, off, 64), oi = __shfl_xor(best_idx, off, 64);
            if (ob > best || (ob == best && oi < best_idx)) { best = ob; best_idx = oi; }
        }
        if (lane == 0) {
            if (p.argmax) p.argmax[s] = best_idx;
            if (p.counts) {
                const uint32_t at = slot_use(p.slots, (uint64_t)s).row * p.classes + best_idx;
                atomicAdd(p.slots.pairs > 1 ? &p.counts[at] : &hist[at], 1u);
            }
        }
    }
    __syncthreads();
    if (p.counts && p.slots.pairs == 1)
        for (int i = threadIdx.x; i < 2 * p.classes; i += 256)
            if (hist[i]) atomicAdd(&p.counts[i], hist[i]);
}

// The same for long feature vectors, with the four waves of a workgroup on ONE sample: each wave
// sums a quarter of K for all classes (lane = class) with 16 independent weight loads in
// flight, the partial sums meet in LDS.  The one-wave form above waits for memory 128 times in
// a row at K = 2048.  Integer sums, so the order of the additions is free.
__global__ __launch_bounds__(256) void fc_vote_ksplit_kernel(const FcParams p) {
    __shared__ int part[4][FC_MAX_CLASSES];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int kq = p.Kp >> 2;                        // K bytes per wave, a multiple of 256
    for (long s = blockIdx.x; s < p.B; s += gridDim.x) {
        const int8_t *a = p.in + s * p.Kp + wave * kq;
        for (int c = lane; c < p.classes; c += 64) {
            const int8_t *w = p.w + ((long)(wave * kq >> 4) * p.classes_p + c) * 16;
            int acc = 0;
            for (int k0 = 0; k0 < kq; k0 += 256) {
                v4i vw[16];
#pragma unroll
                for (int j = 0; j < 16; ++j) vw[j] = *(const v4i *)(w + (long)((k0 >> 4) + j) * p.classes_p * 16);
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const v4i va = *(const v4i *)(a + k0 + 16 * j);
#pragma unroll
                    for (int d = 0; d < 4; ++d) acc = __builtin_amdgcn_sdot4(va[d], vw[j][d], acc, false);
                }
            }
            part[wave][c] = acc;
        }
        __syncthreads();
        if (wave == 0) {
            int best = INT32_MIN, best_idx = 0x7FFFFFFF;
            for (int c = lane; c < p.classes; c += 64) {
                const int acc = p.bias[c] + part[0][c] + part[1][c] + part[2][c] + part[3][c];
                if (p.logits) p.logits[s * p.classes + c] = acc;
                if (acc > best) { best = acc; best_idx = c; }   // ascending c keeps the lowest index
            }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                int ob = __shfl_xor(best, off, 64), oi = __shfl_xor(best_idx, off, 64);
                if (ob > best || (ob == best && oi < best_idx)) { best = ob; best_idx = oi; }
            }
            if (lane == 0) {
                if (p.argmax) p.argmax[s] = best_idx;
                if (p.counts) {
                    atomicAdd(&p.counts[(size_t)slot_use(p.slots, (uint64_t)s).row * p.classes + best_idx], 1u);
                }
            }
        }
        __syncthreads();   // part is free for the next sample
    }
}

hipError_t launch_fc(const FcParams &p, hipStream_t st) {
    if (p.B <= 0) return hipSuccess;
    if (p.classes < 1 || p.classes > FC_MAX_CLASSES || p.Kp % 16 != 0 || p.classes_p < p.classes || (p.counts && !valid_slots(p.slots))) return hipErrorInvalidValue;
    if (p.Kp % 1024 == 0) {
        long blocks = p.B;
        if (blocks > 256 * 16) blocks = 256 * 16;
        set_kernel_name("fc_vote_ksplit_kernel");
        hipLaunchKernelGGL(fc_vote_ksplit_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p);
        return hipGetLastError();
    }
    long blocks = ((long)p.B + 3) / 4;
    if (blocks > 256 * 8) blocks = 256 * 8;
    set_kernel_name("fc_vote_kernel");
    hipLaunchKernelGGL(fc_vote_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p);
    return hipGetLastError();
}

// Tallies to the host's pinned memory, and zeros in their place for the next call, then `seq` to `flag`: the host that watches it has
// them 4 to 5 us before the end of the stream is reported (api.cpp, publish).  Every store goes past the caches by its scope and is
// complete (vmcnt) before the workgroup's barrier, so the flag is the last to arrive without a write-back of the L2.  2560 tallies
// are the most that were measured, by one workgroup in ten turns (256 pairs of 10 classes 266 -> 261 us a call).
__global__ __launch_bounds__(256) void publish_kernel(uint32_t *counts, uint32_t *host, uint32_t n, uint32_t *flag, uint32_t seq) {
    for (uint32_t i = threadIdx.x; i < n; i += 256) {
        __hip_atomic_store(&host[i], counts[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&counts[i], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(flag, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// the same for many tallies, whose host waits for the stream
__global__ void publish_many_kernel(uint32_t *counts, uint32_t *host, size_t n) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        host[i] = counts[i];
        counts[i] = 0;
    }
}

hipError_t launch_publish(uint32_t *counts, uint32_t *host, size_t n, uint32_t *flag, uint32_t seq, hipStream_t st) {
    if (n == 0) return hipErrorInvalidValue;
    if (flag) {
        if (n > PUBLISH_WATCHED) return hipErrorInvalidValue;
        hipLaunchKernelGGL(publish_kernel, dim3(1), dim3(256), 0, st, counts, host, (uint32_t)n, flag, seq);
    } else {
        size_t blocks = (n + 255) / 256;
        if (blocks > 1024) blocks = 1024;
        hipLaunchKernelGGL(publish_many_kernel, dim3((unsigned)blocks), dim3(256), 0, st, counts, host, n);
    }
    return hipGetLastError();
}

__global__ void fill_u32_kernel(uint32_t *p, uint32_t v, size_t n) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) p[i] = v;
}

hipError_t launch_fill_u32(uint32_t *p, uint32_t value, size_t n, hipStream_t st) {
    if (n == 0) return hipSuccess;
    size_t blocks = (n + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p, value, n);
    return hipGetLastError();
}

}  // namespace isr
