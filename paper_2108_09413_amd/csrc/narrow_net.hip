// The nets on 32 x 32 images (stages of 16 channels at 32 x 32, 32 at 16 x 16, 64 at 8 x 8 pixels), one launch per stage:
//   [first layer: noise draws + 3x3 convolution into 16 channels]   stage 16 only; else the stage's input is loaded
//   identity blocks  t = conv3x3(x), x = add(conv3x3(t), x)         any number
//   [down-sampling block into the next stage, or its first convolution alone]
//   [global average pooling, fully connected layer, argmax, vote]
// A workgroup of four waves keeps NI whole images in LDS from the first of these to the last: x and t as (S+2) x (S+2) x C
// int8 tiles whose border holds the tensor's zero-point, so that taps need no bounds checks and contribute 0.  The sum of
// a block replaces x in place (a lane reads the residual at its own pixel and writes there; the second convolution
// reads only t).  Memory sees the noise table, the stage's result and the weights (L2-resident, a few KiB a convolution).
//
// The 16 K-bytes of an MFMA operand lane are 16 channels of one tap = one aligned 128-bit LDS read at a tap-shifted
// address.  Bank conflicts: the LDS serves such a read 16 lanes at a time from 64 banks; 16 lanes are 16 pixels of a row
// (C = 16, 32) or 8 pixels of two rows (C = 64), C bytes apart, and would meet 2 (4) times in a bank at 32 (64) channels.
// Chunk c of the pixel at padded (y, x) therefore sits at chunk c ^ s, with s = x / 8 mod 2 at 32 channels and
// (x / 4 mod 2) + 2 (y mod 2) at 64: pixels of one row that share a residue mod 8 (4) then differ in s, and so do the two
// rows.  Per kernel column one base address (two at 64 channels, for the row parity) is kept in a register; rows and
// fragments are immediate offsets.
//
// What bounds it: issue of the requantisation arithmetic, the matrix unit and the LDS reads of the pixel operands, all three
// within a factor of two of each other (cycles of a CU per image and block at 16 / 32 / 64 channels: arithmetic
// 2660 / 1330 / 660, MFMA 1540 / 1150 / 1150, LDS reads 1620 / 1280 / 1280).  Workgroups per CU: four at 16 channels, three
// at 32 and 64 (LDS); more images per workgroup amortise the weight and constant loads of a convolution at 32 and 64
// channels, where a wave has one or two fragments per image.  Launches with few images take one image per workgroup:
// they are bound by the serial chain of convolutions, not by throughput.
#include <string>

#include "conv_device.h"
#include "noise_device.h"

namespace isr {

namespace {

typedef int v4acc __attribute__((ext_vector_type(4)));

// chunk position of the pixel at padded (y, x)
template <int C>
__device__ __forceinline__ int tile_swz(int y, int x) {
    return C == 64 ? (((x >> 2) & 1) | ((y & 1) << 1)) : C == 32 ? ((x >> 3) & 1) : 0;
}
template <int C, int S>
__device__ __forceinline__ int tile_at(int y, int x, int chunk) { return ((y * (S + 2) + x) * (C / 16) + (chunk ^ tile_swz<C>(y, x))) * 16; }
template <int C, int S>
constexpr int tile_bytes() { return (S + 2) * (S + 2) * C; }

// this wave's LDS operations are complete, then the workgroup's barrier; loads from memory stay in flight
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// border pixel b of a padded (S+2) x (S+2) tile: top row, bottom row, left and right columns without the corners
template <int S>
__device__ __forceinline__ void border_pixel(int b, int &y, int &x) {
    constexpr int P = S + 2;
    if (b < P) { y = 0; x = b; }
    else if (b < 2 * P) { y = P - 1; x = b - P; }
    else if (b < 3 * P - 2) { y = b - 2 * P + 1; x = 0; }
    else { y = b - (3 * P - 2) + 1; x = P - 1; }
}
template <int C, int S, int NI>
__device__ __forceinline__ void fill_ring(int8_t *tile, int zp, int tid) {
    constexpr int CH = C / 16, N = (4 * (S + 2) - 4) * CH;
    const int z = (int)((uint32_t)(zp & 0xFF) * 0x01010101u);
    for (int i = tid; i < NI * N; i += 256) {
        const int im = i / N, j = i % N;
        int y, x;
        border_pixel<S>(j / CH, y, x);
        *(v4i *)(tile + im * tile_bytes<C, S>() + ((y * (S + 2) + x) * CH + j % CH) * 16) = v4i{z, z, z, z};   // every chunk of the pixel: order is free
    }
}

// One lane's view of a 3x3 convolution over tiles of 32 or 64 channels: K steps of 32 bytes, 32-pixel fragments
// (2 rows of 16 or 4 rows of 8 pixels).
template <int C, int S>
struct WideConv {
    static constexpr int P = S + 2, KS = 9 * C / 32, KP = (9 * C + 63) / 64 * 64, MF = C / 32, NF = S * S / 32;
    static constexpr int ROWS = 32 / S, FRAG = ROWS * P * C;   // rows of a fragment; bytes from one to the next
    int base[3][C == 64 ? 2 : 1];
    int out;                      // the lane's chunk of its own pixel (fragment 0) for M fragment mf
    int mf, half, l;

    __device__ __forceinline__ WideConv(int lane, int wave) {
        l = lane & 31; half = lane >> 5; mf = wave % MF;
        const int y = l / S, x = l % S;
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) {
            base[kx][0] = tile_at<C, S>(y, x + kx, half);
            if constexpr (C == 64) base[kx][1] = base[kx][0] ^ 32;
        }
        out = tile_at<C, S>(y + 1, x + 1, 2 * mf + half);
    }
    __device__ __forceinline__ void load_weights(const int8_t *w, v4i (&fa)[KS]) const {
        const int8_t *row = w + (mf * 32 + l) * KP + half * 16;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) fa[ks] = *(const v4i *)(row + ks * 32);
    }
    __device__ __forceinline__ v16i run(const int8_t *frag, const v4i (&fa)[KS], v16i acc) const {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int tap = C == 64 ? ks >> 1 : ks, cc = C == 64 ? ks & 1 : 0, ky = tap / 3, kx = tap % 3;
            const v4i fb = *(const v4i *)(frag + base[kx][C == 64 ? (cc ^ (ky & 1)) : 0] + ky * P * C);
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[ks], fb, acc, 0, 0, 0);
        }
        return acc;
    }
};

// A lane's constants of N consecutive output channels from the packed form [4][C].  The top form keeps them in registers
// across the fragments of a convolution; the others, for the few layers that need them, read them where they are used.
template <int N, int RQ, bool TOP = RQ == RQ_TOP>
struct LaneConsts {
    int b[N], m0[N], chi, sh[N];
    __device__ __forceinline__ LaneConsts(const int *prm, int C, int c0) {
#pragma unroll
        for (int i = 0; i < N; ++i) { b[i] = prm[c0 + i]; m0[i] = prm[C + c0 + i]; sh[i] = prm[3 * C + c0 + i]; }
        chi = prm[2 * C + c0];
    }
    __device__ __forceinline__ void fragment() const {}   // start of a fragment
    __device__ __forceinline__ int bias(int i) const { return b[i]; }
    __device__ __forceinline__ int conv(int acc, int i, int lo) const { return rq_conv<RQ>(acc, m0[i], chi, sh[i], lo); }
};
template <int N, int RQ>
struct LaneConsts<N, RQ, false> {
    const int *at;
    int C;
    __device__ __forceinline__ LaneConsts(const int *prm, int C_, int c0) : at(prm + c0), C(C_) {}
    __device__ __forceinline__ void fragment() const { asm volatile("" ::: "memory"); }   // no constant is carried over in a register
    __device__ __forceinline__ int bias(int i) const { return at[i]; }
    __device__ __forceinline__ int conv(int acc, int i, int lo) const {
        return rq_conv<RQ>(acc, at[C + i], at[2 * C + (rq_is_top(RQ) ? 0 : i)], at[3 * C + i], lo);
    }
};
template <int N, int RQ>
__device__ __forceinline__ auto bias_vector(const LaneConsts<N, RQ> &k) {
    typedef int vec __attribute__((ext_vector_type(N)));
    vec v;
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = k.bias(i);
    return v;
}

// f with the compile-time forms of a descriptor's `form`; TOPA: the add's form next to RQ_TOP
template <int TOPA, class F>
__device__ __forceinline__ void with_form(int form, F f) {
    using std::integral_constant;
    if (form == 0) f(integral_constant<int, RQ_TOP>{}, integral_constant<int, TOPA>{});
    else if (form == 1) f(integral_constant<int, RQ_TOP_TIES>{}, integral_constant<int, RQ_ANY>{});
    else f(integral_constant<int, RQ_ANY>{}, integral_constant<int, RQ_ANY>{});
}

// Global average pooling of NI tiles, fully connected layer, argmax and votes.  `scratch` is LDS that nothing else uses.
template <int C, int S, int NI>
__device__ __forceinline__ void narrow_head(const NarrowParams &p, const int8_t *tile, int8_t *scratch, long img0, int tid) {
    constexpr int WORDS = C / 4, ITEMS = NI * WORDS, PARTS = 256 / ITEMS, PPP = S * S / PARTS;   // pixels per part
    static_assert(ITEMS <= 256 && 256 % ITEMS == 0 && S * S % PARTS == 0, "one part per thread");
    int *sums = (int *)scratch;                       // [NI][C]
    int8_t *feat = scratch + NI * C * 4;              // [NI][C]
    int *best_of = (int *)(feat + NI * C);            // [NI]
    const int lane = tid & 63, wave = tid >> 6;
    for (int i = tid; i < NI * C; i += 256) sums[i] = 0;
    lds_barrier();
    {
        const int item = tid % ITEMS, part = tid / ITEMS, im = item / WORDS, word = item % WORDS;
        const int8_t *t = tile + im * tile_bytes<C, S>();
        int s[4] = {0, 0, 0, 0};
        for (int i = 0; i < PPP; ++i) {
            const int pix = part * PPP + i;
            const uint32_t v = *(const uint32_t *)(t + tile_at<C, S>(pix / S + 1, pix % S + 1, word >> 2) + (word & 3) * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] += (int)(int8_t)(v >> (8 * e));
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) atomicAdd(&sums[im * C + word * 4 + e], s[e]);
    }
    lds_barrier();
    for (int i = tid; i < NI * C; i += 256) {
        // RHA of the scaled sum, as the pooling kernel
        const long v = (long)(sums[i] - S * S * p.gap_zp_in) * p.gap_M0;
        const int sh = 31 + p.gap_sh;
        const unsigned long mag = (unsigned long)(v < 0 ? -v : v);
        const long q = (long)((mag + (1ul << (sh - 1))) >> sh);
        const int r = p.gap_zp_out + (int)(v < 0 ? -q : q);
        feat[i] = (int8_t)(r < -128 ? -128 : (r > 127 ? 127 : r));
    }
    lds_barrier();
    for (int im = wave; im < NI; im += 4) {
        const long g = img0 + im;
        int best = INT32_MIN, best_idx = 0x7FFFFFFF;
        for (int c = lane; c < p.classes; c += 64) {
            int acc = p.fc_bias[c];
#pragma unroll
            for (int k = 0; k < C / 16; ++k) {
                const v4i vw = *(const v4i *)(p.fc_w + ((long)k * p.classes_p + c) * 16), va = *(const v4i *)(feat + im * C + k * 16);
#pragma unroll
                for (int d = 0; d < 4; ++d) acc = __builtin_amdgcn_sdot4(va[d], vw[d], acc, false);
            }
            if (p.logits && g < p.B) p.logits[g * p.classes + c] = acc;
            if (acc > best) { best = acc; best_idx = c; }   // ascending c keeps the lowest index
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const int ob = __shfl_xor(best, off, 64), oi = __shfl_xor(best_idx, off, 64);
            if (ob > best || (ob == best && oi < best_idx)) { best = ob; best_idx = oi; }
        }
        if (lane == 0) {
            if (p.argmax && g < p.B) p.argmax[g] = best_idx;
            best_of[im] = g < p.B ? best_idx : -1;
        }
    }
    if (!p.counts) return;
    lds_barrier();
    if (tid < NI && best_of[tid] >= 0) {
        // one global addition per distinct (row, class) of the workgroup, by its first image
        auto row = [&](int im) { return p.n_per_item ? (uint32_t)((p.slot_begin + (uint64_t)(img0 + im)) / p.n_per_item) : 0u; };
        const uint32_t r = row(tid);
        uint32_t n = 0;
        bool first = true;
        for (int im = 0; im < NI; ++im)
            if (best_of[im] == best_of[tid] && (im == tid || row(im) == r)) {
                ++n;
                first = first && im >= tid;
            }
        if (first) atomicAdd(&p.counts[(size_t)r * p.classes + best_of[tid]], n);
    }
}

template <int C, int S, int NI>
__global__ __launch_bounds__(256, C == 16 ? 4 : 3) void narrow_kernel(const NarrowParams p) {
    constexpr int P = S + 2, CH = C / 16, C2 = 2 * C, S2 = S / 2;
    constexpr int TB = tile_bytes<C, S>();
    constexpr bool TAIL = C < 64;                    // there is a next stage
    static_assert((C == 16 && S == 32 && NI == 1) || (C == 32 && S == 16) || (C == 64 && S == 8), "shape");
    __shared__ __attribute__((aligned(256))) int8_t X[NI * TB];
    __shared__ __attribute__((aligned(256))) int8_t T[NI * TB];
    __shared__ __attribute__((aligned(16))) int prm[2][4 * C];                // constants of a block's two convolutions
    __shared__ __attribute__((aligned(16))) int tprm[TAIL ? 3 * 4 * C2 : 4];  // of the tail

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const long img0 = (long)blockIdx.x * NI;
    typedef const __attribute__((address_space(4))) NarrowBlock *block_ptr;   // scalar loads
    const block_ptr blocks = (block_ptr)(uintptr_t)p.blocks;
    const bool to_memory = !p.tail && !p.head;       // the last block stores its sum instead of keeping it in LDS

    // ---- the stage's input ----
    if (p.nblocks)
        for (int i = tid; i < 4 * C; i += 256) prm[0][i] = blocks[0].prm1[i];
    if (TAIL && p.tail)
        for (int i = tid; i < 3 * 4 * C2; i += 256) tprm[i] = p.tprm[i];
    if (p.nblocks) fill_ring<C, S, NI>(X, blocks[0].zp_x, tid);
    else if (p.tail) fill_ring<C, S, NI>(X, p.tzp_x, tid);
    if (C == 16 && p.stem) {
        if constexpr (C == 16) {
            // the noisy image as NHWC4 words, one pixel of padding left, three right; behind it the sampler's table
            constexpr int PW = S + 4;
            int *img = (int *)T;
            NoiseLds *tab = (NoiseLds *)(T + (S + 2) * PW * 4);
            static_assert((S + 2) * PW * 4 % 16 == 0 && (S + 2) * PW * 4 + sizeof(NoiseLds) <= sizeof(T), "image and table fit");
            const int zb = (int)((uint32_t)(p.zp_in & 0xFF) * 0x01010101u);
            for (int i = tid; i < 2 * PW + 4 * S; i += 256) {
                int y, x;
                if (i < PW) { y = 0; x = i; }
                else if (i < 2 * PW) { y = S + 1; x = i - PW; }
                else { y = 1 + ((i - 2 * PW) >> 2); x = (i & 3) == 0 ? 0 : S + (i & 3); }
                img[y * PW + x] = zb;
            }
            const int y = tid / (S / 4), x4 = tid % (S / 4);   // one quad of pixels per thread
            uint32_t v[4];
            if (p.fused_noise) {
                const uint8_t *xim;
                const DeviceNoiseTable *src;
                uint32_t image_id, sample;
                resolve_noise_source(p.noise, img0, xim, src, image_id, sample);
                stage_noise_table(*tab, src, tid, 256);
                const int n = (int)src->n, dmin = src->dmin;
                lds_barrier();
                noisy_quad(*tab, n, dmin, xim, p.noise.C, S, S, y, x4, sample, image_id, p.noise.phase, p.noise.key0, p.noise.key1, v);
            } else {
                const v4i w = *(const v4i *)(p.in + ((img0 * S + y) * S + 4 * x4) * 4);
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = (uint32_t)w[j];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) img[(y + 1) * PW + 1 + 4 * x4 + j] = (int)v[j];
            lds_barrier();
            // one v_mfma_i32_16x16x64_i8 per 16 pixels: lane group ky reads the 16 contiguous bytes of kernel row ky (4 pixels x
            // 4 stored channels, the fourth pixel and channel meeting zero weights), the fourth group zero weights
            const int l = lane & 15, kg = lane >> 4, kr = kg < 3 ? kg : 0;
            const v4i fa = *(const v4i *)(p.w0 + l * 64 + kg * 16);
            const int x = 16 * (wave & 1) + l, row0 = 16 * (wave >> 1);
            const bool store = to_memory && p.nblocks == 0;
            with_form<RQ_TOP>(p.form0, [&](auto rq, auto) {
                constexpr int RQ = decltype(rq)::value;
                const LaneConsts<4, RQ> k(p.prm0, 16, 4 * kg);
                const int *src = img + (row0 + kr) * PW + x;
                int8_t *dst = X + ((row0 + 1) * P + x + 1) * 16 + 4 * kg;
                int8_t *gdst = p.out + ((img0 * S + row0) * S + x) * 16 + 4 * kg;
#pragma unroll 4
                for (int r = 0; r < 16; ++r) {
                    const v4i fb = {src[r * PW], src[r * PW + 1], src[r * PW + 2], src[r * PW + 3]};
                    k.fragment();
                    const v4acc acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa, fb, bias_vector<4, RQ>(k), 0, 0, 0);
                    const uint32_t q = rq_pack<RQ>(k.conv(acc[0], 0, p.lo0), k.conv(acc[1], 1, p.lo0), k.conv(acc[2], 2, p.lo0), k.conv(acc[3], 3, p.lo0));
                    if (store) *(uint32_t *)(gdst + r * S * 16) = q;
                    else *(uint32_t *)(dst + r * P * 16) = q;
                }
            });
        }
    } else {
        for (int i = tid; i < NI * S * S * CH; i += 256) {
            const int im = i / (S * S * CH), j = i % (S * S * CH), pix = j / CH, c = j % CH;
            long g = img0 + im;
            if (g >= p.B) g = p.B - 1;                   // images past the end repeat the last one; never stored
            *(v4i *)(X + im * TB + tile_at<C, S>(pix / S + 1, pix % S + 1, c)) = *(const v4i *)(p.in + (g * S * S + pix) * C + c * 16);
        }
    }

    // ---- identity blocks ----
    int zp_t = 256;   // zero-point in the border of t; none yet
    for (int blk = 0; blk < p.nblocks; ++blk) {
        const auto &d = blocks[blk];
        const bool last = blk + 1 == p.nblocks;
        lds_barrier();            // x, its border and the first convolution's constants are in LDS; the previous block is done with t
        for (int i = tid; i < 4 * C; i += 256) prm[1][i] = d.prm2[i];
        if (d.zp_t != zp_t) { fill_ring<C, S, NI>(T, d.zp_t, tid); zp_t = d.zp_t; }
        // what the next user of x wants in its border (this block reads x's border in its first convolution only)
        const int zp_next = last ? (p.tail ? p.tzp_x : d.zp_x) : blocks[last ? blk : blk + 1].zp_x;
        with_form<RQ_TOP>(d.form, [&](auto rq, auto rqa) {
            constexpr int RQ = decltype(rq)::value, RQA = decltype(rqa)::value;
            if constexpr (C == 16) {
                // 16 channels: a K step of v_mfma_i32_16x16x64_i8 is one kernel row -- lane group kg holds tap (ky = step, kx = kg),
                // the fourth group zero weights -- and a wave walks down 16 rows of a 16-pixel column strip: the operands of
                // rows y + 1, y + 2 of one output row are those of rows y, y + 1 of the next, one new LDS read per output fragment
                constexpr int KP = (9 * C + 63) / 64 * 64;
                const int l = lane & 15, kg = lane >> 4, kx = kg < 3 ? kg : 0;
                const int x = 16 * (wave & 1) + l, row0 = 16 * (wave >> 1);
                auto conv = [&](const int8_t *src, const int8_t *w, const int *pr, auto emit) {
                    v4i fa[3];
#pragma unroll
                    for (int ky = 0; ky < 3; ++ky) {
                        fa[ky] = *(const v4i *)(w + l * KP + (ky * 3 + kx) * 16);
                        if (kg == 3) fa[ky] = v4i{0, 0, 0, 0};
                    }
                    const LaneConsts<4, RQ> k(pr, 16, 4 * kg);
                    const int8_t *col = src + (row0 * P + x + kx) * C;   // padded (row0, x + kx) = tap (0, kx) of output (row0, x)
                    v4i b0 = *(const v4i *)col, b1 = *(const v4i *)(col + P * C);
#pragma unroll 4
                    for (int r = 0; r < 16; ++r) {
                        const v4i b2 = *(const v4i *)(col + (r + 2) * P * C);
                        k.fragment();
                        v4acc acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[0], b0, bias_vector<4, RQ>(k), 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[1], b1, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[2], b2, acc, 0, 0, 0);
                        emit(r, acc, k);
                        b0 = b1;
                        b1 = b2;
                    }
                };
                const int at = ((row0 + 1) * P + x + 1) * 16 + 4 * kg;      // the lane's four channels of its pixel in row 0
                conv(X, d.w1, prm[0], [&](int r, const v4acc &a, const LaneConsts<4, RQ> &k) {
                    *(uint32_t *)(T + at + r * P * 16) = rq_pack<RQ>(k.conv(a[0], 0, d.lo1), k.conv(a[1], 1, d.lo1), k.conv(a[2], 2, d.lo1), k.conv(a[3], 3, d.lo1));
                });
                lds_barrier();
                if (!last)
                    for (int i = tid; i < 4 * C; i += 256) prm[0][i] = blocks[blk + 1].prm1[i];
                if (zp_next != d.zp_x) fill_ring<C, S, NI>(X, zp_next, tid);
                const AddConst ac = {d.add.ms, d.add.mr, d.add.c0, d.add.k, d.add.sh, d.add.lo};
                int8_t *gdst = p.out + ((img0 * S + row0) * S + x) * 16 + 4 * kg;
                const bool store = last && to_memory;
                conv(T, d.w2, prm[1], [&](int r, const v4acc &a, const LaneConsts<4, RQ> &k) {
                    uint32_t *res = (uint32_t *)(X + at + r * P * 16);
                    const uint32_t rw = *res;
                    int q[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) q[i] = rq_add<RQ, RQA>(k.conv(a[i], i, d.lo2), rw, i, ac);
                    const uint32_t o = rq_pack<RQA>(q[0], q[1], q[2], q[3]);
                    if (store) *(uint32_t *)(gdst + r * S * 16) = o;
                    else *res = o;
                });
            } else {
                const WideConv<C, S> wc(lane, wave);
                constexpr int MF = wc.MF, NF = wc.NF, FRAGS = NI * NF * MF / 4;   // fragments per wave
                v4i fa[wc.KS];
                wc.load_weights(d.w1, fa);
                {
                    const LaneConsts<16, RQ> k(prm[0], C, wc.mf * 32 + wc.half * 16);
#pragma unroll 1
                    for (int i = 0; i < FRAGS; ++i) {
                        const int f = wave / MF + i * (4 / MF), off = (f / NF) * TB + (f % NF) * wc.FRAG;
                        k.fragment();
                        const v16i a = wc.run(X + off, fa, bias_vector<16, RQ>(k));
                        int q[16];
#pragma unroll
                        for (int e = 0; e < 16; ++e) q[e] = k.conv(a[e], e, d.lo1);
                        *(v4i *)(T + off + wc.out) = rq_pack16<RQ>(q);
                    }
                }
                wc.load_weights(d.w2, fa);
                lds_barrier();
                if (!last)
                    for (int i = tid; i < 4 * C; i += 256) prm[0][i] = blocks[blk + 1].prm1[i];
                if (zp_next != d.zp_x) fill_ring<C, S, NI>(X, zp_next, tid);
                const AddConst ac = {d.add.ms, d.add.mr, d.add.c0, d.add.k, d.add.sh, d.add.lo};
                const LaneConsts<16, RQ> k(prm[1], C, wc.mf * 32 + wc.half * 16);
                const bool store = last && to_memory;
#pragma unroll 1
                for (int i = 0; i < FRAGS; ++i) {
                    const int f = wave / MF + i * (4 / MF), im = f / NF, off = im * TB + (f % NF) * wc.FRAG;
                    k.fragment();
                    const v16i a = wc.run(T + off, fa, bias_vector<16, RQ>(k));
                    v4i *res = (v4i *)(X + off + wc.out);
                    const v4i rv = *res;
                    int q[16];
#pragma unroll
                    for (int e = 0; e < 16; ++e) q[e] = rq_add<RQ, RQA>(k.conv(a[e], e, d.lo2), (uint32_t)rv[e >> 2], e & 3, ac);
                    const v4i o = rq_pack16<RQA>(q);
                    const long g = img0 + im;
                    if (!store) *res = o;
                    else if (g < p.B) *(v4i *)(p.out + ((g * S * S + (f % NF) * 32 + wc.l) * C + (2 * wc.mf + wc.half) * 16)) = o;
                }
            }
        });
    }

    // ---- down-sampling into the next stage ----
    if constexpr (TAIL) {
        if (p.tail) {
            constexpr int TB2 = tile_bytes<C2, S2>(), KP1 = (9 * C + 63) / 64 * 64, KS1 = (9 * C + 31) / 32;
            static_assert(NI * TB2 <= NI * TB, "the next stage's tile fits the middle tensor's");
            const WideConv<C2, S2> wc(lane, wave);
            constexpr int MF = wc.MF, NF = wc.NF, FRAGS = NI * NF * MF / 4;
            const int l = wc.l, half = wc.half, mf = wc.mf;
            const int oy0 = l / S2, ox = l % S2;       // the lane's output pixel in fragment 0
            v4i f1[KS1];
#pragma unroll
            for (int ks = 0; ks < KS1; ++ks) f1[ks] = *(const v4i *)(p.tw1 + (mf * 32 + l) * KP1 + ks * 32 + half * 16);
            // tap (ky, kx) of output (oy, ox) is padded input (2 oy + ky, 2 ox + kx).  16 input channels: a K step is two taps,
            // the lane half picks one (the tenth has zero weights); 32: one tap, the half picks 16 channels
            int b1[KS1];
#pragma unroll
            for (int ks = 0; ks < KS1; ++ks) {
                int tap = C == 16 ? 2 * ks + half : ks;
                if (tap > 8) tap = 0;
                b1[ks] = tile_at<C, S>(2 * oy0 + tap / 3, 2 * ox + tap % 3, C == 16 ? 0 : half);
            }
            constexpr int FRAG1 = 2 * (32 / S2) * P * C;   // input bytes from one output fragment to the next (an even number of rows)
            lds_barrier();            // x is complete, the last block is done with t
            fill_ring<C2, S2, NI>(T, p.tzp_t, tid);
            with_form<RQ_TOP_WIDE>(p.tform, [&](auto rq, auto rqa) {
                constexpr int RQ = decltype(rq)::value, RQA = decltype(rqa)::value;
                const int c0 = mf * 32 + half * 16;
                {
                    const LaneConsts<16, RQ> k(tprm, C2, c0);
                    const bool store = p.tail == 2 && !p.head;
#pragma unroll 1
                    for (int i = 0; i < FRAGS; ++i) {
                        const int f = wave / MF + i * (4 / MF), im = f / NF;
                        const int8_t *src = X + im * TB + (f % NF) * FRAG1;
                        k.fragment();
                        v16i a = bias_vector<16, RQ>(k);
#pragma unroll
                        for (int ks = 0; ks < KS1; ++ks)
                            a = __builtin_amdgcn_mfma_i32_32x32x32_i8(f1[ks], *(const v4i *)(src + b1[ks]), a, 0, 0, 0);
                        int q[16];
#pragma unroll
                        for (int e = 0; e < 16; ++e) q[e] = k.conv(a[e], e, p.tlo1);
                        const v4i o = rq_pack16<RQ>(q);
                        const long g = img0 + im;
                        if (!store) *(v4i *)(T + im * TB2 + (f % NF) * wc.FRAG + wc.out) = o;
                        else if (g < p.B) *(v4i *)(p.out + ((g * S2 * S2 + (f % NF) * 32 + l) * C2 + c0)) = o;
                    }
                }
                if (p.tail == 1) {
                    v4i fa[wc.KS];
                    wc.load_weights(p.tw2, fa);
                    const v4i fp = *(const v4i *)(p.twp + (mf * 32 + l) * 64 + half * 16);   // channels 0 .. 31 (zeros past C)
                    const int xp = tile_at<C, S>(2 * oy0 + 1, 2 * ox + 1, C == 16 ? 0 : half);
                    lds_barrier();
#pragma unroll 1
                    for (int i = 0; i < FRAGS; ++i) {
                        const int f = wave / MF + i * (4 / MF), im = f / NF;
                        asm volatile("" ::: "memory");   // one convolution's constants at a time
                        int r[16], q[16];
                        {
                            const LaneConsts<16, RQ> k(tprm + 2 * 4 * C2, C2, c0);
                            const v16i a = __builtin_amdgcn_mfma_i32_32x32x32_i8(fp, *(const v4i *)(X + im * TB + (f % NF) * FRAG1 + xp), bias_vector<16, RQ>(k), 0, 0, 0);
#pragma unroll
                            for (int e = 0; e < 16; ++e) r[e] = k.conv(a[e], e, p.tlop);
                        }
                        asm volatile("" ::: "memory");
                        {
                            const LaneConsts<16, RQ> k(tprm + 4 * C2, C2, c0);
                            const v16i a = wc.run(T + im * TB2 + (f % NF) * wc.FRAG, fa, bias_vector<16, RQ>(k));
#pragma unroll
                            for (int e = 0; e < 16; ++e) {
                                const int u = k.conv(a[e], e, p.tlo2);
                                q[e] = rq_add_value<RQ, RQA>(r[e], rq_is_top(RQ) ? u >> 24 : u, p.tadd);
                            }
                        }
                        const long g = img0 + im;
                        if (g < p.B) *(v4i *)(p.out + ((g * S2 * S2 + (f % NF) * 32 + l) * C2 + c0)) = rq_pack16<RQA>(q);
                    }
                }
            });
            if (p.head) {   // tail == 2: the pooling reads the convolution just computed
                lds_barrier();
                if constexpr (C == 16) narrow_head<C2, S2, NI>(p, T, X, img0, tid);
            }
            return;
        }
    }
    if (p.head) {
        lds_barrier();
        if constexpr (C == 64) narrow_head<C, S, NI>(p, X, T, img0, tid);
    }
}

template <int C, int S, int NI>
hipError_t launch_stage(const NarrowParams &p, hipStream_t st) {
    static const std::string name = "narrow_kernel<" + std::to_string(C) + ", " + std::to_string(S) + ", " + std::to_string(NI) + ">";
    set_kernel_name(name.c_str());
    hipLaunchKernelGGL((narrow_kernel<C, S, NI>), dim3((unsigned)((p.B + NI - 1) / NI)), dim3(256), 0, st, p);
    return hipGetLastError();
}

}  // namespace

// Shapes with a kernel: identity blocks of 16 channels at 32 x 32, 32 at 16 x 16, 64 at 8 x 8 (the three stages of
// the CIFAR-style residual nets), down-sampling blocks 16 -> 32 at 32 x 32 -> 16 x 16 and 32 -> 64 at 16 x 16 -> 8 x 8.
bool basic_block_supported(int channels, int size) {
    return (channels == 16 && size == 32) || (channels == 32 && size == 16) || (channels == 64 && size == 8);
}
bool trans_block_supported(int cout, int size_out) { return (cout == 32 && size_out == 16) || (cout == 64 && size_out == 8); }

hipError_t launch_narrow(const NarrowParams &p, int channels, hipStream_t st) {
    if (p.B <= 0) return hipSuccess;
    const bool from_image = channels == 16 && p.stem;
    if ((p.nblocks > 0 && !p.blocks) || p.nblocks < 0 || (p.nblocks == 0 && !p.tail && !from_image) || (!p.head && !p.out) ||
        (from_image ? !p.w0 || !p.prm0 || (!p.fused_noise && !p.in) : !p.in || p.stem))
        return hipErrorInvalidValue;
    if (p.fused_noise) {
        const NoiseSource &ns = p.noise;
        if (!from_image || !ns.x || !ns.table || ns.C < 1 || ns.C > 3 || ns.H != 32 || ns.W != 32 || (ns.items && ns.n_per_item == 0)) return hipErrorInvalidValue;
    }
    if (p.tail && (channels == 64 || !p.tw1 || !p.tprm || (p.tail == 1 && (!p.tw2 || !p.twp)) || p.tail > 2)) return hipErrorInvalidValue;
    if (p.head && (!(channels == 64 || (channels == 16 && p.tail == 2)) || (p.tail && channels == 64) || !p.fc_w || !p.fc_bias || p.classes < 1 ||
                   p.classes_p < p.classes || (channels == 64 && p.nblocks == 0)))
        return hipErrorInvalidValue;
    // one image per workgroup while that leaves no CU with more than one workgroup; beyond, several share the weights
    const bool few = p.B <= 256;
    if (channels == 16) return launch_stage<16, 32, 1>(p, st);
    if (channels == 32) return few ? launch_stage<32, 16, 1>(p, st) : launch_stage<32, 16, 2>(p, st);
    if (channels == 64) return few ? launch_stage<64, 8, 1>(p, st) : launch_stage<64, 8, 4>(p, st);
    return hipErrorInvalidValue;
}

}  // namespace isr
