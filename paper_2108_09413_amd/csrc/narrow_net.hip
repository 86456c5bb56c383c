// The nets on 32 x 32 images (stages of 16 channels at 32 x 32, 32 at 16 x 16, 64 at 8 x 8 pixels), one launch per stage (of few copies one for all):
//   [first layer: noise draws + 3x3 convolution into 16 channels]   stage 16 only; else the stage's input is loaded
//   identity blocks  t = conv3x3(x), x = add(conv3x3(t), x)         any number
//   [down-sampling block into the next stage, or its first convolution alone]
//   [global average pooling, fully connected layer, argmax, vote]
// A workgroup of four waves (eight: see launch_narrow) keeps NI whole images in LDS from the first of these to the last: x and t as (S+2) x (S+2) x C
// int8 tiles whose border holds the tensor's zero-point, so that taps need no bounds checks and contribute 0.  The sum of
// a block replaces x in place (a lane reads the residual at its own pixel and writes there; the second convolution
// reads only t).  Memory sees the noise table, the stage's result and the weights (L2-resident, a few KiB a convolution).
//
// The 16 K-bytes of an MFMA operand lane are 16 channels of one tap = one aligned 128-bit LDS read at a tap-shifted
// address.  Bank conflicts: the LDS serves the lanes {0-3, 12-15, 20-27} of such a read together, then {4-11, 16-19, 28-31}
// (and the same of the upper half), from 64 banks of 4 bytes.  At 32 channels (a fragment is two rows of 16 pixels, 32
// bytes a pixel) each of these sets takes from either row 8 pixels that are all different mod 8, at 64 channels (four rows of
// 8 pixels, 64 bytes a pixel) from each row 4 that are different mod 4: with chunk c of the pixel at padded (y, x) at chunk
// c ^ (y mod 2), resp. c ^ (0, 2, 1, 3 for y mod 4), no two lanes of a set meet in a bank, nor those of a read of two rows of 8
// pixels and four chunks.  Columns and rows of a tap are immediate
// offsets from a base address per parity of the row.
//
// What bounds it: issue of the requantisation arithmetic, the matrix unit and the LDS reads of the pixel operands, all three
// within a factor of two of each other (cycles of a CU per image and block at 16 / 32 / 64 channels: arithmetic
// 2660 / 1330 / 660, MFMA 1540 / 1150 / 1150, LDS reads 1620 / 1280 / 1280), at a clock that the power limit holds near 1.9
// of 2.4 GHz.  So the three have to overlap: the arithmetic of a fragment stands between the MFMAs of the next.  Four
// workgroups share a CU at 16 channels, two at 32 and 64, where the operands in flight take the registers of a third (two
// with pairs of fragments measured 1.81 / 1.40 / 1.11 ms for the stages of a 110-layer net on 16 700 images, three without
// 1.88 / 1.45 / 1.23 ms).  With one workgroup on a CU there is nothing to overlap with: descriptors, weights and constants of
// a convolution are fetched while the one before runs, and 16 channels take eight waves (predictions with 100 copies: ResNet-20
// 52.3 -> 50.0 us, ResNet-110 171 -> 153, the two-convolution net 24.5 -> 23.8; before the stages shared a launch and the host watched for the tallies).  More images per workgroup amortise the weight and constant loads of a convolution at 32 and 64
// channels, where a wave has one or two fragments per image.  The certification of the 110-layer net at 100 000 samples took
// 43.3 ms with one launch per block, 31.6 with one per stage, 27.0 with the overlap.
#include <cstddef>
#include <string>

#include "conv_device.h"
#include "noise_device.h"

namespace isr {

namespace {

// byte offset of a chunk of the pixel at padded (y, x).  STRIDED: the layout of x for the stride-2 reads of the tail, where
// all rows of a read have the same parity and columns 8 apart must differ.
template <int C, int S, bool STRIDED = false>
__device__ __forceinline__ int tile_at(int y, int x, int chunk) {
    const int s = C == 64 ? 2 * (y & 1) + (y >> 1 & 1) : C == 32 ? (STRIDED ? (x >> 3) & 1 : y & 1) : 0;
    return ((y * (S + 2) + x) * (C / 16) + (chunk ^ s)) * 16;
}
template <int C, int S>
constexpr int tile_bytes() { return (S + 2) * (S + 2) * C; }

// border pixel b of a padded (S+2) x (S+2) tile: top row, bottom row, left and right columns without the corners
template <int S>
__device__ __forceinline__ void border_pixel(int b, int &y, int &x) {
    constexpr int P = S + 2;
    if (b < P) { y = 0; x = b; }
    else if (b < 2 * P) { y = P - 1; x = b - P; }
    else if (b < 3 * P - 2) { y = b - 2 * P + 1; x = 0; }
    else { y = b - (3 * P - 2) + 1; x = P - 1; }
}
template <int C, int S, int NI, int NT>
__device__ __forceinline__ void fill_ring(int8_t *tile, int zp, int tid) {
    constexpr int CH = C / 16, N = (4 * (S + 2) - 4) * CH;
    const int z = (int)((uint32_t)(zp & 0xFF) * 0x01010101u);
    for (int i = tid; i < NI * N; i += NT) {
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
    int base[C == 64 ? 6 : 2];    // by kernel row (mod 2 at 32 channels) and half of the 64 channels
    int out, out_strided;         // the lane's chunk of its own pixel (fragment 0) for M fragment mf; the same in the strided layout
    int mf, half, l;

    __device__ __forceinline__ WideConv(int lane, int wave) {
        l = lane & 31; half = lane >> 5; mf = wave % MF;
        const int y = l / S, x = l % S;
        if constexpr (C == 64) {
#pragma unroll
            for (int ky = 0; ky < 3; ++ky) {
                base[2 * ky] = tile_at<C, S>(y + ky, x, half);
                base[2 * ky + 1] = base[2 * ky] ^ 32;
            }
        } else {
            base[0] = tile_at<C, S>(y, x, half);
            base[1] = base[0] ^ 16;   // rows of the other parity: chunk position swapped, row offset in the immediate
        }
        out = tile_at<C, S>(y + 1, x + 1, 2 * mf + half);
        out_strided = tile_at<C, S, true>(y + 1, x + 1, 2 * mf + half);
    }
    __device__ __forceinline__ const int8_t *weight_row(const int8_t *w) const { return w + (mf * 32 + l) * KP + half * 16; }
    __device__ __forceinline__ void load_weights(const int8_t *w, v4i (&fa)[KS]) const {
        const int8_t *row = weight_row(w);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) fa[ks] = *(const v4i *)(row + ks * 32);
    }
    __device__ __forceinline__ v4i operand(const int8_t *frag, int ks) const {   // pixel operand of K step ks
        const int tap = C == 64 ? ks >> 1 : ks, ky = tap / 3, kx = tap % 3;
        return *(const v4i *)(frag + (C == 64 ? base[2 * ky + (ks & 1)] + kx * C : base[ky & 1] + (ky * P + kx) * C));
    }
    __device__ __forceinline__ v16i run(const int8_t *frag, const v4i (&fa)[KS], v16i acc) const {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[ks], operand(frag, ks), acc, 0, 0, 0);
        return acc;
    }
};

// The K loop of a group of P fragments with the epilogue of the group before between its MFMAs: a step issues P independent
// MFMAs (32 cycles of the matrix unit each) and a KS-th of the other group's requantisation (EPI), and reads the pixel
// operands of three steps later.  Left to itself the compiler puts the chain of MFMAs first, its operand reads at most two
// ahead, and the arithmetic behind it.  NEXT: as a step's weights have seen their last MFMA, those of the next convolution
// are fetched into their registers (`next`: the lane's weight row there).
template <int P, bool EPI, bool NEXT, int C, int S, class Elem>
__device__ __forceinline__ void wide_group(const WideConv<C, S> &wc, const int8_t *const (&src)[P], v4i (&fa)[WideConv<C, S>::KS], v16i (&acc)[P],
                                           const int8_t *next, Elem elem) {
    constexpr int KS = WideConv<C, S>::KS, AHEAD = 3, PER = (16 * P + KS - 2) / (KS - 1);   // elements per step; none in the first
    v4i fb[AHEAD + 1][P];
#pragma unroll
    for (int ks = 0; ks < AHEAD; ++ks)
#pragma unroll
        for (int q = 0; q < P; ++q) fb[ks][q] = wc.operand(src[q], ks);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        if (ks + AHEAD < KS)
#pragma unroll
            for (int q = 0; q < P; ++q) fb[(ks + AHEAD) % (AHEAD + 1)][q] = wc.operand(src[q], ks + AHEAD);
#pragma unroll
        for (int q = 0; q < P; ++q) {
            acc[q] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[ks], fb[ks % (AHEAD + 1)][q], acc[q], 0, 0, 0);
            if constexpr (EPI) {
                const int first = (ks - 1) * PER + q * (PER / P), end = q + 1 < P ? first + PER / P : ks * PER;
#pragma unroll
                for (int e = first; e < end; ++e)
                    if (e >= 0 && e < 16 * P) elem(e);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (NEXT) fa[ks] = *(const v4i *)(next + ks * 32);
    }
}

// A lane's constants of N consecutive output channels from the packed form [4][C].  The pair form keeps them in registers
// across the fragments of a convolution; the other reads them for each fragment, where they are used or (FETCH) ahead of its products.
template <int N, int RQ, bool FETCH = false, bool PAIR = RQ == RQ_PAIR>
struct LaneConsts {
    int m0[N], b4[4];
    RqLayer layer;
    const int *b;                 // 16 channels: the bias is read into the accumulator, registers are short
    __device__ __forceinline__ LaneConsts(const int *prm, int C, int c0) : b(prm + c0) {
#pragma unroll
        for (int i = 0; i < N; ++i) m0[i] = prm[C + c0 + i];
#pragma unroll
        for (int i = 0; i < 4; ++i) b4[i] = prm[c0 + i];
        layer = rq_layer<RQ>(prm[2 * C], prm[3 * C]);
    }
    __device__ __forceinline__ void fragment() const { if (N == 16) asm volatile("" ::: "memory"); }   // start of a fragment: the bias is not kept
    __device__ __forceinline__ int bias(int i) const { return N == 4 ? b4[i & 3] : b[i]; }
    __device__ __forceinline__ int conv(int acc, int i, int lo) const { return rq_conv<RQ>(acc, m0[i], 0, 0, lo, layer); }
};
template <int N, int RQ, bool FETCH>
struct LaneConsts<N, RQ, FETCH, false> {
    const int *at;
    int C, m0[N], chi[N], sh[N];   // FETCH: of the fragment under way
    RqLayer layer = {};
    __device__ __forceinline__ LaneConsts(const int *prm, int C_, int c0) : at(prm + c0), C(C_) {}
    __device__ __forceinline__ void fragment() {
        asm volatile("" ::: "memory");   // no constant is carried over in a register
        if (FETCH)
#pragma unroll
            for (int i = 0; i < N; ++i) { m0[i] = at[C + i]; chi[i] = at[2 * C + i]; sh[i] = at[3 * C + i]; }
    }
    __device__ __forceinline__ int bias(int i) const { return at[i]; }
    __device__ __forceinline__ int conv(int acc, int i, int lo) const {
        return FETCH ? rq_conv<RQ>(acc, m0[i], chi[i], sh[i], lo, layer) : rq_conv<RQ>(acc, at[C + i], at[2 * C + i], at[3 * C + i], lo, layer);
    }
};
template <int N, int RQ, bool FETCH>
__device__ __forceinline__ auto bias_vector(const LaneConsts<N, RQ, FETCH> &k) {
    typedef int vec __attribute__((ext_vector_type(N)));
    vec v;
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = k.bias(i);
    return v;
}

// FRAGS fragments of one convolution of a wave, weights in `fa`, which afterwards holds those at `next`: source(i) is
// fragment i's tile address; element(i, q, e, value) consumes the accumulator of element e (in the order of e), after
// start(i, q) and before finish(i); q: which of a group's fragments, a constant wherever it indexes registers.
// The general form (shifts that differ by channel, exact halves) takes one fragment after the other, its arithmetic covered by other
// workgroups.  Its operands too are read three steps ahead and its constants (FETCH) before the products: left to the compiler, whether
// a product waits for the read in front of it changed with the code around it.  us of the 64-channel stage of a 110-layer net with
// 300 / 10 000 copies 118 / 1150 -> 105 / 975, of the 32-channel one 109 / 1380 -> 106 / 1323; the whole net with 100 copies in one
// launch 200 -> 188.
template <int FRAGS, bool PAIRS, int RQ, int C, int S, class Source, class Start, class Element, class Finish>
__device__ __forceinline__ void wide_fragments(const WideConv<C, S> &wc, v4i (&fa)[WideConv<C, S>::KS], LaneConsts<16, RQ, true> &k, const int8_t *next,
                                               Source source, Start start, Element element, Finish finish) {
    if constexpr (RQ == RQ_PAIR) {
        constexpr int P = PAIRS && FRAGS >= 2 ? 2 : 1, G = FRAGS / P;
        static_assert(FRAGS % P == 0, "whole groups");
        const int8_t *row = wc.weight_row(next);
        v16i acc[P];
        auto begin = [&](int g, const int8_t *(&src)[P]) {
            k.fragment();
#pragma unroll
            for (int q = 0; q < P; ++q) { src[q] = source(g * P + q); acc[q] = bias_vector(k); }
        };
        {
            const int8_t *src[P];
            begin(0, src);
            wide_group<P, false, G == 1>(wc, src, fa, acc, row, [](int) {});
        }
#pragma unroll
        for (int g = 1; g < G; ++g) {
            v16i prev[P];
#pragma unroll
            for (int q = 0; q < P; ++q) { prev[q] = acc[q]; start((g - 1) * P + q, q); }
            const int8_t *src[P];
            begin(g, src);
            auto elem = [&](int e) {
                const int i = (g - 1) * P + e / 16;
                element(i, e / 16, e & 15, prev[e / 16][e & 15]);
                if ((e & 15) == 15) finish(i);
            };
            if (g + 1 < G) wide_group<P, true, false>(wc, src, fa, acc, row, elem);
            else wide_group<P, true, true>(wc, src, fa, acc, row, elem);
        }
#pragma unroll
        for (int q = 0; q < P; ++q) {
            start((G - 1) * P + q, q);
#pragma unroll
            for (int e = 0; e < 16; ++e) element((G - 1) * P + q, q, e, acc[q][e]);
            finish((G - 1) * P + q);
        }
    } else {
#pragma unroll 1
        for (int i = 0; i < FRAGS; ++i) {
            k.fragment();
            v16i acc[1] = {bias_vector(k)};
            const int8_t *const src[1] = {source(i)};
            wide_group<1, false, false>(wc, src, fa, acc, nullptr, [](int) {});
            start(i, 0);
#pragma unroll
            for (int e = 0; e < 16; ++e) element(i, 0, e, acc[0][e]);
            finish(i);
        }
        wc.load_weights(next, fa);
    }
}

// f with the compile-time forms of a descriptor's `form`
template <class F>
__device__ __forceinline__ void with_form(int form, F f) {
    using std::integral_constant;
    if (form == 0) f(integral_constant<int, RQ_PAIR>{}, integral_constant<int, RQ_PAIR>{});
    else if (form == 1) f(integral_constant<int, RQ_PAIR>{}, integral_constant<int, RQ_ANY>{});
    else f(integral_constant<int, RQ_ANY>{}, integral_constant<int, RQ_ANY>{});
}

// Global average pooling of NI tiles, fully connected layer, argmax and votes.  `scratch` is LDS that nothing else uses.
template <int C, int S, int NI, int NT>
__device__ __forceinline__ void narrow_head(const NarrowParams &p, const int8_t *tile, int8_t *scratch, long img0, int tid) {
    constexpr int WORDS = C / 4, ITEMS = NI * WORDS, PARTS = NT / ITEMS, PPP = S * S / PARTS;   // pixels per part
    static_assert(ITEMS <= NT && S * S % PARTS == 0, "one part per thread");
    int *sums = (int *)scratch;                       // [NI][C]
    int8_t *feat = scratch + NI * C * 4;              // [NI][C]
    int *best_of = (int *)(feat + NI * C);            // [NI]
    const int lane = tid & 63, wave = tid >> 6;
    for (int i = tid; i < NI * C; i += NT) sums[i] = 0;
    lds_barrier();
    if (tid < ITEMS * PARTS) {
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
    for (int i = tid; i < NI * C; i += NT) {
        // RHA of the scaled sum, as the pooling kernel
        const long v = (long)(sums[i] - S * S * p.gap_zp_in) * p.gap_M0;
        const int sh = 31 + p.gap_sh;
        const unsigned long mag = (unsigned long)(v < 0 ? -v : v);
        const long q = (long)((mag + (1ul << (sh - 1))) >> sh);
        const int r = p.gap_zp_out + (int)(v < 0 ? -q : q);
        feat[i] = (int8_t)(r < -128 ? -128 : (r > 127 ? 127 : r));
    }
    lds_barrier();
    for (int im = wave; im < NI; im += NT / 64) {
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
            // a call of few copies: the host watches for every vote, no launch behind this one
            if (p.votes && g < p.B)
                __hip_atomic_store(&p.votes[p.slots.begin + (uint64_t)g], (uint64_t)p.seq << 32 | (uint32_t)best_idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            best_of[im] = g < p.B ? best_idx : -1;
        }
    }
    if (!p.counts) return;
    lds_barrier();
    if (wave) return;
    auto &part = p.parts->part[blockIdx.x % TALLY_PARTS];   // where there are parts
    if (tid < NI && best_of[tid] >= 0) {
        // one global addition per distinct (row, class) of the workgroup, by its first image
        auto row = [&](int im) { return slot_use(p.slots, (uint64_t)(img0 + im)).row; };
        const uint32_t r = row(tid);
        uint32_t n = 0;
        bool first = true;
        for (int im = 0; im < NI; ++im)
            if (best_of[im] == best_of[tid] && (im == tid || row(im) == r)) {
                ++n;
                first = first && im >= tid;
            }
        if (first) atomicAdd((p.parts ? part.votes : p.counts) + (size_t)r * p.classes + best_of[tid], n);
    }
    // A call's tallies by the last workgroup to finish, with no launch for them behind this one (us a call, in turn: ResNet-20 with
    // 400 / 1100 copies 61.2 -> 60.3 / 104.5 -> 103.7).  Additions are complete (vmcnt) before the next level counts them, and the
    // exchanges read each counter where they were made.  One word for the finished workgroups of the two-convolution net held 1100 of them
    // up for 11 us, and its votes, one a workgroup, are what bounds a call while they are added to one line of 64 bytes, as those of a
    // prediction are: with 600 / 2000 / 10 000 copies 27.2 -> 25.0 / 45.5 -> 37.1 / 149 -> 121 in parts (certifications of up to 4096, whose
    // counters lie in two lines, are within 0.8 us either way).
    if (p.tallies) {
        const uint32_t parts = gridDim.x < TALLY_PARTS ? gridDim.x : TALLY_PARTS;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        uint32_t last = 0;
        if (lane == 0 && __hip_atomic_fetch_add(&part.finished, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (gridDim.x - 1 - blockIdx.x % TALLY_PARTS) / TALLY_PARTS)
            last = __hip_atomic_fetch_add(&p.parts->complete, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == parts - 1;
        if (!__builtin_amdgcn_readfirstlane(last)) return;
        auto take = [](uint32_t *w) { return __hip_atomic_exchange(w, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
        for (uint32_t i = lane; i < p.tallies; i += 64) {
            uint32_t n = take(&p.counts[i]);
#pragma unroll
            for (uint32_t k = 0; k < TALLY_PARTS; ++k) n += take(&p.parts->part[k].votes[i]);
            __hip_atomic_store(&p.tally_host[i], n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        if (lane < TALLY_PARTS) take(&p.parts->part[lane].finished);
        if (lane == 0) take(&p.parts->complete);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (lane == 0) __hip_atomic_store(p.flag, p.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// A block's descriptor.  AHEAD: dword by dword in the lanes of a register, by a vector load two blocks ahead; else by scalar loads
// where its fields are used, which other workgroups of the CU cover; it is then made anew for each block, since what is alive across
// the convolutions costs these kernels their last registers (256 with 2 spilled instead of 253).
template <bool AHEAD>
struct Block {
    int lanes;
    const __attribute__((address_space(4))) NarrowBlock *at;
    __device__ __forceinline__ Block(const NarrowParams &p, int blk, int lane) {
        constexpr int N = sizeof(NarrowBlock) / 4;
        const NarrowBlock *b = p.blocks + (blk < p.nblocks ? blk : p.nblocks ? p.nblocks - 1 : 0);
        at = (const __attribute__((address_space(4))) NarrowBlock *)(uintptr_t)b;
        lanes = 0;
        if (AHEAD && p.nblocks) lanes = ((const int *)b)[lane < N ? lane : N - 1];
    }
    __device__ __forceinline__ int field(size_t offset) const { return __builtin_amdgcn_readlane(lanes, (int)(offset / 4)); }
    template <class T>
    __device__ __forceinline__ const T *pointer(size_t offset) const {
        typedef const __attribute__((address_space(1))) T *global;
        return (const T *)(global)(uintptr_t)((uint64_t)(uint32_t)field(offset) | (uint64_t)(uint32_t)field(offset + 4) << 32);
    }
#define ISR_FIELD(name) (AHEAD ? field(offsetof(NarrowBlock, name)) : at->name)
    __device__ __forceinline__ const int8_t *w1() const { return AHEAD ? pointer<int8_t>(offsetof(NarrowBlock, w1)) : at->w1; }
    __device__ __forceinline__ const int8_t *w2() const { return AHEAD ? pointer<int8_t>(offsetof(NarrowBlock, w2)) : at->w2; }
    __device__ __forceinline__ const int *prm1() const { return AHEAD ? pointer<int>(offsetof(NarrowBlock, prm1)) : at->prm1; }
    __device__ __forceinline__ const int *prm2() const { return AHEAD ? pointer<int>(offsetof(NarrowBlock, prm2)) : at->prm2; }
    __device__ __forceinline__ int zp_x() const { return ISR_FIELD(zp_x); }
    __device__ __forceinline__ int zp_t() const { return ISR_FIELD(zp_t); }
    __device__ __forceinline__ int lo1() const { return ISR_FIELD(lo1); }
    __device__ __forceinline__ int lo2() const { return ISR_FIELD(lo2); }
    __device__ __forceinline__ int form() const { return ISR_FIELD(form); }
    __device__ __forceinline__ AddConst add() const { return {ISR_FIELD(add.ms), ISR_FIELD(add.mr), ISR_FIELD(add.c0), ISR_FIELD(add.k), ISR_FIELD(add.sh), ISR_FIELD(add.lo)}; }
#undef ISR_FIELD
};

// SHORT: a whole net of two convolutions, the second with stride 2, in LDS for five workgroups a CU (narrow_short).
template <int C, int S, int NI, int NW, bool SHORT = false>
__device__ __forceinline__ void narrow_stage(const NarrowParams &p) {
    constexpr int NT = 64 * NW;                      // threads
    constexpr int P = S + 2, CH = C / 16, C2 = 2 * C, S2 = S / 2;
    constexpr int TB = tile_bytes<C, S>();
    constexpr bool TAIL = C < 64;                    // there is a next stage
    constexpr int R = 64 / NW;                       // 16 channels: rows of a wave's strip of 16 columns
    // One workgroup on a CU: nothing else runs while a convolution waits for its descriptor, its weights and its constants, which
    // are therefore all fetched while the one before runs.
    constexpr bool AHEAD = NI == 1 && (C > 16 || NW > 4);
    static_assert((C == 16 && S == 32 && NI == 1) || (C == 32 && S == 16) || (C == 64 && S == 8), "shape");
    static_assert(!SHORT || C == 16, "from the image");
    constexpr int TPRM = TAIL ? (SHORT ? 1 : 3) * 4 * C2 : 4;
    __shared__ __attribute__((aligned(256))) int8_t X[NI * TB];
    __shared__ __attribute__((aligned(256))) int8_t T[SHORT ? tile_bytes<C2, S2>() : NI * TB];
    __shared__ __attribute__((aligned(16))) int prm[2][4 * C];                // constants of a block's two convolutions
    __shared__ __attribute__((aligned(16))) int tprm[TPRM];                   // of the tail
    const int nblocks = SHORT ? 0 : p.nblocks, tail = SHORT ? 2 : p.tail;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const long img0 = (long)blockIdx.x * NI;

    // ---- the stage's input ----
    // constants, the sampler's table and the first weights are all on their way before any of them is waited for
    constexpr bool WIDE = C > 16;
    constexpr int NTP = TAIL ? (TPRM + NT - 1) / NT : 1;
    static_assert(4 * C <= 256, "one constant a thread");
    const bool from_image = SHORT || (C == 16 && p.stem);
    int v0 = 0, v1 = 0, vt[NTP] = {};
    v4i fa0 = {0, 0, 0, 0};
    NoiseStage<NT> vn;
    const uint8_t *xim = nullptr;
    const DeviceNoiseTable *table = nullptr;
    uint32_t image_id = 0;
    SlotUse use{};
    if (from_image) {
        v1 = p.prm0[tid & 63];
        fa0 = *(const v4i *)(p.w0 + (lane & 15) * 64 + (lane >> 4) * 16);
        if (p.fused_noise) {
            use = resolve_noise_source(p.noise, img0, xim, table, image_id);
            vn = fetch_noise_table<NT>(table, tid);
        }
    }
    if (nblocks && tid < 4 * C) v0 = p.first.prm1[tid];
    if (TAIL && tail)
#pragma unroll
        for (int j = 0; j < NTP; ++j)
            if (tid + NT * j < TPRM) vt[j] = p.tprm[tid + NT * j];
    // One image of 64 channels: a wave makes 16 channels of all pixels, so that every weight enters the CU once; with 32 channels x half of
    // the pixels a wave, each weight twice, those 72 KB took most of a convolution's 2900 to 3600 cycles (the one launch of the 110-layer
    // net with 100 copies 136 -> 121.5 us, ResNet-20's 33.3 -> 30.6, together with the results in pairs).  The down-sampling
    // block's weights are fetched where they are used: a convolution ahead they took registers from it all, 126 and 31.8 us.
    constexpr bool SLIM = C == 64 && NI == 1;
    v4i fa[SLIM ? 9 : WIDE ? WideConv<WIDE ? C : 32, WIDE ? S : 16>::KS : 3];   // weights of the convolution to come
    auto slim_weights = [&](const int8_t *w, v4i (&f)[9]) {
        const int row = 32 * (wave >> 1) + 8 * ((lane & 15) >> 2) + 4 * (wave & 1) + (lane & 3);   // of channel 16 wave + (lane & 15), in MFMA row order
#pragma unroll
        for (int ks = 0; ks < 9; ++ks) f[ks] = *(const v4i *)(w + row * 576 + ks * 64 + (lane >> 4) * 16);
    };
    // 16 channels: a lane's weights, by kernel row; the fourth lane group's are the zeros behind the nine taps
    auto narrow_weights = [&](const int8_t *w, v4i (&f)[3]) {
        constexpr int KP = (9 * 16 + 63) / 64 * 64;
        const int kg = lane >> 4;
#pragma unroll
        for (int ky = 0; ky < 3; ++ky) f[ky] = *(const v4i *)(w + (lane & 15) * KP + (kg < 3 ? ky * 3 + kg : 9 + ky) * 16);
    };
    int vp = 0;   // AHEAD: constants of the convolution after the next
    Block<AHEAD> cur(p, 0, lane), nxt(p, 1, lane);
    if (nblocks) {
        if constexpr (SLIM) slim_weights(p.first.w1, fa);
        else if constexpr (WIDE) WideConv<C, S>(lane, wave).load_weights(p.first.w1, fa);
        else if constexpr (AHEAD) narrow_weights(p.first.w1, fa);
        if (AHEAD && tid < 4 * C) vp = p.first.prm2[tid];
    }
    auto store_constants = [&]() {
        if (nblocks && tid < 4 * C) prm[0][tid] = v0;
        if (TAIL && tail)
#pragma unroll
            for (int j = 0; j < NTP; ++j)
                if (tid + NT * j < TPRM) tprm[tid + NT * j] = vt[j];
    };
    if (nblocks) fill_ring<C, S, NI, NT>(X, p.first.zp_x, tid);
    else if (!SHORT && tail) fill_ring<C, S, NI, NT>(X, p.tzp_x, tid);
    if (from_image) {
        if constexpr (C == 16) {
            // the noisy image as NHWC4 words, one pixel of padding left, three right; behind it the sampler's table
            constexpr int PW = S + 4;
            int *img = (int *)T;
            NoiseLds *tab = (NoiseLds *)(SHORT ? X : T + (S + 2) * PW * 4);
            static_assert((S + 2) * PW * 4 % 16 == 0 && (SHORT ? sizeof(NoiseLds) <= sizeof(X) : (S + 2) * PW * 4 + sizeof(NoiseLds) <= sizeof(T)), "image and table fit");
            const int zb = (int)((uint32_t)(p.zp_in & 0xFF) * 0x01010101u);
            for (int i = tid; i < 2 * PW + 4 * S; i += NT) {
                int y, x;
                if (i < PW) { y = 0; x = i; }
                else if (i < 2 * PW) { y = S + 1; x = i - PW; }
                else { y = 1 + ((i - 2 * PW) >> 2); x = (i & 3) == 0 ? 0 : S + (i & 3); }
                img[y * PW + x] = zb;
            }
            static_assert(S * S / 4 == 256, "one quad of pixels per thread of the first four waves");
            const int y = (tid & 255) / (S / 4), x4 = tid % (S / 4);
            int *dst = img + (y + 1) * PW + 1 + 4 * x4;
            if (p.fused_noise) {
                store_noise_table<NT>(*tab, vn, tid);
                const NoiseSampler smp = table->s;
                lds_barrier();
                if constexpr (NW == 4) {
                    uint32_t v[4];
                    noisy_quad(*tab, smp, table, xim, p.noise.C, S, S, y, x4, use.sample, image_id, use.phase, p.noise.key0, p.noise.key1, v);
#pragma unroll
                    for (int j = 0; j < 4; ++j) dst[j] = (int)v[j];
                } else {   // a channel of a quad at a time (the fourth byte of a pixel meets zero weights)
                    for (int c = tid >> 8; c < 3; c += NT / 256) {
                        int v[4];
                        noisy_values(*tab, smp, table, xim, c < p.noise.C, (uint32_t)((c * S + y) * S + x4 * 4), use.sample, image_id, use.phase, p.noise.key0,
                                     p.noise.key1, v);
#pragma unroll
                        for (int j = 0; j < 4; ++j) ((int8_t *)(dst + j))[c] = (int8_t)v[j];
                    }
                }
            } else if (tid < 256) {
                const v4i w = *(const v4i *)(p.in + ((img0 * S + y) * S + 4 * x4) * 4);
#pragma unroll
                for (int j = 0; j < 4; ++j) dst[j] = w[j];
            }
            if (tid < 64) prm[1][tid] = v1;
            store_constants();
            lds_barrier();
            if (SHORT) fill_ring<C, S, NI, NT>(X, p.tzp_x, tid);   // the table is done with
            // one v_mfma_i32_16x16x64_i8 per 16 pixels: lane group ky reads the 16 contiguous bytes of kernel row ky (4 pixels x
            // 4 stored channels, the fourth pixel and channel meeting zero weights), the fourth group zero weights
            const int l = lane & 15, kg = lane >> 4, kr = kg < 3 ? kg : 0;
            const int x = 16 * (wave & 1) + l, row0 = R * (wave >> 1);
            with_form(p.form0, [&](auto rq, auto) {
                constexpr int RQ = decltype(rq)::value;
                LaneConsts<4, RQ> k(prm[1], 16, 4 * kg);
                const int *src = img + (row0 + kr) * PW + x;
                int8_t *dst = X + ((row0 + 1) * P + x + 1) * 16 + 4 * kg;
#pragma unroll 4
                for (int r = 0; r < R; ++r) {
                    const v4i fb = {src[r * PW], src[r * PW + 1], src[r * PW + 2], src[r * PW + 3]};
                    k.fragment();
                    const v4acc acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa0, fb, bias_vector(k), 0, 0, 0);
                    const uint32_t q = rq_pack<RQ>(k.conv(acc[0], 0, p.lo0), k.conv(acc[1], 1, p.lo0), k.conv(acc[2], 2, p.lo0), k.conv(acc[3], 3, p.lo0), k.layer);
                    *(uint32_t *)(dst + r * P * 16) = q;
                }
            });
        }
    } else {
        for (int i = tid; i < NI * S * S * CH; i += NT) {
            const int im = i / (S * S * CH), j = i % (S * S * CH), pix = j / CH, c = j % CH;
            long g = img0 + im;
            if (g >= p.B) g = p.B - 1;                   // images past the end repeat the last one; never stored
            const int y = pix / S + 1, x = pix % S + 1;
            const int at = nblocks ? tile_at<C, S>(y, x, c) : tile_at<C, S, true>(y, x, c);
            *(v4i *)(X + im * TB + at) = *(const v4i *)(p.in + (g * S * S + pix) * C + c * 16);
        }
        store_constants();
    }

    // ---- identity blocks ----
    int zp_t = 256;   // zero-point in the border of t; none yet
    for (int blk = 0; blk < nblocks; ++blk) {
        const bool last = blk + 1 == nblocks;
        if constexpr (!AHEAD) {   // nothing of a descriptor is kept across the convolutions
            cur = Block<AHEAD>(p, blk, lane);
            nxt = Block<AHEAD>(p, last ? blk : blk + 1, lane);
        }
        const Block<AHEAD> after(p, AHEAD ? blk + 2 : 0, lane);
        const int zp_x = cur.zp_x(), zp_mid = cur.zp_t(), lo1 = cur.lo1(), lo2 = cur.lo2();
        lds_barrier();            // x, its border and the first convolution's constants are in LDS; the previous block is done with t
        if (tid < 4 * C) {
            prm[1][tid] = AHEAD ? vp : cur.prm2()[tid];
            if (AHEAD) vp = nxt.prm1()[tid];
        }
        if (zp_mid != zp_t) { fill_ring<C, S, NI, NT>(T, zp_mid, tid); zp_t = zp_mid; }
        // what the next user of x wants in its border (this block reads x's border in its first convolution only)
        const int zp_next = last ? (tail ? p.tzp_x : zp_x) : nxt.zp_x();
        auto second_constants = [&]() {   // between the convolutions
            lds_barrier();
            if (tid < 4 * C && !last) {
                prm[0][tid] = AHEAD ? vp : nxt.prm1()[tid];
                if (AHEAD) vp = nxt.prm2()[tid];
            }
            if (zp_next != zp_x) fill_ring<C, S, NI, NT>(X, zp_next, tid);
        };
        with_form(cur.form(), [&](auto rq, auto rqa) {
            constexpr int RQ = decltype(rq)::value, RQA = decltype(rqa)::value;
            if constexpr (C == 16) {
                // 16 channels: a K step of v_mfma_i32_16x16x64_i8 is one kernel row -- lane group kg holds tap (ky = step, kx = kg),
                // the fourth group zero weights -- and a wave walks down R rows of a 16-pixel column strip: the operands of
                // rows y + 1, y + 2 of one output row are those of rows y, y + 1 of the next, one new LDS read per output fragment
                const int l = lane & 15, kg = lane >> 4, kx = kg < 3 ? kg : 0;
                const int x = 16 * (wave & 1) + l, row0 = R * (wave >> 1);
                // The MFMAs of row r + 1 stand between the elements of row r's epilogue: element(r, e, value), then finish(r).
                auto conv = [&](const int8_t *src, const int8_t *w, const int *pr, auto make) {   // w: AHEAD the next convolution's
                    v4i fn[3];
                    narrow_weights(w, AHEAD ? fn : fa);
                    LaneConsts<4, RQ> k(pr, 16, 4 * kg);
                    const int8_t *col = src + (row0 * P + x + kx) * C;   // padded (row0, x + kx) = tap (0, kx) of output (row0, x)
                    auto operand = [&](int y) { return *(const v4i *)(col + (y < R + 2 ? y : R + 1) * P * C); };   // tile rows of the strip: 0 .. R + 1
                    v4i b[6];   // rows r + 1 .. r + 5 of the ring, read four rows ahead
#pragma unroll
                    for (int y = 0; y < 6; ++y) b[y] = operand(y);
                    v4acc acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[0], b[0], bias_vector(k), 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[1], b[1], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[2], b[2], acc, 0, 0, 0);
                    auto row = make(k);
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        b[r % 6] = operand(r + 6);
                        k.fragment();
                        v4acc next = acc;
                        // (no row R: the last step has no MFMAs)
                        if (r < R - 1) next = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[0], b[(r + 1) % 6], bias_vector(k), 0, 0, 0);
                        row(r, 0, acc[0]);
                        row(r, 1, acc[1]);
                        if (RQ == RQ_PAIR) __builtin_amdgcn_sched_barrier(0);
                        if (r < R - 1) next = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[1], b[(r + 2) % 6], next, 0, 0, 0);
                        row(r, 2, acc[2]);
                        if (RQ == RQ_PAIR) __builtin_amdgcn_sched_barrier(0);
                        if (r < R - 1) next = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[2], b[(r + 3) % 6], next, 0, 0, 0);
                        row(r, 3, acc[3]);
                        if (RQ == RQ_PAIR) __builtin_amdgcn_sched_barrier(0);
                        acc = next;
                    }
                    if (AHEAD)
#pragma unroll
                        for (int ky = 0; ky < 3; ++ky) fa[ky] = fn[ky];
                };
                const int at = ((row0 + 1) * P + x + 1) * 16 + 4 * kg;      // the lane's four channels of its pixel in row 0
                conv(X, AHEAD ? cur.w2() : cur.w1(), prm[0], [&](const LaneConsts<4, RQ> &k) {
                    return [&, q = v4acc{}](int r, int e, int a) mutable {
                        q[e] = k.conv(a, e, lo1);
                        if (e == 3) *(uint32_t *)(T + at + r * P * 16) = rq_pack<RQ>(q[0], q[1], q[2], q[3], k.layer);
                    };
                });
                second_constants();
                const AddConst ac = cur.add();
                conv(T, AHEAD ? nxt.w1() : cur.w2(), prm[1], [&](const LaneConsts<4, RQ> &k) {
                    auto residual = [&](int r) { return *(const uint32_t *)(X + at + (r < R ? r : R - 1) * P * 16); };
                    return [&, residual, q = v4acc{}, rw0 = residual(0), rw1 = residual(1), rw2 = residual(2)](int r, int e, int a) mutable {
                        q[e] = k.conv(a, e, lo2);
                        if (e == 3) {
                            *(uint32_t *)(X + at + r * P * 16) = rq_add4<RQ, RQA>(q[0], q[1], q[2], q[3], rw0, ac, k.layer);
                            rw0 = rw1; rw1 = rw2; rw2 = residual(r + 3);   // read three rows ahead
                        }
                    };
                });
            } else if constexpr (SLIM) {
                // v_mfma_i32_16x16x64_i8, a K step is a tap: lane group g holds its chunk g, a block of 16 pixels is two rows, the lane's
                // result four channels of a pixel of each of the four blocks
                const int px = lane & 15, g = lane >> 4, r = px >> 3;
                int base[4];   // by the row of the tap, mod 4, of the lane's upper pixel
#pragma unroll
                for (int j = 0; j < 4; ++j) base[j] = tile_at<C, S>(r + j, px & 7, g) - j * P * C;
                const int out = tile_at<C, S>(r + 1, (px & 7) + 1, wave) + 4 * g, out2 = tile_at<C, S>(r + 3, (px & 7) + 1, wave) + 4 * g;   // blocks 0 and 1
                auto place = [&](int nb) { return (nb & 1 ? out2 : out) + (nb >> 1) * 4 * P * C; };
                // weights w; those at `next` are fetched into `wn` meanwhile; result(block, accumulators, constants)
                auto conv = [&](const int8_t *src, const v4i (&w)[9], const int8_t *next, v4i (&wn)[9], const int *pr, auto result) {
                    slim_weights(next, wn);
                    LaneConsts<4, RQ> k(pr, C, 16 * wave + 4 * g);
                    k.fragment();
                    auto operand = [&](int ks, int nb) { const int y = 2 * nb + ks / 3; return *(const v4i *)(src + base[y & 3] + (y * P + ks % 3) * C); };
                    constexpr int RING = 3;
                    v4i b[RING][4];
                    v4acc acc[4];
#pragma unroll
                    for (int ks = 0; ks < RING - 1; ++ks)
#pragma unroll
                        for (int nb = 0; nb < 4; ++nb) b[ks][nb] = operand(ks, nb);
#pragma unroll
                    for (int nb = 0; nb < 4; ++nb) acc[nb] = bias_vector(k);
#pragma unroll
                    for (int ks = 0; ks < 9; ++ks) {
                        if (ks + RING - 1 < 9)
#pragma unroll
                            for (int nb = 0; nb < 4; ++nb) b[(ks + RING - 1) % RING][nb] = operand(ks + RING - 1, nb);
#pragma unroll
                        for (int nb = 0; nb < 4; ++nb) acc[nb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w[ks], b[ks % RING][nb], acc[nb], 0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                    }
#pragma unroll
                    for (int nb = 0; nb < 4; ++nb) result(nb, acc[nb], k);
                };
                v4i fn[9];
                conv(X, fa, cur.w2(), fn, prm[0], [&](int nb, const v4acc &a, const LaneConsts<4, RQ> &k) {
                    *(uint32_t *)(T + place(nb)) = rq_pack<RQ>(k.conv(a[0], 0, lo1), k.conv(a[1], 1, lo1), k.conv(a[2], 2, lo1), k.conv(a[3], 3, lo1), k.layer);
                });
                second_constants();
                const AddConst ac = cur.add();
                uint32_t rv[4];
#pragma unroll
                for (int nb = 0; nb < 4; ++nb) rv[nb] = *(const uint32_t *)(X + place(nb));
                conv(T, fn, nxt.w1(), fa, prm[1], [&](int nb, const v4acc &a, const LaneConsts<4, RQ> &k) {
                    *(uint32_t *)(X + place(nb)) = rq_add4<RQ, RQA>(k.conv(a[0], 0, lo2), k.conv(a[1], 1, lo2), k.conv(a[2], 2, lo2), k.conv(a[3], 3, lo2), rv[nb], ac, k.layer);
                });
            } else {
                typedef WideConv<C, S> Wide;
                constexpr int MF = Wide::MF, NF = Wide::NF, FRAGS = NI * NF * MF / NW;   // fragments per wave
                auto offset = [&](int i) { const int f = wave / MF + i * (NW / MF); return (f / NF) * TB + (f % NF) * Wide::FRAG; };
                // a lane's addresses are worked out anew for each convolution: kept across them they would be spilled
                int ln = lane;
                asm volatile("" : "+v"(ln));
                {
                    const Wide wc(ln, wave);
                    LaneConsts<16, RQ, true> k(prm[0], C, wc.mf * 32 + wc.half * 16);
                    int q[4];
                    v4i o;
                    wide_fragments<FRAGS, true>(wc, fa, k, cur.w2(), [&](int i) { return X + offset(i); }, [](int, int) {},
                        [&](int, int, int e, int a) {
                            q[e & 3] = k.conv(a, e, lo1);
                            if ((e & 3) == 3) o[e >> 2] = (int)rq_pack<RQ>(q[0], q[1], q[2], q[3], k.layer);
                        },
                        [&](int i) { *(v4i *)(T + offset(i) + wc.out) = o; });
                }
                asm volatile("" : "+v"(ln));
                second_constants();
                const AddConst ac = cur.add();
                const Wide wc(ln, wave);
                LaneConsts<16, RQ, true> k(prm[1], C, wc.mf * 32 + wc.half * 16);
                // a lane writes where it, or the lane with the other half of its pixel in this wave, has read
                const int dst = last && tail ? wc.out_strided : wc.out;
                int q[4];
                v4i o, rv[2];   // residuals of the two fragments of a group
                wide_fragments<FRAGS, RQA == RQ_PAIR>(wc, fa, k, nxt.w1(), [&](int i) { return T + offset(i); },
                    [&](int i, int j) { rv[j] = *(const v4i *)(X + offset(i) + wc.out); },
                    [&](int, int j, int e, int a) {
                        q[e & 3] = k.conv(a, e, lo2);
                        if ((e & 3) == 3) o[e >> 2] = (int)rq_add4<RQ, RQA>(q[0], q[1], q[2], q[3], (uint32_t)rv[j][e >> 2], ac, k.layer);
                    },
                    [&](int i) { *(v4i *)(X + offset(i) + dst) = o; });
            }
        });
        if constexpr (AHEAD) {
            cur = nxt;
            nxt = after;
        }
    }

    // ---- down-sampling into the next stage ----
    if constexpr (TAIL) {
        if (tail) {
            constexpr int TB2 = tile_bytes<C2, S2>(), KP1 = (9 * C + 63) / 64 * 64, KS1 = (9 * C + 31) / 32;
            static_assert(NI * TB2 <= NI * TB, "the next stage's tile fits the middle tensor's");
            typedef WideConv<C2, S2> Wide;
            constexpr int MF = Wide::MF, NF = Wide::NF, FRAGS = (NI * NF * MF + NW - 1) / NW;   // fragments per wave (of fewer fragments than waves: one of the first waves)
            constexpr int FRAG1 = 2 * (32 / S2) * P * C;   // input bytes from one output fragment to the next (an even number of rows)
            lds_barrier();            // x is complete, the last block is done with t
            fill_ring<C2, S2, NI, NT>(T, p.tzp_t, tid);
            with_form(p.tform, [&](auto rq, auto rqa) {
                constexpr int RQ = decltype(rq)::value, RQA = decltype(rqa)::value;
                int ln = lane;
                asm volatile("" : "+v"(ln));
                {
                    const Wide wc(ln, wave);
                    const int l = wc.l, half = wc.half, mf = wc.mf, c0 = mf * 32 + half * 16;
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
                        b1[ks] = tile_at<C, S, true>(2 * oy0 + tap / 3, 2 * ox + tap % 3, C == 16 ? 0 : half);
                    }
                    LaneConsts<16, RQ> k(tprm, C2, c0);
                    const bool store = !SHORT && tail == 2 && !p.head;
#pragma unroll 1
                    for (int i = 0; i < FRAGS; ++i) {
                        const int f = wave / MF + i * (NW / MF), im = f / NF;
                        if (NI * NF * MF < NW && f >= NI * NF) break;
                        const int8_t *src = X + im * TB + (f % NF) * FRAG1;
                        k.fragment();
                        v16i a = bias_vector(k);
#pragma unroll
                        for (int ks = 0; ks < KS1; ++ks)
                            a = __builtin_amdgcn_mfma_i32_32x32x32_i8(f1[ks], *(const v4i *)(src + b1[ks]), a, 0, 0, 0);
                        int q[16];
#pragma unroll
                        for (int e = 0; e < 16; ++e) q[e] = k.conv(a[e], e, p.tlo1);
                        const v4i o = rq_pack16<RQ>(q, k.layer);
                        const long g = img0 + im;
                        if (!store) *(v4i *)(T + im * TB2 + (f % NF) * wc.FRAG + wc.out) = o;
                        else if (g < p.B) *(v4i *)(p.out + ((g * S2 * S2 + (f % NF) * 32 + l) * C2 + c0)) = o;
                    }
                }
                if (tail == 1) {
                    asm volatile("" : "+v"(ln));
                    const Wide wc(ln, wave);
                    const int l = wc.l, half = wc.half, mf = wc.mf, c0 = mf * 32 + half * 16;
                    const int oy0 = l / S2, ox = l % S2;
                    v4i fa[Wide::KS];
                    wc.load_weights(p.tw2, fa);
                    const v4i fp = *(const v4i *)(p.twp + (mf * 32 + l) * 64 + half * 16);   // channels 0 .. 31 (zeros past C)
                    const int xp = tile_at<C, S, true>(2 * oy0 + 1, 2 * ox + 1, C == 16 ? 0 : half);
                    lds_barrier();
#pragma unroll 1
                    for (int i = 0; i < FRAGS; ++i) {
                        const int f = wave / MF + i * (NW / MF), im = f / NF;
                        if (NI * NF * MF < NW && f >= NI * NF) break;
                        asm volatile("" ::: "memory");   // one convolution's constants at a time
                        v4i r, y;   // the projection, the sum
                        {
                            LaneConsts<16, RQ> k(tprm + 2 * 4 * C2, C2, c0);
                            const v16i a = __builtin_amdgcn_mfma_i32_32x32x32_i8(fp, *(const v4i *)(X + im * TB + (f % NF) * FRAG1 + xp), bias_vector(k), 0, 0, 0);
                            int q[16];
#pragma unroll
                            for (int e = 0; e < 16; ++e) q[e] = k.conv(a[e], e, p.tlop);
                            r = rq_pack16<RQ>(q, k.layer);
                        }
                        asm volatile("" ::: "memory");
                        {
                            LaneConsts<16, RQ> k(tprm + 4 * C2, C2, c0);
                            const v16i a = wc.run(T + im * TB2 + (f % NF) * wc.FRAG, fa, bias_vector(k));
                            int u[16];
#pragma unroll
                            for (int e = 0; e < 16; ++e) u[e] = k.conv(a[e], e, p.tlo2);
                            const AddConst add = {p.tadd.mr, p.tadd.ms, p.tadd.c0, p.tadd.k, p.tadd.sh, p.tadd.lo};   // "self" is u here
#pragma unroll
                            for (int i = 0; i < 4; ++i) y[i] = (int)rq_add4<RQ, RQA>(u[4 * i], u[4 * i + 1], u[4 * i + 2], u[4 * i + 3], (uint32_t)r[i], add, k.layer);
                        }
                        const long g = img0 + im;
                        if (g < p.B) *(v4i *)(p.out + ((g * S2 * S2 + (f % NF) * 32 + l) * C2 + c0)) = y;
                    }
                }
            });
            if (SHORT || p.head) {   // tail == 2: the pooling reads the convolution just computed
                lds_barrier();
                if constexpr (C == 16) narrow_head<C2, S2, NI, NT>(p, T, X, img0, tid);
            }
            return;
        }
    }
    lds_barrier();
    if (!p.head) {   // the stage's result
        for (int i = tid; i < NI * S * S * CH; i += NT) {
            const int im = i / (S * S * CH), j = i % (S * S * CH), pix = j / CH, c = j % CH;
            const long g = img0 + im;
            if (g < p.B) *(v4i *)(p.out + (g * S * S + pix) * C + c * 16) = *(const v4i *)(X + im * TB + tile_at<C, S>(pix / S + 1, pix % S + 1, c));
        }
    } else {
        if constexpr (C == 64) narrow_head<C, S, NI, NT>(p, X, T, img0, tid);
    }
}

template <int C, int S, int NI, int NW>
__global__ __launch_bounds__(64 * NW, C == 16 ? 4 : 2) void narrow_kernel(const NarrowParams p) { narrow_stage<C, S, NI, NW>(p); }
// A whole net without blocks: bound by instruction issue (the noise, the requantisations) and, a few to a CU, by latencies, so that five
// workgroups a CU (92 registers, 30 KB of LDS: the sampler's table lies where the first layer then writes) instead of the general
// kernel's four (120, 39 KB) help at all sizes: us a certification with 1100 / 5100 / 20 100 copies 34.0 / 76.0 / 236 -> 32.6 / 71.6 / 218.
__global__ __launch_bounds__(256, 5) void short_net_kernel(const NarrowParams p) { narrow_stage<16, 32, 1, 4, true>(p); }

// The three stages of a net in one launch (narrow_chain_wanted): a workgroup reads back only what it has written, so that nothing but
// its barrier orders the stages; other images are at other stages meanwhile, so that the tensors have to lie apart (images_apart).
// The waves that the later stages do not take end early.
struct NarrowChain { NarrowParams stage[3]; };
__global__ __launch_bounds__(512, 2) void narrow_chain_kernel(const NarrowChain c) {
    narrow_stage<16, 32, 1, 8>(c.stage[0]);
    __syncthreads();   // the stage's result is stored
    if (threadIdx.x >= 256) return;
    narrow_stage<32, 16, 1, 4>(c.stage[1]);
    __syncthreads();
    narrow_stage<64, 8, 1, 4>(c.stage[2]);
}

template <int C, int S, int NI, int NW>
hipError_t launch_stage(const NarrowParams &p, hipStream_t st) {
    static const std::string name = "narrow_kernel<" + std::to_string(C) + ", " + std::to_string(S) + ", " + std::to_string(NI) + (NW == 4 ? "" : ", " + std::to_string(NW) + " waves") + ">";
    set_kernel_name(name.c_str());
    hipLaunchKernelGGL((narrow_kernel<C, S, NI, NW>), dim3((unsigned)((p.B + NI - 1) / NI)), dim3(64 * NW), 0, st, p);
    return hipGetLastError();
}

hipError_t launch_short(const NarrowParams &p, hipStream_t st) {
    set_kernel_name("short_net_kernel");
    hipLaunchKernelGGL(short_net_kernel, dim3((unsigned)p.B), dim3(256), 0, st, p);
    return hipGetLastError();
}
}  // namespace

bool narrow_short(const NarrowParams &p) { return p.stem && p.nblocks == 0 && p.tail == 2 && p.head; }

// Shapes with a kernel: identity blocks of 16 channels at 32 x 32, 32 at 16 x 16, 64 at 8 x 8 (the three stages of
// the CIFAR-style residual nets), down-sampling blocks 16 -> 32 at 32 x 32 -> 16 x 16 and 32 -> 64 at 16 x 16 -> 8 x 8.
bool basic_block_supported(int channels, int size) {
    return (channels == 16 && size == 32) || (channels == 32 && size == 16) || (channels == 64 && size == 8);
}
bool trans_block_supported(int cout, int size_out) { return (cout == 32 && size_out == 16) || (cout == 64 && size_out == 8); }

static bool narrow_valid(const NarrowParams &p, int channels) {
    const bool from_image = channels == 16 && p.stem;
    if ((p.nblocks > 0 && !p.blocks) || p.nblocks < 0 || (p.nblocks == 0 && !p.tail && !from_image) || (!p.head && !p.out) ||
        (from_image ? !p.w0 || !p.prm0 || (!p.fused_noise && !p.in) : !p.in || p.stem))
        return false;
    if (p.fused_noise) {
        const NoiseSource &ns = p.noise;
        if (!from_image || !ns.x || !ns.table || ns.C < 1 || ns.C > 3 || ns.H != 32 || ns.W != 32 || !valid_slots(ns.slots)) return false;
    }
    if (p.tail && (channels == 64 || !p.tw1 || !p.tprm || (p.tail == 1 && (!p.tw2 || !p.twp)) || p.tail > 2)) return false;
    if (p.head && (!(channels == 64 || (channels == 16 && p.tail == 2)) || (p.tail && channels == 64) || !p.fc_w || !p.fc_bias || p.classes < 1 ||
                   p.classes_p < p.classes || (channels == 64 && p.nblocks == 0)))
        return false;
    if (p.head && p.counts && !valid_slots(p.slots)) return false;
    if (p.parts && (!p.head || !p.counts || (uint64_t)(p.slots.n[1] ? 2 : 1) * p.slots.pairs * (uint64_t)p.classes > SENT_TALLIES)) return false;
    if (p.tallies && (!p.parts || p.tallies > SENT_TALLIES || !p.tally_host || !p.flag)) return false;
    if (p.votes && (!p.head || p.counts || p.slots.begin + (uint64_t)p.B > DIRECT_VOTES)) return false;
    return true;
}

hipError_t launch_narrow(const NarrowParams &p, int channels, hipStream_t st) {
    if (p.B <= 0) return hipSuccess;
    if (!narrow_valid(p, channels)) return hipErrorInvalidValue;
    // Images per workgroup: one while there is a CU for each; two while all workgroups run at once (two per CU); beyond, as many
    // as fit, to share the weights.  A second image in a workgroup costs about what a second workgroup on its CU costs with
    // 32 channels, and less with 64: us of the two stages of ResNet-20 with one / two / most images a workgroup
    //   copies        256              384              512              768              1024             1536
    //   32 channels   13 / 18 / 21     17 / 18 / 21     18 / 18 / 21     22 / 24 / 22     27 / 24 / 29     36 / 35 / 31
    //   64 channels   15 / 15 / 24     19 / 16 / 24     20 / 17 / 24     27 / 20 / 25     32 / 21 / 25     45 / 29 / 27
    const bool one = p.B <= 256, two = p.B <= 1024;
    // Waves: eight for 16 channels while every image has a CU for itself, where a convolution is a chain of latencies (first kernel of
    // ResNet-20 / -110 at 100 copies 2.1 / 11 us shorter; from two workgroups a CU on the same or longer: 300 copies + 0.2,
    // 1000 + 2).  At 32 channels four waves stay ahead at all sizes: each fetches the whole weight matrix (3 us more for 9 blocks).
    // (A net of two convolutions with 156 / 256 copies 21.1 / 21.8 us so, 22.5 / 22.9 by its own kernel's four waves; that is ahead from there on.)
    if (channels == 16 && !one && narrow_short(p)) return launch_short(p, st);
    if (channels == 16) return one ? launch_stage<16, 32, 1, 8>(p, st) : launch_stage<16, 32, 1, 4>(p, st);
    if (channels == 32) return one ? launch_stage<32, 16, 1, 4>(p, st) : two ? launch_stage<32, 16, 2, 4>(p, st) : launch_stage<32, 16, 3, 4>(p, st);
    if (channels == 64) return one ? launch_stage<64, 8, 1, 4>(p, st) : two ? launch_stage<64, 8, 2, 4>(p, st) : launch_stage<64, 8, 6, 4>(p, st);
    return hipErrorInvalidValue;
}

// All stages in one launch while every image has a CU for itself: predictions with 100 copies 45.8 -> 42.6 us (ResNet-20), 148 -> 145
// (ResNet-110), with 250 47.6 -> 44.0.  The kernel takes the registers of the widest stage, one workgroup a CU: a 257th image
// would wait for a whole round, where three launches share the CUs (300 copies 60 us).
bool narrow_chain_wanted(int copies) { return copies <= 256; }

hipError_t launch_narrow_chain(const NarrowParams &s16, const NarrowParams &s32, const NarrowParams &s64, hipStream_t st) {
    if (s16.B <= 0) return hipSuccess;
    if (!narrow_valid(s16, 16) || !narrow_valid(s32, 32) || !narrow_valid(s64, 64) || s16.B != s32.B || s16.B != s64.B || s16.tail != 1 || s32.tail != 1 || s16.head ||
        s16.out != s32.in || s32.out != s64.in)
        return hipErrorInvalidValue;
    set_kernel_name("narrow_chain_kernel");
    hipLaunchKernelGGL(narrow_chain_kernel, dim3((unsigned)s16.B), dim3(512), 0, st, NarrowChain{{s16, s32, s64}});
    return hipGetLastError();
}

}  // namespace isr
