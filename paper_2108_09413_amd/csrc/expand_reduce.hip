// The closing 1x1 convolution + residual add of a bottleneck block with 128 middle channels and the opening
// 1x1 convolution of the NEXT block in one kernel: y = add(requant(W3 t2), x) is written once and the next
// block's t1' = relu(requant(W1' y)) is computed from the copy of y that is still in LDS, so the 512-channel
// tensor is not read back from memory by a second kernel.
//
// A workgroup of eight waves owns 32 consecutive pixels with ALL 512 channels and walks over such tiles
// (persistent grid).  Per tile:
//   * x (32 x 512 bytes) and t2 (32 x 128 bytes) arrive by direct-to-LDS loads two tiles ahead (three buffers);
//   * expand: wave w computes channels 64 w .. 64 w + 63 of the 32 pixels (two 32x32x32 MFMA tiles, K = 128);
//     its weight fragments stay in registers for the whole launch (fragment-major copy of the weights, made
//     when the model is loaded), the pixel fragments come from the t2 tile;
//   * the epilogue requantises, reads the residual from the x tile, adds, writes y to memory AND over x in LDS;
//   * reduce: wave w computes output channels 16 w .. 16 w + 15 of the 32 pixels with v_mfma_i32_16x16x64_i8
//     over K = 512 channels of the y tile (its weight fragments, too, stay in registers), requantises and
//     stores t1'.
// Two barriers per tile.  LDS rows of the x / y tile are 512 bytes: 16-byte chunk c of pixel p sits at chunk
// c ^ (p & 15), so that 16 consecutive pixels reading one logical chunk cover the 64 banks exactly once, for the
// epilogue's 32x32 layout and for the 16x16x64 fragment reads alike.
//
// A second kernel does the same for a stage's FIRST block, whose residual is not a stored tensor but a projection
// 1x1 convolution (256 -> 512 channels) of the block input: y = add(requant(W3 t2), requant(Wp x0)).  Sixteen waves,
// 32 channels each, hold the fragments of all three weight matrices; x0 (32 x 256 bytes) takes the place of x
// among the loads and the y tile is written, not overwritten.
#include "conv_device.h"

namespace isr {

namespace {

constexpr int XK1 = 128, XC = 512, XN2 = 128, XPX = 32, XNW = 8, XNT = XNW * 64;
constexpr int XNB = 3;   // tile buffers: loads run two tiles ahead

template <int RQ, int RQA>
__global__ __launch_bounds__(XNT, 4) void expand_reduce_kernel(const XrParams p) {
    __shared__ __attribute__((aligned(256))) int8_t XY[XNB][XPX * XC];
    __shared__ __attribute__((aligned(16))) int8_t T2[XNB][XPX * XK1];
    __shared__ __attribute__((aligned(16))) int prm1[4][XC];    // bias, M0, chi, shift-1 of the expanding convolution
    __shared__ __attribute__((aligned(16))) int prm2[4][XN2];   // the same of the reducing convolution

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ntiles = (p.npix + XPX - 1) / XPX, G = gridDim.x;
    const AddConst ac = add_const<RQA>(p);
    const uint32_t xy_lds = lds_address(&XY[0][0]), t2_lds = lds_address(&T2[0][0]);

    // direct-to-LDS loads of a tile: wave-load q of the x tile covers pixels 2 q, 2 q + 1 (wave w issues q = 2 w,
    // 2 w + 1); wave-load q of the t2 tile covers pixels 8 q .. 8 q + 7 (waves 0 .. 3).  Pixels past the end
    // re-read the last pixel; their results are never stored.
    auto issue_tile = [&](int tile, int buf) {
        const int n0 = tile * XPX;
        int l = lane;
        asm volatile("" : "+v"(l));   // recompute the per-lane offsets per call: kept across the tile loop they would be spilled
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int q = 2 * wave + j, px = 2 * q + (l >> 5), c = (l & 31) ^ (px & 15);
            int n = n0 + px;
            n = n < p.npix ? n : p.npix - 1;
            ISR_GLOBAL_TO_LDS16_AT(p.x + ((uint32_t)n * (uint32_t)XC + (uint32_t)(c * 16)), xy_lds + buf * (XPX * XC) + q * 1024);
        }
        if (wave < 4) {
            const int row = 8 * wave + (l >> 3), c = (l & 7) ^ swz<8>(row);
            int n = n0 + row;
            n = n < p.npix ? n : p.npix - 1;
            ISR_GLOBAL_TO_LDS16_AT(p.t2 + ((uint32_t)n * (uint32_t)XK1 + (uint32_t)(c * 16)), t2_lds + buf * (XPX * XK1) + wave * 1024);
        }
    };

    int tile = blockIdx.x;
    if (tile < ntiles) issue_tile(tile, 0);
    if (tile + G < ntiles) issue_tile(tile + G, 1);
    // constants and weights, all on their way before any is waited for
    const int i1 = tid < XC ? tid : 0, i2 = tid < XN2 ? tid : 0;
    const RqRaw r1 = rq_fetch(p.bias1, p.m0s1, p.chi1, p.shm11, i1), r2 = rq_fetch(p.bias2, p.m0s2, p.chi2, p.shm12, i2);
    // weight fragments, kept in registers for the whole launch: expand [fm][ksub] (32 output channels x 32 K bytes
    // each), reduce [kstep] (16 output channels x 64 K bytes each)
    const uint32_t lane16 = (uint32_t)lane * 16;
    v4i a1[2][XK1 / 32], a2[XC / 64];
#pragma unroll
    for (int fm = 0; fm < 2; ++fm)
#pragma unroll
        for (int ks = 0; ks < XK1 / 32; ++ks)
            a1[fm][ks] = *(const v4i *)(p.a1 + (size_t)wave * (2 * (XK1 / 32) * 1024) + (lane16 + (uint32_t)((fm * (XK1 / 32) + ks) * 1024)));
#pragma unroll
    for (int ks = 0; ks < XC / 64; ++ks) a2[ks] = *(const v4i *)(p.a2 + (size_t)wave * (XC / 64) * 1024 + (lane16 + (uint32_t)(ks * 1024)));
    if (tid < XC) rq_store<RQ>(prm1, r1, i1);
    if (tid < XN2) rq_store<RQ>(prm2, r2, i2);
    wait_vmcnt<0>();
    __syncthreads();   // the constants are in LDS, the first tile has landed
    const RqLayer L1 = rq_layer<RQ>(prm1[2][0], prm1[3][0]), L2 = rq_layer<RQ>(prm2[2][0], prm2[3][0]);

    int buf = 0;
    for (int it = 0; tile < ntiles; tile += G, ++it) {
        const int n0 = tile * XPX;
        // per-lane positions, recomputed per tile (a handful of instructions) instead of held in registers next to the
        // 64 registers of weight fragments
        int l = lane;
        asm volatile("" : "+v"(l));
        const int half = l >> 5, px1 = l & 31;            // expand: the lane's pixel and channel half
        const int g = l >> 4, px2 = l & 15;               // reduce: the lane's K / channel group and pixel
        const int b_off1 = px1 * XK1 + ((half ^ swz<8>(px1)) << 4);   // t2 fragment of K sub-step 0; sub-step k flips bits 5..6 by k
        const bool prefetch = tile + 2 * G < ntiles;
        if (it > 0) {
            // The loads of this tile were issued two tiles ago.  Vector memory operations complete in issue order, so
            // they have landed once at most the operations issued after them are outstanding: the four stores of each of
            // the two tiles since, and the loads of the tile issued one tile ago (three for waves 0 .. 3, two for the
            // others).  Where the sequence differs (the second tile, which has one tile of stores behind it) the wave
            // waits for everything.
            if (it >= 2 && tile + G < ntiles) {
                if (wave < 4) wait_vmcnt<11>();
                else wait_vmcnt<10>();
            } else {
                wait_vmcnt<0>();
            }
            lds_barrier();   // every wave's loads of this tile landed; every wave is done with the previous tile's buffers
        }
        if (prefetch) issue_tile(tile + 2 * G, buf >= 1 ? buf - 1 : XNB - 1);   // the buffer of the previous tile

        // ---- expand: 64 channels x 32 pixels per wave, 32 channels at a time ----
        const int8_t *t2b = T2[buf];
        int8_t *xyb = XY[buf];
        const long n1 = (long)n0 + px1;
#pragma unroll
        for (int fm = 0; fm < 2; ++fm) {
            const int oc = wave * 64 + fm * 32 + half * 16;
            v16i acc;
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] = prm1[0][oc + i];
#pragma unroll
            for (int ks = 0; ks < XK1 / 32; ++ks) {
                const v4i fb = *(const v4i *)(t2b + (b_off1 ^ (ks << 5)));
                acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a1[fm][ks], fb, acc, 0, 0, 0);
            }
            int8_t *cell = xyb + px1 * XC + ((((oc >> 4)) ^ (px1 & 15)) << 4);
            const v4i rv = *(const v4i *)cell;
            v4i yv;
            // four channels at a time: their constants are three 16-byte LDS reads, the results one packed dword
#pragma unroll
            for (int gi = 0; gi < 4; ++gi) {
                const v4i mm = *(const v4i *)&prm1[1][oc + 4 * gi], ch = rq_chi4<RQ>(&prm1[2][oc + 4 * gi]), ss = *(const v4i *)&prm1[3][oc + 4 * gi];
                int q[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) q[i] = rq_conv<RQ>(acc[4 * gi + i], mm[i], ch[i], ss[i], p.lo1, L1);
                yv[gi] = (int)rq_add4<RQ, RQA>(q[0], q[1], q[2], q[3], (uint32_t)rv[gi], ac, L1);
            }
            *(v4i *)cell = yv;
            if (n1 < p.npix) *(v4i *)(p.y + n1 * XC + oc) = yv;
        }
        lds_barrier();   // the y tile is complete (its stores to memory may still be under way)
        asm volatile("" ::: "memory");

        // ---- reduce: 16 channels x 32 pixels per wave, K = 512 channels of the y tile ----
        v4acc acc2[2];
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc2[nb][i] = prm2[0][wave * 16 + g * 4 + i];
#pragma unroll
        for (int ks = 0; ks < XC / 64; ++ks) {
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) {
                const int px = px2 + 16 * nb;
                const v4i fb = *(const v4i *)(xyb + px * XC + (((4 * ks + g) ^ px2) << 4));
                acc2[nb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a2[ks], fb, acc2[nb], 0, 0, 0);
            }
        }
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            const long n2 = (long)n0 + px2 + 16 * nb;
            int q[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int c = wave * 16 + g * 4 + i;
                q[i] = rq_conv<RQ>(acc2[nb][i], prm2[1][c], prm2[2][rq_chi_at<RQ>(c)], prm2[3][c], p.lo2, L2);
            }
            if (n2 < p.npix) *(uint32_t *)(p.t1n + n2 * XN2 + wave * 16 + g * 4) = rq_pack<RQ>(q[0], q[1], q[2], q[3], L2);
        }
        buf = buf + 1 == XNB ? 0 : buf + 1;
    }
}

// ---- the same with the residual computed by a projection convolution of the block input ----

constexpr int XPK = 256, XNW2 = 16, XNT2 = XNW2 * 64;

template <int RQ, int RQA>
__global__ __launch_bounds__(XNT2, 4) void proj_expand_reduce_kernel(const XrParams p) {
    __shared__ __attribute__((aligned(256))) int8_t Y[2][XPX * XC];   // one is reduced while the next is made
    __shared__ __attribute__((aligned(256))) int8_t X0[XNB][XPX * XPK];
    __shared__ __attribute__((aligned(16))) int8_t T2[XNB][XPX * XK1];
    __shared__ __attribute__((aligned(16))) int prm1[4][XC];    // bias, M0, chi, shift-1 of the expanding convolution
    __shared__ __attribute__((aligned(16))) int prmp[4][XC];    // of the projection
    __shared__ __attribute__((aligned(16))) int prm2[4][XN2];   // of the reducing convolution

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ntiles = (p.npix + XPX - 1) / XPX, G = gridDim.x;
    const AddConst ac = add_const<RQA>(p);
    const uint32_t x0_lds = lds_address(&X0[0][0]), t2_lds = lds_address(&T2[0][0]);

    // direct-to-LDS loads of a tile: wave-load q of the x0 tile covers pixels 4 q .. 4 q + 3 (waves 0 .. 7), wave-load q
    // of the t2 tile pixels 8 q .. 8 q + 7 (waves 8 .. 11)
    auto issue_tile = [&](int tile, int buf) {
        const int n0 = tile * XPX;
        int l = lane;
        asm volatile("" : "+v"(l));   // recompute the per-lane offsets per call: kept across the tile loop they would be spilled
        if (wave < 8) {
            const int px = 4 * wave + (l >> 4), c = (l & 15) ^ (px & 15);
            int n = n0 + px;
            n = n < p.npix ? n : p.npix - 1;
            // the projection may be strided: output pixel (b, y, x) reads input pixel (b, s y, s x)
            const int HoWo = p.Ho * p.Wo, b = n / HoWo, rem = n - b * HoWo, y = rem / p.Wo, x = rem - y * p.Wo;
            const uint32_t src = (uint32_t)((b * p.Hin + y * p.pstride) * p.Win + x * p.pstride);
            ISR_GLOBAL_TO_LDS16_AT(p.in2 + (src * (uint32_t)XPK + (uint32_t)(c * 16)), x0_lds + buf * (XPX * XPK) + wave * 1024);
        } else if (wave < 12) {
            const int q = wave - 8, row = 8 * q + (l >> 3), c = (l & 7) ^ swz<8>(row);
            int n = n0 + row;
            n = n < p.npix ? n : p.npix - 1;
            ISR_GLOBAL_TO_LDS16_AT(p.t2 + ((uint32_t)n * (uint32_t)XK1 + (uint32_t)(c * 16)), t2_lds + buf * (XPX * XK1) + q * 1024);
        }
    };

    int tile = blockIdx.x;
    if (tile < ntiles) issue_tile(tile, 0);
    if (tile + G < ntiles) issue_tile(tile + G, 1);
    if (tile + 2 * G < ntiles) issue_tile(tile + 2 * G, 2);
    // constants and weights, all on their way before any is waited for
    const int i1 = tid < XC ? tid : 0, i2 = tid < XN2 ? tid : 0;
    const RqRaw r1 = rq_fetch(p.bias1, p.m0s1, p.chi1, p.shm11, i1), r2 = rq_fetch(p.bias2, p.m0s2, p.chi2, p.shm12, i2);
    const RqRaw rp = rq_fetch(p.biasp, p.m0sp, p.chip, p.shm1p, i1);
    // weight fragments, kept in registers for the whole launch: wave w owns channels 32 w .. 32 w + 31 of the expanding
    // convolution [ksub] and of the projection [ksub], and 16 channels x 16 pixels of the reducing convolution [kstep]
    const uint32_t lane16 = (uint32_t)lane * 16;
    v4i a1[XK1 / 32], ap[XPK / 32], a2[XC / 64];
#pragma unroll
    for (int ks = 0; ks < XK1 / 32; ++ks) a1[ks] = *(const v4i *)(p.a1 + (size_t)wave * (XK1 / 32) * 1024 + (lane16 + (uint32_t)(ks * 1024)));
#pragma unroll
    for (int ks = 0; ks < XPK / 32; ++ks) ap[ks] = *(const v4i *)(p.ap + (size_t)wave * (XPK / 32) * 1024 + (lane16 + (uint32_t)(ks * 1024)));
#pragma unroll
    for (int ks = 0; ks < XC / 64; ++ks) a2[ks] = *(const v4i *)(p.a2 + (size_t)(wave >> 1) * (XC / 64) * 1024 + (lane16 + (uint32_t)(ks * 1024)));
    if (tid < XC) {
        rq_store<RQ>(prm1, r1, i1);
        rq_store<RQ>(prmp, rp, i1);
    }
    if (tid < XN2) rq_store<RQ>(prm2, r2, i2);
    wait_vmcnt<0>();
    __syncthreads();   // the constants are in LDS, the first tile has landed
    const RqLayer L1 = rq_layer<RQ>(prm1[2][0], prm1[3][0]), L2 = rq_layer<RQ>(prm2[2][0], prm2[3][0]);
    const RqLayer Lp = rq_layer<RQ>(prmp[2][0], prmp[3][0]);

    // the y tile: projection of the block input (the residual), expand, add; 32 channels x 32 pixels per wave
    auto make = [&](int tile, int buf, int8_t *Yb) {
        if constexpr (RQ == RQ_PAIR) __builtin_amdgcn_s_setprio(3);
        int l = lane;
        asm volatile("" : "+v"(l));   // per-lane values are recomputed per tile
        const int half = l >> 5, px1 = l & 31, oc = wave * 32 + half * 16;
        v4i rq;
        {
            v16i acc;
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] = prmp[0][oc + i];
            const int8_t *xb = X0[buf];
            const int x_off = px1 * XPK + ((half ^ (px1 & 15)) << 4);   // chunk (2 k + half) ^ (px & 15): sub-step k flips bits 5..7 by k
            auto operand = [&](int ks) { return *(const v4i *)(xb + (x_off ^ (ks << 5))); };
            v4i fb[3] = {operand(0), operand(1)};
#pragma unroll
            for (int ks = 0; ks < XPK / 32; ++ks) {
                if (ks + 2 < XPK / 32) fb[(ks + 2) % 3] = operand(ks + 2);
                acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(ap[ks], fb[ks % 3], acc, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int gi = 0; gi < 4; ++gi) {
                __builtin_amdgcn_sched_barrier(0);   // one group's constants at a time: the registers are needed for weight fragments
                const v4i mm = *(const v4i *)&prmp[1][oc + 4 * gi], ch = rq_chi4<RQ>(&prmp[2][oc + 4 * gi]), ss = *(const v4i *)&prmp[3][oc + 4 * gi];
                int q[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) q[i] = rq_conv<RQ>(acc[4 * gi + i], mm[i], ch[i], ss[i], p.lop, Lp);
                rq[gi] = (int)rq_pack<RQ>(q[0], q[1], q[2], q[3], Lp);
            }
        }
        if constexpr (RQ == RQ_PAIR) __builtin_amdgcn_s_setprio(2);
        {
            v16i acc;
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] = prm1[0][oc + i];
            const int8_t *t2b = T2[buf];
            const int b_off1 = px1 * XK1 + ((half ^ swz<8>(px1)) << 4);
            auto operand = [&](int ks) { return *(const v4i *)(t2b + (b_off1 ^ (ks << 5))); };
            v4i fb[3] = {operand(0), operand(1)};
#pragma unroll
            for (int ks = 0; ks < XK1 / 32; ++ks) {
                if (ks + 2 < XK1 / 32) fb[(ks + 2) % 3] = operand(ks + 2);
                acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a1[ks], fb[ks % 3], acc, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (RQ == RQ_PAIR) __builtin_amdgcn_s_setprio(1);
            v4i yv;
#pragma unroll
            for (int gi = 0; gi < 4; ++gi) {
                __builtin_amdgcn_sched_barrier(0);
                const v4i mm = *(const v4i *)&prm1[1][oc + 4 * gi], ch = rq_chi4<RQ>(&prm1[2][oc + 4 * gi]), ss = *(const v4i *)&prm1[3][oc + 4 * gi];
                int q[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) q[i] = rq_conv<RQ>(acc[4 * gi + i], mm[i], ch[i], ss[i], p.lo1, L1);
                yv[gi] = (int)rq_add4<RQ, RQA>(q[0], q[1], q[2], q[3], (uint32_t)rq[gi], ac, L1);
            }
            *(v4i *)(Yb + px1 * XC + (((oc >> 4) ^ (px1 & 15)) << 4)) = yv;
            const long n1 = (long)tile * XPX + px1;
            if (n1 < p.npix) *(v4i *)(p.y + n1 * XC + oc) = yv;
        }
    };
    // reduce: wave w computes channels 16 (w / 2) .. + 15 of pixels 16 (w % 2) .. + 15
    auto reduce = [&](int tile, const int8_t *Yb) {
        int l = lane;
        asm volatile("" : "+v"(l));
        const int g = l >> 4, px2 = l & 15, mb = wave >> 1, px = px2 + 16 * (wave & 1);
        v4acc acc2;
#pragma unroll
        for (int i = 0; i < 4; ++i) acc2[i] = prm2[0][mb * 16 + g * 4 + i];
        auto operand = [&](int ks) { return *(const v4i *)(Yb + px * XC + (((4 * ks + g) ^ px2) << 4)); };
        v4i fb[4] = {operand(0), operand(1), operand(2)};
#pragma unroll
        for (int ks = 0; ks < XC / 64; ++ks) {
            if (ks + 3 < XC / 64) fb[(ks + 3) % 4] = operand(ks + 3);
            acc2 = __builtin_amdgcn_mfma_i32_16x16x64_i8(a2[ks], fb[ks % 4], acc2, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        int q[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int c = mb * 16 + g * 4 + i;
            q[i] = rq_conv<RQ>(acc2[i], prm2[1][c], prm2[2][rq_chi_at<RQ>(c)], prm2[3][c], p.lo2, L2);
        }
        const long n2 = (long)tile * XPX + px;
        if (n2 < p.npix) *(uint32_t *)(p.t1n + n2 * XN2 + mb * 16 + g * 4) = rq_pack<RQ>(q[0], q[1], q[2], q[3], L2);
    };

    // One barrier a tile: between two of them the workgroup reduces a tile and makes the next, half of the waves of each SIMD in this order,
    // the others in the other, so that one half's MFMAs and LDS reads stand beside the other's arithmetic (two barriers, all waves in step:
    // 226 -> 219 us for 668 copies; expand_reduce256_kernel 200 -> 189).
    // The fewer steps a wave has behind it, the higher its priority: in the hardware's order the oldest wave of a SIMD reaches the barrier
    // long before the youngest, which then runs alone (214 -> 210 us; expand_reduce256_kernel 185 -> 183, expand_reduce1024_kernel 103 -> 100; in
    // expand_reduce_kernel, whose CUs hold two workgroups, 149 -> 151, so not there; 4 % in all forms of expand_reduce1024_kernel, 0 to 4 % in those of
    // expand_reduce256_kernel).  In the pair form: in the others of this kernel the compiler would spill around them.
    if (tile < ntiles) make(tile, 0, Y[0]);
    int buf = 0;
    for (int it = 0; tile < ntiles; tile += G, ++it) {
        const int nbuf = buf + 1 == XNB ? 0 : buf + 1;
        const bool more = tile + G < ntiles;
        if (more) {
            // Vector memory operations complete in issue order: the loads of the next tile, issued two intervals ago, have landed once at most
            // what was issued after them is outstanding: two stores in each interval since and the load of the tile behind (waves 0 .. 11).
            if (it >= 2 && tile + 2 * G < ntiles) {
                if (wave < 12) wait_vmcnt<5>();
                else wait_vmcnt<4>();
            } else {
                wait_vmcnt<0>();
            }
        }
        lds_barrier();   // this tile's y is complete, the next tile's operands have landed, everybody is done with the tile before
        if (tile + 3 * G < ntiles) issue_tile(tile + 3 * G, buf);
        asm volatile("" ::: "memory");   // the stores that the wait counts come behind these loads
        if (wave >= 8) {
            if (more) make(tile + G, nbuf, Y[(it + 1) & 1]);
            if constexpr (RQ == RQ_PAIR) __builtin_amdgcn_s_setprio(0);
            reduce(tile, Y[it & 1]);
        } else {
            if constexpr (RQ == RQ_PAIR) __builtin_amdgcn_s_setprio(3);
            reduce(tile, Y[it & 1]);
            if (more) make(tile + G, nbuf, Y[(it + 1) & 1]);
        }
        buf = nbuf;
    }
}

// ---- identity block followed by a block with 256 middle channels (the first block of the next stage) ----
// As expand_reduce_kernel, but the reducing convolution has 256 outputs: sixteen waves, wave w owns channels
// 32 w .. 32 w + 31 of the expanding convolution and channels 16 w .. 16 w + 15 (all 32 pixels) of the reducing one.

constexpr int XN2W = 256;

template <int RQ, int RQA>
__global__ __launch_bounds__(XNT2, 4) void expand_reduce256_kernel(const XrParams p) {
    __shared__ __attribute__((aligned(256))) int8_t XY[XNB + 1][XPX * XC];   // one is reduced, one expanded into, two are on their way
    __shared__ __attribute__((aligned(16))) int8_t T2[XNB + 1][XPX * XK1];
    __shared__ __attribute__((aligned(16))) int prm1[4][XC];     // bias, M0, chi, shift-1 of the expanding convolution
    __shared__ __attribute__((aligned(16))) int prm2[4][XN2W];   // of the reducing convolution

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ntiles = (p.npix + XPX - 1) / XPX, G = gridDim.x;
    const AddConst ac = add_const<RQA>(p);
    const uint32_t xy_lds = lds_address(&XY[0][0]), t2_lds = lds_address(&T2[0][0]);

    // direct-to-LDS loads of a tile: wave w fetches pixels 2 w, 2 w + 1 of the x tile, waves 0 .. 3 also pixels
    // 8 w .. 8 w + 7 of the t2 tile
    auto issue_tile = [&](int tile, int buf) {
        const int n0 = tile * XPX;
        int l = lane;
        asm volatile("" : "+v"(l));   // recompute the per-lane offsets per call: kept across the tile loop they would be spilled
        {
            const int px = 2 * wave + (l >> 5), c = (l & 31) ^ (px & 15);
            int n = n0 + px;
            n = n < p.npix ? n : p.npix - 1;
            ISR_GLOBAL_TO_LDS16_AT(p.x + ((uint32_t)n * (uint32_t)XC + (uint32_t)(c * 16)), xy_lds + buf * (XPX * XC) + wave * 1024);
        }
        if (wave < 4) {
            const int row = 8 * wave + (l >> 3), c = (l & 7) ^ swz<8>(row);
            int n = n0 + row;
            n = n < p.npix ? n : p.npix - 1;
            ISR_GLOBAL_TO_LDS16_AT(p.t2 + ((uint32_t)n * (uint32_t)XK1 + (uint32_t)(c * 16)), t2_lds + buf * (XPX * XK1) + wave * 1024);
        }
    };

    int tile = blockIdx.x;
    if (tile < ntiles) issue_tile(tile, 0);
    if (tile + G < ntiles) issue_tile(tile + G, 1);
    if (tile + 2 * G < ntiles) issue_tile(tile + 2 * G, 2);
    // constants and weights, all on their way before any is waited for
    const int i1 = tid < XC ? tid : 0, i2 = tid < XN2W ? tid : 0;
    const RqRaw r1 = rq_fetch(p.bias1, p.m0s1, p.chi1, p.shm11, i1), r2 = rq_fetch(p.bias2, p.m0s2, p.chi2, p.shm12, i2);
    const uint32_t lane16 = (uint32_t)lane * 16;
    v4i a1[XK1 / 32], a2[XC / 64];   // weight fragments, kept in registers for the whole launch
#pragma unroll
    for (int ks = 0; ks < XK1 / 32; ++ks) a1[ks] = *(const v4i *)(p.a1 + (size_t)wave * (XK1 / 32) * 1024 + (lane16 + (uint32_t)(ks * 1024)));
#pragma unroll
    for (int ks = 0; ks < XC / 64; ++ks) a2[ks] = *(const v4i *)(p.a2 + (size_t)wave * (XC / 64) * 1024 + (lane16 + (uint32_t)(ks * 1024)));
    if (tid < XC) rq_store<RQ>(prm1, r1, i1);
    if (tid < XN2W) rq_store<RQ>(prm2, r2, i2);
    wait_vmcnt<0>();
    __syncthreads();   // the constants are in LDS, the first tile has landed
    const RqLayer L1 = rq_layer<RQ>(prm1[2][0], prm1[3][0]), L2 = rq_layer<RQ>(prm2[2][0], prm2[3][0]);

    // expand + add into the tile of x: 32 channels x 32 pixels per wave
    auto expand = [&](int tile, int buf) {
        __builtin_amdgcn_s_setprio(3);
        int l = lane;
        asm volatile("" : "+v"(l));   // per-lane values are recomputed per tile
        const int half = l >> 5, px1 = l & 31, oc = wave * 32 + half * 16;
        v16i acc;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = prm1[0][oc + i];
        const int8_t *t2b = T2[buf];
        const int b_off1 = px1 * XK1 + ((half ^ swz<8>(px1)) << 4);
        v4i fb[XK1 / 32];
#pragma unroll
        for (int ks = 0; ks < XK1 / 32; ++ks) fb[ks] = *(const v4i *)(t2b + (b_off1 ^ (ks << 5)));
        int8_t *cell = XY[buf] + px1 * XC + (((oc >> 4) ^ (px1 & 15)) << 4);
        const v4i rv = *(const v4i *)cell;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < XK1 / 32; ++ks) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a1[ks], fb[ks], acc, 0, 0, 0);
        v4i yv;
#pragma unroll
        for (int gi = 0; gi < 4; ++gi) {
            __builtin_amdgcn_sched_barrier(0);
            if (gi == 0) __builtin_amdgcn_s_setprio(2);
            if (gi == 2) __builtin_amdgcn_s_setprio(1);
            const v4i mm = *(const v4i *)&prm1[1][oc + 4 * gi], ch = rq_chi4<RQ>(&prm1[2][oc + 4 * gi]), ss = *(const v4i *)&prm1[3][oc + 4 * gi];
            int q[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) q[i] = rq_conv<RQ>(acc[4 * gi + i], mm[i], ch[i], ss[i], p.lo1, L1);
            yv[gi] = (int)rq_add4<RQ, RQA>(q[0], q[1], q[2], q[3], (uint32_t)rv[gi], ac, L1);
        }
        *(v4i *)cell = yv;
        const long n1 = (long)tile * XPX + px1;
        if (n1 < p.npix) *(v4i *)(p.y + n1 * XC + oc) = yv;
    };
    // reduce: wave w computes channels 16 w .. 16 w + 15 of the 32 pixels; pixel fragments read two K steps ahead
    auto reduce = [&](int tile, int buf) {
        int l = lane;
        asm volatile("" : "+v"(l));
        const int g = l >> 4, px2 = l & 15;
        v4acc acc2[2];
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc2[nb][i] = prm2[0][wave * 16 + g * 4 + i];
        auto operand = [&](int ks, int nb) { return *(const v4i *)(XY[buf] + (px2 + 16 * nb) * XC + (((4 * ks + g) ^ px2) << 4)); };
        v4i fb[3][2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) fb[ks][nb] = operand(ks, nb);
#pragma unroll
        for (int ks = 0; ks < XC / 64; ++ks) {
            if (ks + 2 < XC / 64)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) fb[(ks + 2) % 3][nb] = operand(ks + 2, nb);
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) acc2[nb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a2[ks], fb[ks % 3][nb], acc2[nb], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            const long n2 = (long)tile * XPX + px2 + 16 * nb;
            int q[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int c = wave * 16 + g * 4 + i;
                q[i] = rq_conv<RQ>(acc2[nb][i], prm2[1][c], prm2[2][rq_chi_at<RQ>(c)], prm2[3][c], p.lo2, L2);
            }
            if (n2 < p.npix) *(uint32_t *)(p.t1n + n2 * XN2W + wave * 16 + g * 4) = rq_pack<RQ>(q[0], q[1], q[2], q[3], L2);
        }
    };

    // One barrier a tile, as in proj_expand_reduce_kernel
    if (tile < ntiles) expand(tile, 0);
    int buf = 0;
    for (int it = 0; tile < ntiles; tile += G, ++it) {
        const int nbuf = (buf + 1) % (XNB + 1);
        const bool more = tile + G < ntiles;
        if (more) {
            // since the loads of the next tile a wave has issued three stores in each of two intervals and the loads of the tile behind (two in
            // waves 0 .. 3, one in the others)
            if (it >= 2 && tile + 2 * G < ntiles) {
                if (wave < 4) wait_vmcnt<8>();
                else wait_vmcnt<7>();
            } else {
                wait_vmcnt<0>();
            }
        }
        lds_barrier();   // this tile's y is complete, the next tile's operands have landed, everybody is done with the tile before
        if (tile + 3 * G < ntiles) issue_tile(tile + 3 * G, (buf + 3) % (XNB + 1));
        asm volatile("" ::: "memory");   // the stores that the wait counts come behind these loads
        if (wave >= 8) {
            if (more) expand(tile + G, nbuf);
            __builtin_amdgcn_s_setprio(0);
            reduce(tile, buf);
        } else {
            __builtin_amdgcn_s_setprio(3);
            reduce(tile, buf);
            if (more) expand(tile + G, nbuf);
        }
        buf = nbuf;
    }
}

// ---- the 14x14 stage: 256 middle and 1024 block channels ----
// Sixteen waves: wave w owns channels 64 w .. 64 w + 63 of the expanding convolution (K = 256: 64 registers of fragments, kept
// for the whole launch) and channels 16 w .. 16 w + 15 of the reducing one, whose 256 KB of weights no longer fit next to
// them: its fragments are read from L2 for each tile, AW K steps ahead of their MFMAs (contiguous 1 KB wave-loads).
// Tiles of 64 pixels, the most that LDS holds with the next tile of x on its way: half the bytes of weights a pixel and half the barriers.
// Two tiles of x take turns; t2 has one buffer, refilled behind the expanding convolution.
// Bounds (a tile's cycles, of about 21 000): requantisations and add 8000 and the expanding MFMAs 4100 in one phase of 11 000, the reducing
// MFMAs 4100 and the LDS reads for them 4400 in one of 8000, 1300 for the stores; memory 65 us a launch of 668 copies at the rate
// of a large copy.  668 copies: 119 -> 100 us (115 -> 99, another card), 32-pixel tiles with the same order of reads 114.  The y tile is stored in whole rows from LDS
// (in pieces of 32 bytes from the registers: 113 -> 134), the loads of x are spread over the expanding phase (all at its start: each
// wave is held up to 8000 cycles at its four).
// No faster: the two phases of neighbouring tiles side by side in two groups of waves (32 pixels a tile, four buffers; 125).

constexpr int DK1 = 256, DC = 1024, DN2 = 256;

// PX: pixels of a tile
template <int RQ, int RQA, int PX>
__global__ __launch_bounds__(XNT2, 4) void expand_reduce1024_kernel(const XrParams p) {
    constexpr int NF = PX / 32, NB = PX / 16;              // fragments of 32 (expand) and 16 pixels (reduce)
    constexpr int ROWS = PX / 16;                          // rows of the x / y tile that a wave loads and stores
    constexpr bool CHANNEL_SHIFT = RQ != RQ_PAIR;          // the pair form has one shift for a layer
    constexpr int NPRM = CHANNEL_SHIFT ? 3 : 2;
    __shared__ __attribute__((aligned(256))) int8_t XY[2][PX * DC];   // rows of 1024 bytes, chunk c of pixel p at chunk c ^ (p & 15)
    __shared__ __attribute__((aligned(256))) int8_t T2[PX * DK1];     // rows of 256 bytes, the same
    __shared__ __attribute__((aligned(16))) int prm1[NPRM][DC];       // bias, M0, shift-1 in the form's way, of the expanding convolution
    __shared__ __attribute__((aligned(16))) int prm2[NPRM][DN2];      // of the reducing convolution

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ntiles = (p.npix + PX - 1) / PX, G = gridDim.x;
    const AddConst ac = add_const<RQA>(p);
    const uint32_t xy_lds = lds_address(&XY[0][0]), t2_lds = lds_address(&T2[0]);

    // direct-to-LDS loads of a tile: a wave fetches ROWS pixels of x (one 1024-byte row per load) and, a wave for each four pixels, of t2.
    // Pixels past the end re-read the last one; their results are never stored.
    auto issue_x = [&](int tile, int buf, int j) {
        int l = lane;
        asm volatile("" : "+v"(l));   // recompute the per-lane offsets per call: kept across the tile loop they would be spilled
        const int px = ROWS * wave + j, c = l ^ (px & 15);
        int n = tile * PX + px;
        n = n < p.npix ? n : p.npix - 1;
        ISR_GLOBAL_TO_LDS16_AT(p.x + ((uint32_t)n * (uint32_t)DC + (uint32_t)(c * 16)), xy_lds + buf * (PX * DC) + px * 1024);
    };
    auto issue_t2 = [&](int tile) {
        if (wave >= PX / 4) return;
        int l = lane;
        asm volatile("" : "+v"(l));
        const int px = 4 * wave + (l >> 4), c = (l & 15) ^ (px & 15);
        int n = tile * PX + px;
        n = n < p.npix ? n : p.npix - 1;
        ISR_GLOBAL_TO_LDS16_AT(p.t2 + ((uint32_t)n * (uint32_t)DK1 + (uint32_t)(c * 16)), t2_lds + wave * 1024);
    };

    int tile = blockIdx.x;
    if (tile < ntiles) {
#pragma unroll
        for (int j = 0; j < ROWS; ++j) issue_x(tile, 0, j);
        issue_t2(tile);
    }
    // constants and weights, all on their way before any is waited for
    const int i1 = tid < DC ? tid : 0, i2 = tid < DN2 ? tid : 0;
    const int b1 = p.bias1[i1], m1 = p.m0s1[i1], s1 = p.shm11[i1], b2 = p.bias2[i2], m2 = p.m0s2[i2], s2 = p.shm12[i2];
    const int chi1 = p.chi1[0], sh1 = p.shm11[0], chi2 = p.chi2[0], sh2 = p.shm12[0];
    const uint32_t lane16 = (uint32_t)lane * 16;
    // expand fragments [fm][ksub], kept in registers for the whole launch
    const int8_t *a1w = p.a1 + (size_t)wave * (2 * (DK1 / 32) * 1024);
    v4i a1[2 * (DK1 / 32)];
#pragma unroll
    for (int f = 0; f < 2 * (DK1 / 32); ++f) a1[f] = *(const v4i *)(a1w + (lane16 + (uint32_t)(f * 1024)));
    const int8_t *a2w = p.a2 + (size_t)wave * ((DC / 64) * 1024);   // this wave's reduce fragments [kstep]
    // the fragments are in their registers before the tile loop starts (else the compiler carries "load pending" into the
    // loop and waits for every outstanding memory operation at their first use in each tile)
#pragma unroll
    for (int f = 0; f < 2 * (DK1 / 32); ++f) asm volatile("" : "+v"(a1[f]));
    if (tid < DC) {
        prm1[0][i1] = b1; prm1[1][i1] = m1;
        if constexpr (CHANNEL_SHIFT) prm1[NPRM - 1][i1] = rq_sh<RQ>(s1);
    }
    if (tid < DN2) {
        prm2[0][i2] = b2; prm2[1][i2] = m2;
        if constexpr (CHANNEL_SHIFT) prm2[NPRM - 1][i2] = rq_sh<RQ>(s2);
    }
    wait_vmcnt<0>();
    __syncthreads();   // the constants are in LDS, the first tile has landed
    const RqLayer L1 = rq_layer<RQ>(rq_chi<RQ>(chi1, sh1), rq_sh<RQ>(sh1)), L2 = rq_layer<RQ>(rq_chi<RQ>(chi2, sh2), rq_sh<RQ>(sh2));
    // A channel's addend (2 z_out + 1) 2^(shift-2) from its shift, where it is not the same for the layer
    const int z1 = rq_is_top(RQ) ? rq_chi<RQ>(chi1, sh1) : chi1 >> (sh1 - 1), z2 = rq_is_top(RQ) ? rq_chi<RQ>(chi2, sh2) : chi2 >> (sh2 - 1);
    auto addend = [](int z, int s) { return rq_is_top(RQ) ? z : z << (s - 1); };

    // AW weight and FR pixel fragments of the reduce are on their way or in use (more of either is spilled)
    constexpr int AW = CHANNEL_SHIFT ? 3 : 4, FR = CHANNEL_SHIFT ? 3 : 4;
    int buf = 0;
    for (int it = 0; tile < ntiles; tile += G, ++it, buf ^= 1) {
        const int n0 = tile * PX;
        const bool more = tile + G < ntiles;
        if (it > 0) {
            // Vector memory operations complete in issue order: the loads of x stand in front of fragments that have been waited for, the
            // load of t2 in front of the ROWS + NB stores that ended the previous tile (a tile with another behind it is whole).
            wait_vmcnt<ROWS + NB>();
            lds_barrier();   // every wave's loads of this tile have landed; every wave is done with the previous tile
        }
        int8_t *xyb = XY[buf];

        // ---- expand + add into the tile of x: 64 channels x 32 pixels at a time, pixel fragments read two K sub-steps ahead ----
#pragma unroll 1
        for (int nf = 0; nf < NF; ++nf) {
            int l = lane;
            asm volatile("" : "+v"(l));   // per-lane values are recomputed, loads from them are not hoisted out of the loop
            const int half = l >> 5, px1 = nf * 32 + (l & 31);
            if (nf == 0) __builtin_amdgcn_s_setprio(3); else __builtin_amdgcn_s_setprio(1);
            if (more) issue_x(tile + G, buf ^ 1, 2 * nf);
            v16i acc[2];
#pragma unroll
            for (int fm = 0; fm < 2; ++fm)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[fm][i] = prm1[0][wave * 64 + fm * 32 + half * 16 + i];
            const int b_off1 = px1 * DK1 + ((half ^ (px1 & 15)) << 4);   // chunk (2 k + half) ^ (px & 15): sub-step k flips bits 5..7 by k
            auto operand = [&](int ks) { return *(const v4i *)(T2 + (b_off1 ^ (ks << 5))); };
            v4i fb[3] = {operand(0), operand(1)};
#pragma unroll
            for (int ks = 0; ks < DK1 / 32; ++ks) {
                if (ks + 2 < DK1 / 32) fb[(ks + 2) % 3] = operand(ks + 2);
#pragma unroll
                for (int fm = 0; fm < 2; ++fm) acc[fm] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a1[fm * (DK1 / 32) + ks], fb[ks % 3], acc[fm], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int fm = 0; fm < 2; ++fm) {
                if (nf == 0) __builtin_amdgcn_s_setprio(2); else if (fm == 0) __builtin_amdgcn_s_setprio(1); else __builtin_amdgcn_s_setprio(0);
                const int oc = wave * 64 + fm * 32 + half * 16;
                int8_t *cell = xyb + px1 * DC + (((oc >> 4) ^ (px1 & 15)) << 4);
                const v4i rv = *(const v4i *)cell;
                v4i yv;
#pragma unroll
                for (int gi = 0; gi < 4; ++gi) {
                    __builtin_amdgcn_sched_barrier(0);   // one group's constants at a time: the registers are needed for weight fragments
                    const v4i mm = *(const v4i *)&prm1[1][oc + 4 * gi], ss = *(const v4i *)&prm1[NPRM - 1][oc + 4 * gi];
                    int q[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) q[i] = rq_conv<RQ>(acc[fm][4 * gi + i], mm[i], addend(z1, ss[i]), ss[i], p.lo1, L1);
                    yv[gi] = (int)rq_add4<RQ, RQA>(q[0], q[1], q[2], q[3], (uint32_t)rv[gi], ac, L1);
                }
                *(v4i *)cell = yv;
                if (fm == 0 && more) issue_x(tile + G, buf ^ 1, 2 * nf + 1);
            }
        }
        // ---- reduce: 16 channels of the PX pixels, K = 1024; pixel fragments read FR - 1 ahead ----
        int l = lane;
        asm volatile("" : "+v"(l));
        v4i a2c[AW];
#pragma unroll
        for (int i = 0; i < AW; ++i) {   // in the order of their use
            __builtin_amdgcn_sched_barrier(0);
            a2c[i] = *(const v4i *)(a2w + ((uint32_t)l * 16 + (uint32_t)(i * 1024)));
        }
        lds_barrier();   // the y tile is complete, everybody is done with t2
        // Here and not behind the last weight fragment, whose wait this load then lengthens: from there it lands too late for the next tile (668 copies,
        // pair form: 99 -> 106 us; the other forms the same within 2 %).
        if (more) issue_t2(tile + G);
        v4acc acc2[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc2[nb][i] = prm2[0][wave * 16 + (l >> 4) * 4 + i];
        {
            const int g = l >> 4, px2 = l & 15;
            const int y_off = px2 * DC + ((g ^ px2) << 4);   // chunk (4 k + g) ^ px2: step k flips bits 6..9 by k
            auto operand = [&](int i) { return *(const v4i *)(xyb + (y_off ^ (i / NB << 6)) + i % NB * (16 * DC)); };
            constexpr int KS = DC / 64;
            v4i fb[FR];
#pragma unroll
            for (int i = 0; i < FR - 1; ++i) fb[i] = operand(i);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                if (ks == 0) __builtin_amdgcn_s_setprio(3);
                if (ks == 5) __builtin_amdgcn_s_setprio(2);
                if (ks == 10) __builtin_amdgcn_s_setprio(1);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    const int i = ks * NB + nb;
                    if (i + FR - 1 < KS * NB) fb[(i + FR - 1) % FR] = operand(i + FR - 1);
                    acc2[nb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a2c[ks % AW], fb[i % FR], acc2[nb], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (ks + AW < KS) a2c[ks % AW] = *(const v4i *)(a2w + ((uint32_t)l * 16 + (uint32_t)((ks + AW) * 1024)));
            }
        }
        l = lane;
        asm volatile("" : "+v"(l)::"memory");
        const int g = l >> 4, px2 = l & 15;
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {   // y in whole rows
            if (j == 0) __builtin_amdgcn_s_setprio(0);
            const int px = ROWS * wave + j;
            const long n1 = (long)n0 + px;
            if (n1 < p.npix) *(v4i *)(p.y + n1 * DC + (uint32_t)l * 16) = *(const v4i *)(xyb + px * DC + ((l ^ (px & 15)) << 4));
        }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const long n2 = (long)n0 + px2 + 16 * nb;
            int q[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int c = wave * 16 + g * 4 + i, ss = prm2[NPRM - 1][c];
                q[i] = rq_conv<RQ>(acc2[nb][i], prm2[1][c], addend(z2, ss), ss, p.lo2, L2);
            }
            if (n2 < p.npix) *(uint32_t *)(p.t1n + n2 * DN2 + wave * 16 + g * 4) = rq_pack<RQ>(q[0], q[1], q[2], q[3], L2);
        }
    }
}

}  // namespace

// Which of the two convolutions of a fuse_add == 2 descriptor is the projection: the main one (256 input channels, may be
// strided; the expanding convolution is then the second, w2) or the second one.
static bool projection_is_main(const ConvParams &e) { return e.fuse_add == 2 && e.Cin_p == XPK; }

// expand: 1x1, 128 -> 512 channels, with a fused residual add (the residual a stored tensor, or the 1x1 projection of a
// 256-channel tensor computed alongside); reduce: 1x1 stride 1, 512 -> 128, reading the sum; single-multiply tie-free
// requantisations (the add may meet ties); fragment-major weight copies present
bool expand_reduce_supported(const ConvParams &e, const ConvParams &r) {
    if (e.fuse_add == 1 && e.Cin_p == DK1)   // the 14 x 14 stage: 256 -> 1024 + add, then 1024 -> 256
        return e.k == 1 && e.stride == 1 && e.pad == 0 && e.Kp == DK1 && e.Cout_p == DC && e.fast_requant && e.tie_free && !e.c4 && e.wfrag &&
               r.k == 1 && r.stride == 1 && r.pad == 0 && r.Cin_p == DC && r.Kp == DC && r.Cout_p == DN2 && !r.fuse_add && r.fast_requant &&
               r.tie_free && !r.c4 && r.wfrag && e.Ho == r.H && e.Wo == r.W && r.Ho == r.H && r.Wo == r.W;
    bool expand = e.k == 1 && e.pad == 0 && e.Cout_p == XC && e.fast_requant && e.tie_free && !e.c4 && e.wfrag;
    if (e.fuse_add == 1) expand = expand && e.stride == 1 && e.Cin_p == XK1 && e.Kp == XK1;
    else if (projection_is_main(e))   // main: projection 256 -> 512, stride 1 or 2; second: the expanding convolution on the output pixels
        expand = expand && (e.stride == 1 || e.stride == 2) && e.Kp == XPK && e.Cin2_p == XK1 && e.tie_free2 && e.wfrag2 &&
                 (long)e.H * e.W * XPK < (1l << 31);
    else
        expand = expand && e.fuse_add == 2 && e.stride == 1 && e.Cin_p == XK1 && e.Kp == XK1 && e.Cin2_p == XPK && e.tie_free2 && e.wfrag2;
    const bool reduce = r.k == 1 && r.stride == 1 && r.pad == 0 && r.Cin_p == XC && r.Kp == XC &&
                        (r.Cout_p == XN2 || (r.Cout_p == XN2W && e.fuse_add == 1)) && !r.fuse_add && r.fast_requant && r.tie_free &&
                        !r.c4 && r.wfrag;
    return expand && reduce && e.Ho == r.H && e.Wo == r.W && r.Ho == r.H && r.Wo == r.W;
}

// The kernel's arguments from the descriptors of the expanding (+ add) and the reducing convolution and their tensors:
// `a` is the main convolution's input, `b` the add's other operand (fuse_add == 1) or the second convolution's input.
void expand_reduce_params(const ConvParams &e, const ConvParams &r, const int8_t *a, const int8_t *b, int8_t *y, int8_t *t1n,
                          int32_t copies, XrParams &xp) {
    xp = XrParams{};
    xp.y = y; xp.t1n = t1n;
    xp.a2 = r.wfrag; xp.bias2 = r.bias; xp.m0s2 = r.m0s; xp.chi2 = r.chi; xp.shm12 = r.shm1;
    xp.lo2 = r.relu ? r.zp_out : -128;
    xp.rq = e.rq & r.rq & (e.fuse_add == 2 ? e.rq2 : ~0);
    xp.add_rq = e.add_rq;
    xp.add_c0 = e.add_c0; xp.add_k = e.add_k; xp.add_sh = e.add_sh; xp.add_lo = e.add_lo;
    xp.npix = copies * e.Ho * e.Wo;
    xp.n2 = r.Cout_p;
    xp.k1 = e.fuse_add == 1 ? e.Cin_p : XK1;
    xp.Hin = e.H; xp.Win = e.W; xp.Ho = e.Ho; xp.Wo = e.Wo; xp.pstride = 1;
    const int lo_main = e.relu ? e.zp_out : -128;
    if (projection_is_main(e)) {
        xp.in2 = a; xp.pstride = e.stride;
        xp.ap = e.wfrag; xp.biasp = e.bias; xp.m0sp = e.m0s; xp.chip = e.chi; xp.shm1p = e.shm1; xp.lop = lo_main;
        xp.t2 = b;
        xp.a1 = e.wfrag2; xp.bias1 = e.bias2; xp.m0s1 = e.m0s2; xp.chi1 = e.chi2; xp.shm11 = e.shm12; xp.lo1 = e.lo2;
        xp.add_mul_self = e.add_mul_res; xp.add_mul_res = e.add_mul_self;   // "self" in the kernel = the expanding convolution
    } else {
        xp.t2 = a;
        xp.a1 = e.wfrag; xp.bias1 = e.bias; xp.m0s1 = e.m0s; xp.chi1 = e.chi; xp.shm11 = e.shm1; xp.lo1 = lo_main;
        xp.add_mul_self = e.add_mul_self; xp.add_mul_res = e.add_mul_res;
        if (e.fuse_add == 2) {
            xp.in2 = b;
            xp.ap = e.wfrag2; xp.biasp = e.bias2; xp.m0sp = e.m0s2; xp.chip = e.chi2; xp.shm1p = e.shm12; xp.lop = e.lo2;
        } else {
            xp.x = b;
        }
    }
}

// The kernels serve tie-free convolutions only: where with_rq takes the general form for an add with exact halves, they take
// their own next to it.
template <class F>
static void with_tie_free_rq(const XrParams &p, F f) {
    using std::integral_constant;
    if ((p.rq & ~RQ_PAIR) == RQ_TIE_FREE && p.add_rq == RQ_ANY) f(integral_constant<int, RQ_TIE_FREE>{}, integral_constant<int, RQ_ANY>{});
    else with_rq(p.rq, p.add_rq, [&](auto rq, auto rqa) { if constexpr ((decltype(rq)::value & (RQ_TIE_FREE | RQ_PAIR)) != 0) f(rq, rqa); });
}

hipError_t launch_expand_reduce(const XrParams &p, hipStream_t st) {
    if (p.npix <= 0) return hipSuccess;
    if (!(p.rq & RQ_TIE_FREE)) return hipErrorInvalidValue;
    if ((long)p.npix * DC >= (1l << 32)) return hipErrorInvalidValue;   // 32-bit byte offsets inside the tensors
    const int ntiles = (p.npix + XPX - 1) / XPX;
    if (p.k1 == DK1) {
        // us of a launch with r rounds of 256 tiles: 8.5 + 10.7 r with 64 pixels, 7 + 6.7 r with 32 (copies of 14 x 14 pixels 60 / 84 / 100 / 150 /
        // 250 / 668: 17.4 / 27.4 / 29.0 / 30.8 / 42.5 / 100 and 19.0 / 25.5 / 26.2 / 32.8 / 46.2 / 114)
        const int wide = (p.npix + 63) / 64, rounds = (ntiles + 255) / 256, wide_rounds = (wide + 255) / 256;
        const bool narrow = 15 + 107 * wide_rounds > 67 * rounds;
        const int tiles = narrow ? ntiles : wide;
        const dim3 grid((unsigned)(tiles < 256 ? tiles : 256));
        set_kernel_name(narrow ? "expand_reduce_kernel<256, 1024, 256, 32 pixels>" : "expand_reduce_kernel<256, 1024, 256, 64 pixels>");
        with_tie_free_rq(p, [&](auto rq, auto rqa) {
            if (narrow) hipLaunchKernelGGL((expand_reduce1024_kernel<decltype(rq)::value, decltype(rqa)::value, 32>), grid, dim3(XNT2), 0, st, p);
            else hipLaunchKernelGGL((expand_reduce1024_kernel<decltype(rq)::value, decltype(rqa)::value, 64>), grid, dim3(XNT2), 0, st, p);
        });
        return hipGetLastError();
    }
    if (p.in2) {
        const dim3 grid((unsigned)(ntiles < 256 ? ntiles : 256));   // one workgroup of sixteen waves per CU
        set_kernel_name("proj_expand_reduce_kernel<256, 128, 512, 128>");
        with_tie_free_rq(p, [&](auto rq, auto rqa) { hipLaunchKernelGGL((proj_expand_reduce_kernel<decltype(rq)::value, decltype(rqa)::value>), grid, dim3(XNT2), 0, st, p); });
        return hipGetLastError();
    }
    if (p.n2 == XN2W) {
        const dim3 grid((unsigned)(ntiles < 256 ? ntiles : 256));
        set_kernel_name("expand_reduce_kernel<128, 512, 256>");
        with_tie_free_rq(p, [&](auto rq, auto rqa) { hipLaunchKernelGGL((expand_reduce256_kernel<decltype(rq)::value, decltype(rqa)::value>), grid, dim3(XNT2), 0, st, p); });
        return hipGetLastError();
    }
    const dim3 grid((unsigned)(ntiles < 512 ? ntiles : 512));
    set_kernel_name("expand_reduce_kernel<128, 512, 128>");
    with_tie_free_rq(p, [&](auto rq, auto rqa) { hipLaunchKernelGGL((expand_reduce_kernel<decltype(rq)::value, decltype(rqa)::value>), grid, dim3(XNT), 0, st, p); });
    return hipGetLastError();
}

}  // namespace isr
