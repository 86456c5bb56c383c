// Bottleneck residual block with 64 middle channels, resident workgroups (launches of many tiles; bottleneck.hip has the others):
//   t1 = clamp(requant(conv1x1(x)))                     256 -> 64 (identity block) or 64 -> 64 (first block of a stage)
//   t2 = clamp(requant(conv3x3(t1)))                    64 -> 64, stride 1, pad 1
//   y  = add_requant(clamp(requant(conv1x1(t2))), r)    64 -> 256; r = x, or clamp(requant(conv1x1_p(x))) in a first block
// A workgroup of sixteen waves fills a CU and walks over tiles of 8 x 28 output pixels (300 halo pixels).  The 3x3 weights and all constants
// stay in LDS, the 1x1 weights in registers, for the whole launch.  Two barriers a tile:
//   interval 1: t2 of the tile before goes from registers to LDS; first convolution of this tile's halo (wave = 16 channels x 5 groups of
//               16 pixels), its result as the t1 tile to LDS, zero-points outside the image; an identity block's residual, the x of
//               the wave's own channels and pixels, from LDS to registers
//   interval 2: the next tile's x on its way into LDS (nobody reads this one's any more); 3x3 convolution of this tile (wave = 32 channels x
//               32 pixels) into registers, and closing convolution + add + store of the tile BEFORE (wave = 32 channels x seven groups of 16
//               pixels).  One half of each SIMD's waves do it in this order, the other half in the other, so that matrix unit and LDS work
//               of the one stands beside the requantisation arithmetic of the other.
//
// What bounds it (pair form, 668 copies at 56 x 56, counters): a tile of an identity block takes 17 000 cycles a SIMD, for 9600 of which vector
// instructions issue and for 4128 of which the matrix unit works; one of a first block 16 400, 10 600 and 4112.  The two overlap only partly.
// With loads from the cache and no stores a first block takes 280 instead of 283 us, an identity block 254 instead of 286.
// Two workgroups a CU that start, load their weights and end with each tile (bottleneck.hip) take 319 and 329 us where this kernel takes 278 and 288;
// launch_bottleneck has the times of other launches and forms.  Of that: the waves' priority by what they still have to do 3 % (first blocks 5 to
// 10 % in the forms with more constants), the closing convolution in fragments of 16 rows, whose constants are read once a tile instead of once a
// fragment, 5 %, the pixels' places found by five waves for all 4 %.
#include "conv_device.h"

namespace isr {

namespace {

typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

constexpr int TH = 8, TW = 28;                       // output tile
constexpr int HW = TW + 2, NHALO = (TH + 2) * HW;    // halo tile: 10 x 30 = 300 pixels
constexpr int NPX = TH * TW, NP_FR = TW / 4;         // 224 output pixels; fragment f: columns 4 f .. 4 f + 3 of all rows; groups of 16: its upper or lower four rows
constexpr int NGROUPS = (NHALO + 15) / 16;           // groups of 16 halo pixels: 19
constexpr int NROWS = NGROUPS * 16;
constexpr int NT = 1024;
constexpr uint32_t OUTSIDE = 1u << 23;                // tensors are below 2 GiB: at 256 bytes a pixel an index is smaller
constexpr int TPAD = 144, TROW = HW * 64 + TPAD;      // a row of t1: its 4 x 4 pixels lie in different banks without a swizzle, so that taps are immediate offsets
constexpr int W2_CHUNKS = 37;                        // 16-byte chunks per 3x3 weight row: 36 + 1 pad (bank spread)

template <bool PROJ, int RQ, int RQA>
__global__ __launch_bounds__(NT, 4) void bottleneck_stream_kernel(const BneckParams p, const int ntiles) {
    constexpr int CIN = PROJ ? 64 : 256, COUT = 256, KS1 = CIN / 64, XB = NROWS * CIN;
    constexpr int NXB = PROJ ? 3 : 1;   // the projection reads the x of the tile before, next to this one's and the next one's
    // Per-lane positions are computed again for each tile where registers are short: kept, they go to scratch, and a reload waits for the stores and
    // loads in flight.  us of a launch, first block: RQ_ANY 9352 / 5600 tiles 457 / 266 -> 448 / 256, RQ_TIE_FREE 388 / 226 -> 385 / 223, RQ_TOP
    // 2800 tiles 95.9 -> 94.5, at 9352 the same; identity block, RQ_TIE_FREE 345 / 206 -> 338 / 199.  The identity blocks of the forms with exact
    // halves keep 12 to 20 bytes a lane there, which cost nothing that could be measured (RQ_ANY 1 % slower with the places computed again).
    constexpr bool RECOMPUTE = !PROJ || RQ != RQ_PAIR, RECOMPUTE_FIND = PROJ ? RQ != RQ_PAIR : RQ == RQ_TIE_FREE;
    __shared__ __attribute__((aligned(256))) int8_t X[NXB][XB];
    __shared__ __attribute__((aligned(16))) int8_t T1[(TH + 2) * TROW];      // [halo row][column][64 channels]
    __shared__ __attribute__((aligned(16))) int8_t T2[NPX * 64];             // [row half][fragment][pixel of the group][64 channels], 16-byte chunks swizzled
    __shared__ __attribute__((aligned(16))) int8_t W2[64 * W2_CHUNKS * 16];
    __shared__ __attribute__((aligned(16))) int prm[2][4][64];               // bias, M0, chi, shift-1 of the first two convolutions
    __shared__ __attribute__((aligned(16))) int prm3[4][COUT];               // of the closing one
    __shared__ __attribute__((aligned(16))) int prmp[PROJ ? 4 : 1][PROJ ? COUT : 4];   // and of the projection
    __shared__ uint32_t at[3][NROWS];   // tile it in at[it % 3], each halo pixel: index (image, row, column) or OUTSIDE | row of the tile << 24

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // roles: first convolution 16 channels (cg) x 5 of the 19 pixel groups; 3x3 convolution 32 channels x one fragment (waves 0 .. 13);
    // closing convolution 32 channels (cb) x the upper or lower four rows (par), seven groups
    const int cg = wave & 3, pq = wave >> 2;
    const int cb = (wave & 3) | (wave >> 3) << 2, par = (wave >> 2) & 1;
    const bool conv_first = par == 0;
    const int G = gridDim.x, npix = p.B * p.H * p.W;
    // Outside pixels have an index whose bytes lie behind the end of either tensor: loads give 0 (the first convolution's result is replaced
    // there), stores do nothing.
    const auto in_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t *>(p.in), 0, npix * CIN, 0x00027000);
    const auto out_rsrc = __builtin_amdgcn_make_buffer_rsrc(p.out, 0, npix * COUT, 0x00027000);
    // consecutive tiles, which share halo rows, run on the same XCD (workgroup ids are dealt round-robin over 8 XCDs)
    const int tiles_x = (p.W + TW - 1) / TW, per_image = tiles_x * ((p.H + TH - 1) / TH);
    auto find = [&](int id, int buf, int r) {   // halo pixel r of a tile
        const int xcd = id & 7, per = ntiles >> 3, extra = ntiles & 7;
        const int logical = xcd * per + (xcd < extra ? xcd : extra) + (id >> 3);
        const int b = logical / per_image, t = logical % per_image;
        const int hy = r / HW, y = (t / tiles_x) * TH - 1 + hy, x = (t % tiles_x) * TW - 1 + r - hy * HW;
        if (r < NROWS) at[buf][r] = r < NHALO && (unsigned)y < (unsigned)p.H && (unsigned)x < (unsigned)p.W ? (uint32_t)((b * p.H + y) * p.W + x) | (uint32_t)hy << 24 : OUTSIDE | (uint32_t)hy << 24;
    };
    const uint32_t x_lds = lds_address(&X[0][0]);
    // x of a tile's halo, straight into LDS: row r holds K chunk c at c ^ (r & 15) (256 channels) or c ^ swz(r) (64)
    auto issue = [&](int abuf, int buf) {
        constexpr int CH = CIN / 16, RPP = 512 / CH, PASSES = (NROWS + RPP - 1) / RPP;   // chunks a row, rows a pass
        int i = cb * 64 + lane;
        if constexpr (RECOMPUTE) asm volatile("" : "+v"(i));
        const int r0 = i / CH, c = (i % CH) ^ (PROJ ? swz<4>(r0) : r0 & 15);
#pragma unroll
        for (int j = 0; j < PASSES; ++j)
            if ((j + 1) * RPP <= NROWS || cb < (NROWS - j * RPP) * CH / 64)   // wave-uniform
                __builtin_amdgcn_raw_ptr_buffer_load_lds(in_rsrc, (__attribute__((address_space(3))) void *)(uintptr_t)(x_lds + buf * XB + j * 8192 + cb * 1024), 16,
                                                         __umul24(at[abuf][j * RPP + r0], CIN) + c * 16, 0, 0, 0);
    };
    static_assert(NROWS * (256 / 16) % 64 == 0 && NROWS * (64 / 16) % 64 == 0, "whole loads of a wave");

    // ---- once a launch: 3x3 weights, constants, 1x1 weights ----
    int id = blockIdx.x;
    find(id, 0, tid);
    {
        constexpr int TOTAL = 64 * W2_CHUNKS;   // 2368 = 2 * 1024 + 5 * 64
        const uint32_t w2_lds = lds_address(W2);
#pragma unroll
        for (int pass = 0; pass < (TOTAL + NT - 1) / NT; ++pass)
            if (pass * NT + wave * 64 < TOTAL) {   // wave-uniform
                const int q = pass * NT + tid, r = q / W2_CHUNKS, c = q % W2_CHUNKS;
                ISR_GLOBAL_TO_LDS16_AT(p.w2 + r * 576 + (c < 36 ? c : 0) * 16, w2_lds + (pass * NT + wave * 64) * 16);
            }
    }
    v4i w1f[KS1], f3[2], fp[2];
    {
        // the rows of w1 are in the order of a 32-row fragment, whose lane holds 16 consecutive channels: channel c of 32 is row
        // 8 ((c >> 2) & 3) + 4 (c >> 4) + (c & 3)
        const int c = (cg & 1) * 16 + (lane & 15), r = (cg >> 1) * 32 + 8 * ((c >> 2) & 3) + 4 * (c >> 4) + (c & 3);
#pragma unroll
        for (int ks = 0; ks < KS1; ++ks) w1f[ks] = *(const v4i *)(p.w1 + r * CIN + ks * 64 + (lane >> 4) * 16);
        // closing convolution and projection: two fragments of 16 rows, such that a lane gets eight consecutive channels of its pixel
        const int m = lane & 15;
#pragma unroll
        for (int fr = 0; fr < 2; ++fr) {
            const int c3 = 8 * (m >> 2) + 4 * fr + (m & 3), r3 = cb * 32 + 8 * ((c3 >> 2) & 3) + 4 * (c3 >> 4) + (c3 & 3);
            f3[fr] = *(const v4i *)(p.w3 + r3 * 64 + (lane >> 4) * 16);
            if constexpr (PROJ) fp[fr] = *(const v4i *)(p.wp + r3 * 64 + (lane >> 4) * 16);
        }
        const int cv = (tid >> 6) & 1, c12 = tid & 63, ct = tid & (COUT - 1);
        const RqRaw r12 = cv ? rq_fetch(p.bias2, p.m0s2, p.chi2, p.shm12, c12) : rq_fetch(p.bias1, p.m0s1, p.chi1, p.shm11, c12);
        const RqRaw rc = rq_fetch(p.bias3, p.m0s3, p.chi3, p.shm13, ct);
        RqRaw rp{};
        if constexpr (PROJ) rp = rq_fetch(p.biasp, p.m0sp, p.chip, p.shm1p, ct);
        if (tid < 128) rq_store<RQ>(prm[cv], r12, c12);
        if (tid < COUT) {
            rq_store<RQ>(prm3, rc, ct);
            if constexpr (PROJ) rq_store<RQ>(prmp, rp, ct);
        }
    }
    __syncthreads();
    if (conv_first) issue(0, 0);
    wait_vmcnt<0>();
    // pinned: loads that count as pending in the loop would make their uses wait for its loads and stores
#pragma unroll
    for (int ks = 0; ks < KS1; ++ks) asm volatile("" : "+v"(w1f[ks]));
#pragma unroll
    for (int fr = 0; fr < 2; ++fr) {
        asm volatile("" : "+v"(f3[fr]));
        if constexpr (PROJ) asm volatile("" : "+v"(fp[fr]));
    }
    const AddConst ac = add_const<RQA>(p);
    const RqLayer L1 = rq_layer<RQ>(prm[0][2][0], prm[0][3][0]), L2 = rq_layer<RQ>(prm[1][2][0], prm[1][3][0]), L3 = rq_layer<RQ>(prm3[2][0], prm3[3][0]);
    const RqLayer Lp = PROJ ? rq_layer<RQ>(prmp[PROJ ? 2 : 0][0], prmp[PROJ ? 3 : 0][0]) : RqLayer{0, 0};

    // sixteen channels of a 32-pixel fragment, from the constants at c on
    auto requant16 = [&](const v16i &a, const auto &k, int c, int lo, const RqLayer &L, auto use) {
#pragma unroll
        for (int gi = 0; gi < 4; ++gi) {
            __builtin_amdgcn_sched_barrier(0);
            const v4i mm = *(const v4i *)&k[1][c + 4 * gi], ch = rq_chi4<RQ>(&k[2][c + 4 * gi]), ss = *(const v4i *)&k[3][c + 4 * gi];
            int q[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) q[i] = rq_conv<RQ>(a[4 * gi + i], mm[i], ch[i], ss[i], lo, L);
            use(gi, q);
        }
    };
    auto bias16 = [&](v16i &a, const auto &k, int c) {
#pragma unroll
        for (int i = 0; i < 16; ++i) a[i] = k[0][c + i];
    };
    const int half = lane >> 5, l32 = lane & 31, g = lane >> 4, n = lane & 15;
    const int wm = wave & 1, f2 = wave < 2 * NP_FR ? wave >> 1 : 0;
    // closing convolution: the lane's eight channels, the halo position of its pixel in the first group (4 f further in group f)
    const int c0 = cb * 32 + 8 * g, hp0 = (4 * par + (n >> 2) + 1) * HW + (n & 3) + 1;
    const int8_t *const t2_group = T2 + par * NP_FR * 1024 + n * 64 + ((g ^ swz<4>(n)) << 4);
    v4acc bias3[2], biasp[2];
    v4i mm3[2];
#pragma unroll
    for (int fr = 0; fr < 2; ++fr) {
        bias3[fr] = *(const v4acc *)&prm3[0][c0 + 4 * fr];
        mm3[fr] = *(const v4i *)&prm3[1][c0 + 4 * fr];
        asm volatile("" : "+v"(bias3[fr]));
        if constexpr (RQ == RQ_PAIR && !PROJ) asm volatile("" : "+v"(mm3[fr]));
        if constexpr (PROJ) {
            biasp[fr] = *(const v4acc *)&prmp[0][c0 + 4 * fr];
            asm volatile("" : "+v"(biasp[fr]));
        }
    }

    typedef int v2i __attribute__((ext_vector_type(2)));
    v2i resid[PROJ ? 1 : NP_FR];
    auto first_conv = [&](int abuf, int buf) {
        int l = lane;
        if constexpr (RECOMPUTE) asm volatile("" : "+v"(l));
        const int g = l >> 4, n = l & 15, c = cg * 16 + 4 * g, h0 = pq * 80 + n;
        const v4i b4 = *(const v4i *)&prm[0][0][c];
        const int8_t *xb = X[buf] + h0 * CIN + (PROJ ? (g ^ swz<4>(n)) << 4 : 0);
        const int k0 = (g ^ n) << 4;
        v4acc acc[5];
#pragma unroll
        for (int u = 0; u < 5; ++u) acc[u] = v4acc{b4[0], b4[1], b4[2], b4[3]};
#pragma unroll
        for (int ks = 0; ks < KS1; ++ks)
#pragma unroll
            for (int u = 0; u < 5; ++u)
                if (u < 4 || pq < 3) acc[u] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w1f[ks], *(const v4i *)(xb + u * 16 * CIN + (PROJ ? 0 : k0 ^ (ks << 6))), acc[u], 0, 0, 0);
        const uint32_t zt = (uint32_t)(p.zp_t1 & 0xFF) * 0x01010101u;
        const v4i mm = *(const v4i *)&prm[0][1][c], ch = rq_chi4<RQ>(&prm[0][2][c]), ss = *(const v4i *)&prm[0][3][c];
#pragma unroll
        for (int u = 0; u < 5; ++u)
            if (u < 4 || pq < 3) {
                int q[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) q[i] = rq_conv<RQ>(acc[u][i], mm[i], ch[i], ss[i], p.lo1, L1);
                uint32_t v = rq_pack<RQ>(q[0], q[1], q[2], q[3], L1);
                const uint32_t a = at[abuf][h0 + u * 16];
                if (a & OUTSIDE) v = zt;
                if (u < 3 || h0 + u * 16 < NHALO) *(uint32_t *)(T1 + (h0 + u * 16) * 64 + c + __umul24(a >> 24, TPAD)) = v;
            }
    };
    v4i t2{0, 0, 0, 0};
    auto second_conv = [&]() {
        if (wave >= 2 * NP_FR) return;   // wave-uniform
        int l = lane;
        if constexpr (RECOMPUTE) asm volatile("" : "+v"(l));
        const int half = l >> 5, l32 = l & 31, c16 = wm * 32 + 16 * half;
        const int8_t *const t1_tap = T1 + (l32 >> 2) * TROW + (4 * f2 + (l32 & 3)) * 64 + half * 16, *const w2_row = W2 + ((wm * 32 + l32) * W2_CHUNKS + half) * 16;
        v16i acc;
        bias16(acc, prm[1], c16);
        auto weights = [&](int ks) { return *(const v4i *)(w2_row + ks * 32); };
        auto pixels = [&](int ks) { return *(const v4i *)(t1_tap + (ks >> 1) / 3 * TROW + (ks >> 1) % 3 * 64 + (ks & 1) * 32); };
        v4i fa[3] = {weights(0), weights(1)}, fb[3] = {pixels(0), pixels(1)};
#pragma unroll
        for (int ks = 0; ks < 18; ++ks) {
            if (ks + 2 < 18) {
                fa[(ks + 2) % 3] = weights(ks + 2);
                fb[(ks + 2) % 3] = pixels(ks + 2);
            }
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[ks % 3], fb[ks % 3], acc, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        requant16(acc, prm[1], c16, p.lo2, L2, [&](int gi, const int (&q)[4]) { t2[gi] = (int)rq_pack<RQ>(q[0], q[1], q[2], q[3], L2); });
    };
    auto store_t2 = [&]() {
        if (wave >= 2 * NP_FR) return;
        *(v4i *)(T2 + ((l32 >> 4) * NP_FR + f2) * 1024 + n * 64 + (((wm * 2 + half) ^ swz<4>(n)) << 4)) = t2;
    };
    // closing convolution, add, store: a store for every two groups, whichever of its pixels lie in the image (the waits count them); the products of
    // a group stand in front of the arithmetic of the one before
    auto last_conv = [&](int abuf, int buf) {
        int hp1 = hp0;
        if constexpr (PROJ) asm volatile("" : "+v"(hp1));
        auto x_at = [&](int f) {
            const int hp = hp1 + 4 * f;
            return *(const v4i *)(X[buf] + hp * CIN + ((g ^ swz<4>(hp)) << 4));
        };
        auto t_at = [&](int f) { return *(const v4i *)(t2_group + f * 1024); };
        auto consts = [&](const auto &k, const v4i (&kept)[2], int fr, v4i &mm, v4i &ch, v4i &ss) {
            const int c = c0 + 4 * fr;
            if constexpr (RQ == RQ_PAIR && !PROJ) mm = kept[fr]; else mm = *(const v4i *)&k[1][c];
            ch = rq_chi4<RQ>(&k[2][c]);
            ss = *(const v4i *)&k[3][c];
        };
        v4i tn[2] = {t_at(0), t_at(1)}, xn[2];
        if constexpr (PROJ) { xn[0] = x_at(0); xn[1] = x_at(1); }
        constexpr bool AHEAD = !PROJ;   // a projection's would take too many registers
        v4acc a[2][2], ap[2][2];
        auto products = [&](int f) {
#pragma unroll
            for (int fr = 0; fr < 2; ++fr) {
                a[f & 1][fr] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f3[fr], tn[f & 1], bias3[fr], 0, 0, 0);
                if constexpr (PROJ) ap[f & 1][fr] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fp[fr], xn[f & 1], biasp[fr], 0, 0, 0);
            }
        };
        if constexpr (AHEAD) products(0);
        v2u y0{0, 0};
#pragma unroll
        for (int f = 0; f < NP_FR; ++f) {
            // the oldest wave of a SIMD would be done thousands of cycles before the youngest: who has more left goes first
            if (f == 0) __builtin_amdgcn_s_setprio(3);
            if (f == 2) __builtin_amdgcn_s_setprio(2);
            if (f == 4) __builtin_amdgcn_s_setprio(1);
            if (f == 6) __builtin_amdgcn_s_setprio(0);
            if constexpr (!AHEAD) products(f);
            else if (f + 1 < NP_FR) products(f + 1);
            if (f + 2 < NP_FR) {
                tn[f & 1] = t_at(f + 2);
                if constexpr (PROJ) xn[f & 1] = x_at(f + 2);
            }
            const uint32_t px = f + 1 == NP_FR ? at[abuf][hp0 + 4 * f] : f & 1 ? at[abuf][hp0 + 4 * (f - 1) + 4 * (g & 1)] : 0;
            __builtin_amdgcn_sched_barrier(0);
            v2u y;
#pragma unroll
            for (int fr = 0; fr < 2; ++fr) {
                v4i mm, ch, ss;
                int q[4];
                uint32_t r;
                if constexpr (PROJ) {
                    consts(prmp, mm3, fr, mm, ch, ss);
#pragma unroll
                    for (int i = 0; i < 4; ++i) q[i] = rq_conv<RQ>(ap[f & 1][fr][i], mm[i], ch[i], ss[i], p.lop, Lp);
                    r = rq_pack<RQ>(q[0], q[1], q[2], q[3], Lp);
                } else {
                    r = (uint32_t)resid[f][fr];
                }
                consts(prm3, mm3, fr, mm, ch, ss);
#pragma unroll
                for (int i = 0; i < 4; ++i) q[i] = rq_conv<RQ>(a[f & 1][fr][i], mm[i], ch[i], ss[i], p.lo3, L3);
                y[fr] = rq_add4<RQ, RQA>(q[0], q[1], q[2], q[3], r, ac, L3);
            }
            // Two groups' results become one store of 16 bytes a lane: lanes of even g take the first group's pixel with the eight channels of
            // the lanes behind them, lanes of odd g the second group's.
            if (f + 1 == NP_FR) {
                __builtin_amdgcn_raw_buffer_store_b64(y, out_rsrc, (px << 8) + (uint32_t)c0, 0, 0);
            } else if (f & 1) {
                const v2u s0 = __builtin_amdgcn_permlane16_swap(y0[0], y[0], false, false), s1 = __builtin_amdgcn_permlane16_swap(y0[1], y[1], false, false);
                __builtin_amdgcn_raw_buffer_store_b128(v4u{s0[0], s1[0], s0[1], s1[1]}, out_rsrc, (px << 8) + (uint32_t)(cb * 32 + (g >> 1) * 16), 0, 0);
            } else {
                y0 = y;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    int buf = 0, abuf = 0;   // of this tile's x and pixels
    for (int it = 0;; ++it, id += G) {
        const bool have = id < ntiles, more = id + G < ntiles;
        // This tile's x was issued at the start of the last interval, by the waves that convolve first; since then such a wave has issued its
        // stores of the tile before, none in the first round.
        if (it < 2) wait_vmcnt<0>();
        else if (conv_first) wait_vmcnt<(NP_FR + 1) / 2>();
        lds_barrier();   // x has landed; everybody is done with t1 and with the last t2
        const int nabuf = abuf == 2 ? 0 : abuf + 1, pabuf = abuf == 0 ? 2 : abuf - 1;
        if (it > 0) store_t2();
        if (more && wave >= 11) {
            int l = lane;
            if constexpr (RECOMPUTE_FIND) asm volatile("" : "+v"(l));
            find(id + G, nabuf, RECOMPUTE_FIND ? (wave - 11) * 64 + l : tid - 11 * 64);
        }
        v2i rnew[PROJ ? 1 : NP_FR];
        if (have) {
            __builtin_amdgcn_s_setprio(0);
            first_conv(abuf, buf);
            if constexpr (!PROJ) {
                int hp1 = hp0;
                asm volatile("" : "+v"(hp1));
#pragma unroll
                for (int f = 0; f < NP_FR; ++f) {
                    const int hp = hp1 + 4 * f;
                    rnew[f] = *(const v2i *)(X[0] + hp * CIN + (((2 * cb + (g >> 1)) ^ (hp & 15)) << 4) + (g & 1) * 8);
                }
            }
        }
        lds_barrier();   // t1, t2 and the next tile's pixels are complete; everybody is done with an identity block's x
        const int nbuf = NXB == 1 || buf + 1 == NXB ? 0 : buf + 1, pbuf = NXB == 1 ? 0 : buf == 0 ? NXB - 1 : buf - 1;
        __builtin_amdgcn_s_setprio(3);
        if (more && conv_first) issue(nabuf, nbuf);
        asm volatile("" ::: "memory");   // the stores come behind the loads
        if (have && conv_first) second_conv();
        if (it > 0) last_conv(pabuf, pbuf);
        if (!have) break;
        if (!conv_first) second_conv();
        if constexpr (!PROJ)
#pragma unroll
            for (int f = 0; f < NP_FR; ++f) resid[f] = rnew[f];
        buf = nbuf;
        abuf = nabuf;
    }
}

}  // namespace

hipError_t launch_bottleneck_stream(const BneckParams &p, int ntiles, hipStream_t st) {
    const dim3 grid((unsigned)(ntiles < 256 ? ntiles : 256)), block(NT);   // one workgroup a CU
    set_kernel_name(p.proj ? "bottleneck_stream_kernel<block + projection>" : "bottleneck_stream_kernel<block>");
    with_rq(p.rq, p.add_rq, [&](auto rq, auto rqa) {
        constexpr int RQ = decltype(rq)::value, RQA = decltype(rqa)::value;
        if (p.proj) hipLaunchKernelGGL((bottleneck_stream_kernel<true, RQ, RQA>), grid, block, 0, st, p, ntiles);
        else hipLaunchKernelGGL((bottleneck_stream_kernel<false, RQ, RQA>), grid, block, 0, st, p, ntiles);
    });
    return hipGetLastError();
}

}  // namespace isr
