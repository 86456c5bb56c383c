// Bottleneck residual block with 64 middle channels in one kernel:
//   t1 = clamp(requant(conv1x1(x)))                     Cin -> 64
//   t2 = clamp(requant(conv3x3(t1)))                    64 -> 64, stride 1, pad 1
//   y  = add_requant(clamp(requant(conv1x1(t2))), x)    64 -> Cout = Cin   (TAIL only)
// A workgroup of eight waves makes 8 x 28 pixel tiles of images: 224 output pixels = seven full
// 32-pixel MFMA fragments (no padding columns in the two later convolutions, whose requantisation
// arithmetic is what bounds this kernel), 10 x 30 = 300 halo pixels = ten fragments for the first.
//   1. The first convolution runs as a GEMM over the halo pixels (wave = 32 channels x 3 or 2 fragments):
//      K steps of 64 input channels go from global memory straight into three LDS stages.
//      Recomputing the halo costs a third more of this (cheap) GEMM and saves writing and
//      re-reading t1.
//   2. Its int8 result goes into an LDS tile [halo pixel][64 channels]; halo pixels outside the
//      image get t1's zero-point, the padding value of the 3x3 convolution.
//   3. The 3x3 convolution reads its pixel operands from that tile at tap-shifted addresses
//      (no gather from memory) and its weights from LDS (fetched while step 2 runs, into
//      the space of the two operand stages): 18 K steps of 32, no barrier inside
//      (wave = 32 channels x 2 or 1 fragments).
//   4. HEAD: t2 is requantised and stored.  TAIL: t2 replaces t1 in LDS, and the last 1x1
//      convolution + residual add is split over the waves by OUTPUT CHANNEL: each wave owns 32 of
//      every 256 channels for all seven pixel fragments, so that all carry the same load; its weight fragments and
//      multipliers are loaded once, the pixel operands come from the t2 tile, and the residual --
//      x at the wave's own channels, input channels of one K step of step 1 -- was
//      copied from that step's LDS stage into registers: x is read from memory once.
// x is read once (plus halo, mostly cache hits), t1 and t2 never leave the CU.
// Blocks of 256 channels without the next stage's 1x1 run in resident workgroups in launches of many tiles (bottleneck_stream.hip; the rule is
// in launch_bottleneck).
//
// Bounds, 668 images of 56 x 56 x 256, block and next stage's 1x1, 395 to 410 us: memory 0.94 GB = 183 us at the rate of a large copy, vector
// instructions issue for 46 % of the time, the matrix unit works for 22 %, in phases that barriers separate.
// What it gained, measured with blocks of 668 images that run in resident workgroups now: two workgroups of eight waves a CU instead of two of
// four 344 -> 322 us (projection block 360 -> 340);
// all operands of step 1 on their way at once, the weights of steps 3 and 4 fetched a step early, the residual's and the
// output's places in a table (224 divisions by the tile's width instead of one per wave and fragment), t1 and t2 at 80 bytes a
// pixel (taps as immediate offsets): 1640 -> 1350 vector instructions a wave, 354 -> 327 us; projection block 382 -> 344,
// block + next 486 -> 428 (one card).
// With the next stage's 1x1 convolution (256 -> 128) in the kernel the sum is not read back and, under a stride-2
// projection, three quarters of it are not written: when added 441 us against 322 + 157 for two kernels.
#include "conv_device.h"

namespace isr {

namespace {

template <int N>
using Frag = std::integral_constant<int, N>;

constexpr int TH = 8, TW = 28;                 // output tile
constexpr int HH = TH + 2, HW = TW + 2;        // halo tile: 10 x 30 = 300 pixels
constexpr int NHALO = HH * HW;                 // 300
constexpr int NH_FR = 10;                      // fragments (of 32 GEMM columns) covering the halo: 320 columns
constexpr int NP_FR = 7;                       // fragments covering the 224 output pixels, all full
constexpr int RN = 128;                        // outputs of the next stage's first convolution
constexpr int W2_CHUNKS = 37;                  // 16-byte chunks per 3x3 weight row in LDS: 36 + 1 pad (bank spread)
constexpr int NROWS = (NHALO + 15) / 16 * 16;  // pixel rows of a stage: whole loads of a wave
constexpr int TP = 80;                         // bytes per pixel of t1 and t2 in LDS: 64 + 16 (bank spread without a swizzle, so that taps are immediate offsets)

// MODE 0: head (t2 stored); 1: whole identity block (residual = x); 2: whole first block of a stage --
// the residual is itself a 1x1 convolution of x (projection shortcut, Cin = 64), computed here as well; 3: an identity
// block of 256 channels and the 1x1 convolution into 128 channels that reads its sum (the next stage's first); 4: an
// identity block of 256 channels.
template <int MODE, int RQ, int RQA>
__global__ __launch_bounds__(512, 4) void bottleneck_kernel(const BneckParams p) {
    constexpr bool TAIL = MODE != 0, PROJ = MODE == 2, IDENTITY = MODE == 1 || MODE >= 3, REDUCE = MODE == 3;
    constexpr int NK = MODE == 2 ? 1 : MODE >= 3 ? 4 : 0;              // K steps of the first convolution, 0: any number
    constexpr int KB = 64, STAGE = (64 + NROWS) * KB;                 // 64 weight rows, then the pixel rows
    constexpr int TBYTES = NHALO * TP;                                // t1: [halo pixel][64 channels]; later t2: [output pixel][64 channels]
    constexpr int WBYTES = 64 * W2_CHUNKS * 16;                       // 3x3 weights
    constexpr int FRONT = NK == 1 ? WBYTES : 2 * STAGE;
    static_assert(FRONT >= WBYTES && FRONT >= STAGE && STAGE <= TBYTES, "regions");
    // step 1: three stages; from step 2 on the 3x3 weights in the space of the first two, t1 in that of the third
    __shared__ __attribute__((aligned(16))) int8_t Ls[FRONT + TBYTES];
    int8_t *const T = Ls + FRONT;
    __shared__ __attribute__((aligned(8))) uint2 at_s[32 * NP_FR];   // per output pixel: index (image, row, column) or ~0 (outside the image, not stored); byte offset of its row in a stage
    __shared__ int prm[2][4][64];                                     // bias, M0, chi, shift-1 of the first two convolutions
    __shared__ __attribute__((aligned(16))) int prm3[TAIL ? 4 : 1][TAIL ? 256 : 4];
    __shared__ __attribute__((aligned(16))) int prmp[PROJ ? 4 : 1][PROJ ? 256 : 4];   // the same for the projection
    __shared__ __attribute__((aligned(16))) int prmr[REDUCE ? 4 : 1][REDUCE ? RN : 4];  // and for the next stage's convolution

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l = lane & 31, half = lane >> 5;
    // first two convolutions: 32 channels x a quarter of the fragments; waves w and w + 4 share a SIMD and together
    // have the same number of fragments as the other pairs (five of the ten), resp. one more or less (seven)
    const int wm = wave & 1, wn = wave >> 1;
    // tiles that share halo rows run on the same XCD (workgroup ids are dealt round-robin over 8 XCDs)
    const int nblk = gridDim.x;
    const int xcd = blockIdx.x & 7, per = nblk >> 3, extra = nblk & 7;
    const int logical = xcd * per + (xcd < extra ? xcd : extra) + (blockIdx.x >> 3);
    const int tiles_x = (p.W + TW - 1) / TW, tiles_y = (p.H + TH - 1) / TH;
    const int b = logical / (tiles_x * tiles_y), t = logical % (tiles_x * tiles_y);
    const int oy0 = (t / tiles_x) * TH, ox0 = (t % tiles_x) * TW;     // first output pixel of the tile
    const int y0 = oy0 - 1, x0 = ox0 - 1;                            // image position of halo pixel (0, 0)

    // ---- step 1: t1 accumulators over the halo, K = Cin_p in steps of 64 ----
    // LDS position (row, col) of a stage holds K chunk col ^ swz(row); a lane fetches the same
    // chunk `cl` for all its rows (their numbers differ by multiples of 128): the weight row tid / 4 (waves 0 .. 3) or
    // pixel row tid / 4 - 64, and two more pixel rows (the last wave has one: it fetches that twice)
    const int col = tid & 3, row0 = tid >> 2, cl = col ^ swz<4>(row0);
    const bool short_wave = wave == 7;
    static_assert(64 + NROWS == 2 * 128 + 7 * 16, "the last wave's third rows do not exist");
    const int8_t *row[3];
    bool inside[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const int h = row0 + 128 * (j == 2 && short_wave ? 1 : j) - 64, hy = h / HW, hx = h - hy * HW, y = y0 + hy, x = x0 + hx;
        inside[j] = h >= 0 && h < NHALO && (unsigned)y < (unsigned)p.H && (unsigned)x < (unsigned)p.W;
        row[j] = p.in + (((long)b * p.H + y) * p.W + x) * p.Cin_p + cl * 16;
        if (j == 0 && wave < 4) { inside[j] = true; row[j] = p.w1 + (long)row0 * p.Cin_p + cl * 16; }
        // halo pixels outside the image (and the 4 rows past the halo): any readable bytes,
        // their results are replaced in step 2 or never used
        if (!inside[j]) row[j] = p.zpad;
    }
    const uint32_t lds0 = lds_address(Ls);
    auto issue = [&](int ks, int buf) {
#pragma unroll
        for (int j = 0; j < 3; ++j)
            ISR_GLOBAL_TO_LDS16_AT(row[j] + (inside[j] ? ks * KB : 0), lds0 + (buf == 2 ? FRONT : buf * STAGE) + (j == 2 && short_wave ? 1 : j) * 8192 + wave * 1024);
    };
    // With 256 input channels every operand is on its way before any is waited for: steps 0 and 1, the constants behind them,
    // step 2 and, in registers until a stage is free, step 3.
    const int nk = NK ? NK : p.Cin_p / KB;
    issue(0, 0);
    if (NK != 1 && nk > 1) issue(1, 1);
    v4i late[3];
    {
        const int cv = (tid >> 6) & 1, c = tid & 63, ct = tid < p.Cout_p ? tid : 0;
        const RqRaw r12 = cv ? rq_fetch(p.bias2, p.m0s2, p.chi2, p.shm12, c) : rq_fetch(p.bias1, p.m0s1, p.chi1, p.shm11, c);
        RqRaw r3{}, rp{};
        if constexpr (TAIL) r3 = rq_fetch(p.bias3, p.m0s3, p.chi3, p.shm13, ct);
        if constexpr (PROJ) rp = rq_fetch(p.biasp, p.m0sp, p.chip, p.shm1p, ct);
        if constexpr (REDUCE) rp = rq_fetch(p.biasp, p.m0sp, p.chip, p.shm1p, tid & (RN - 1));
        asm volatile("" ::: "memory");   // the loads above come first
        if (NK != 1 && nk > 2) issue(2, 2);
        if constexpr (NK == 4)
#pragma unroll
            for (int j = 0; j < 3; ++j) late[j] = *(const v4i *)(row[j] + (inside[j] ? 3 * KB : 0));
        if (tid < 32 * NP_FR) {
            const int oy = tid / TW, ox = tid - oy * TW, hp = (oy + 1) * HW + ox + 1;   // the output pixel's own halo position
            const bool store = oy0 + oy < p.H && ox0 + ox < p.W && !(REDUCE && p.sparse && ((oy | ox) & 1));   // (a tile starts at an even pixel)
            at_s[tid] = make_uint2(store ? (uint32_t)((b * p.H + oy0 + oy) * p.W + ox0 + ox) : ~0u, (uint32_t)(64 * KB + hp * KB + (swz<4>(hp) << 4)));
        }
        if (tid < 128) rq_store<RQ>(prm[cv], r12, c);
        if constexpr (TAIL)
            if (tid < p.Cout_p) {
                rq_store<RQ>(prm3, r3, ct);
                if constexpr (PROJ) rq_store<RQ>(prmp, rp, ct);
            }
        if constexpr (REDUCE)
            if (tid < RN) rq_store<RQ>(prmr, rp, tid);
    }
    if constexpr (NK == 4) wait_vmcnt<6>();   // steps 0 and 1 landed
    else if (nk > 2) wait_vmcnt<3>();
    else wait_vmcnt<0>();
    lds_barrier();   // they and the constants are visible

    const int c16 = wm * 32 + 16 * half;   // first of the lane's 16 channels in the first two convolutions
    const int f1 = wn * 3 - (wn == 3), n1 = wn < 2 ? 3 : 2;   // first fragment and their number: 3, 3, 2, 2
    v16i acc[3];
#pragma unroll
    for (int f = 0; f < 3; ++f)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[f][i] = prm[0][0][c16 + i];
    // TAIL: the residual of the closing add is x itself.  Wave w will own output channels [32 w, 32 w + 32) there,
    // input channels of K step w / 2 of this GEMM: while that step's pixel rows sit in the LDS stage the wave copies
    // its residual values (its 32 channels of the seven fragments' pixels) into registers, so x is not read from memory
    // a second time.
    // (With a projection shortcut x has only 64 channels and is the pixel operand of a second GEMM: it is
    // read again from memory -- cache hits, a fifth of the block's traffic at most.)
    v4i resid[NP_FR];
    {
        int aoff[2], boffs[2][3];   // [K half of the step][fragment]
#pragma unroll
        for (int ksub = 0; ksub < 2; ++ksub) {
            const int c = ksub * 2 + half;
            const int ra = wm * 32 + l;
            aoff[ksub] = ra * KB + ((c ^ swz<4>(ra)) << 4);
#pragma unroll
            for (int f = 0; f < 3; ++f) {
                const int rb = (f1 + (f < n1 ? f : 0)) * 32 + l;
                boffs[ksub][f] = 64 * KB + rb * KB + ((c ^ swz<4>(rb)) << 4);
            }
        }
        auto compute = [&](int ks, int buf) {
            const int8_t *base = buf == 2 ? T : Ls + buf * STAGE;
            if constexpr (IDENTITY) {
                if (ks == wave >> 1) {   // wave-uniform
#pragma unroll
                    for (int f = 0; f < NP_FR; ++f) resid[f] = *(const v4i *)(base + (at_s[f * 32 + l].y ^ (uint32_t)((wm * 2 + half) << 4)));
                }
            }
#pragma unroll
            for (int ksub = 0; ksub < 2; ++ksub) {
                const v4i fa = *(const v4i *)(base + aoff[ksub]);
                v4i fb[3];
#pragma unroll
                for (int f = 0; f < 3; ++f) fb[f] = *(const v4i *)(base + boffs[ksub][f]);
#pragma unroll
                for (int f = 0; f < 3; ++f)
                    if (f < 2 || n1 == 3) acc[f] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa, fb[f], acc[f], 0, 0, 0);
            }
        };
        if constexpr (NK == 4) {
            compute(0, 0);
            compute(1, 1);
            wait_vmcnt<3>();
            lds_barrier();   // step 2 landed; every wave is done with step 0
#pragma unroll
            for (int j = 0; j < 3; ++j) *(v4i *)(Ls + (j == 2 && short_wave ? 1 : j) * 8192 + tid * 16) = late[j];
            compute(2, 2);
            lds_barrier();
            compute(3, 0);
        } else {
            for (int ks = 0, buf = 0; ks < nk; ++ks) {   // buffer: ks mod 3
                if (ks > 0) {
                    if (ks + 1 < nk) wait_vmcnt<3>();
                    else wait_vmcnt<0>();
                    lds_barrier();   // every wave's loads of step ks landed; every wave is done with step ks - 1
                    if (ks + 2 < nk) issue(ks + 2, buf == 0 ? 2 : buf - 1);
                }
                compute(ks, buf);
                buf = buf == 2 ? 0 : buf + 1;
            }
        }
    }
    __syncthreads();   // every wave is done with the operand stages

    // 3x3 weights -> LDS (the space of the stages): row r at chunk r * 37, 36 chunks + 1 pad
    {
        constexpr int TOTAL = 64 * W2_CHUNKS;            // 2368 = 4 * 512 + 5 * 64: the last pass is waves 0 .. 4
#pragma unroll
        for (int pass = 0; pass < (TOTAL + 511) / 512; ++pass) {
            if (pass * 512 + wave * 64 < TOTAL) {        // wave-uniform
                const int q = pass * 512 + tid, r = q / W2_CHUNKS, c = q % W2_CHUNKS;
                ISR_GLOBAL_TO_LDS16_AT(p.w2 + (long)r * 576 + (c < 36 ? c : 0) * 16, lds0 + (pass * 512 + wave * 64) * 16);
            }
        }
    }

    // ---- step 2: requantise t1 into the LDS tile ----
    {
        const uint32_t zt = (uint32_t)(p.zp_t1 & 0xFF) * 0x01010101u;
        int mm[16], ch[16], ss[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) { mm[i] = prm[0][1][c16 + i]; ch[i] = prm[0][2][c16 + rq_chi_at<RQ>(i)]; ss[i] = prm[0][3][c16 + i]; }
        const RqLayer L = rq_layer<RQ>(prm[0][2][0], prm[0][3][0]);
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            if (f == 2 && n1 != 3) continue;   // wave-uniform
            const int h = (f1 + f) * 32 + l, hy = h / HW, hx = h - hy * HW, y = y0 + hy, x = x0 + hx;
            const bool ok = h < NHALO && (unsigned)y < (unsigned)p.H && (unsigned)x < (unsigned)p.W;
            int q[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) q[i] = rq_conv<RQ>(acc[f][i], mm[i], ch[i], ss[i], p.lo1, L);
            v4i v = rq_pack16<RQ>(q, L);
            if (!ok) v = v4i{(int)zt, (int)zt, (int)zt, (int)zt};
            if (h < NHALO) *(v4i *)(T + h * TP + (wm * 2 + half) * 16) = v;
        }
    }
    wait_vmcnt<0>();
    __syncthreads();   // t1 tile and 3x3 weights in LDS

    // the lane's weights of the 1x1 convolutions to come: on their way while the 3x3 runs
    auto rows64 = [&](const int8_t *w, v4i (&fa)[2]) {
#pragma unroll
        for (int ksub = 0; ksub < 2; ++ksub) fa[ksub] = *(const v4i *)(w + (wave * 32 + l) * 64 + ksub * 32 + half * 16);
    };
    v4i f3[2], fp[2], fr[4];
    if (TAIL && wave * 32 < p.Cout_p) {
        rows64(p.w3, f3);
        if constexpr (PROJ) rows64(p.wp, fp);
    }

    // ---- step 3: 3x3 convolution from LDS: this wave's 32 channels x its 2 (wn < 3) or 1 fragments ----
    const int nfr = wn < 3 ? 2 : 1;   // wave-uniform
    const int8_t *tb[2];                  // the lane's chunk of halo pixel (0, 0) of the taps of its output pixel in fragment f
#pragma unroll
    for (int f = 0; f < 2; ++f) {
        const int o = (wn * 2 + f) * 32 + l, oo = o < TH * TW ? o : 0, oy = oo / TW, ox = oo - oy * TW;
        tb[f] = T + (oy * HW + ox) * TP + half * 16;
    }
    const int8_t *wb = Ls + ((wm * 32 + l) * W2_CHUNKS + half) * 16;
    {
        v16i init;
#pragma unroll
        for (int i = 0; i < 16; ++i) init[i] = prm[1][0][c16 + i];
#pragma unroll
        for (int f = 0; f < 2; ++f) acc[f] = init;
    }
#pragma unroll
    for (int ks = 0; ks < 18; ++ks) {
        const int tap = ks >> 1, ky = tap / 3, kx = tap % 3;
        const v4i fa = *(const v4i *)(wb + ks * 32);
        v4i fb[2];
#pragma unroll
        for (int f = 0; f < 2; ++f) fb[f] = *(const v4i *)(tb[f] + (ky * HW + kx) * TP + (ks & 1) * 32);
#pragma unroll
        for (int f = 0; f < 2; ++f)
            if (f < 1 || nfr == 2) acc[f] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa, fb[f], acc[f], 0, 0, 0);
    }

    // ---- step 4: requantise t2 ----
    v4i t2[2];
    {
        int mm[16], ch[16], ss[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) { mm[i] = prm[1][1][c16 + i]; ch[i] = prm[1][2][c16 + rq_chi_at<RQ>(i)]; ss[i] = prm[1][3][c16 + i]; }
        const RqLayer L = rq_layer<RQ>(prm[1][2][0], prm[1][3][0]);
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            if (f == 1 && nfr != 2) { t2[f] = v4i{0, 0, 0, 0}; continue; }
            int q[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) q[i] = rq_conv<RQ>(acc[f][i], mm[i], ch[i], ss[i], p.lo2, L);
            t2[f] = rq_pack16<RQ>(q, L);
        }
    }
    if constexpr (!TAIL) {
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            if (f == 1 && nfr != 2) continue;
            const int o = (wn * 2 + f) * 32 + l, oy = o / TW, ox = o - oy * TW;
            if (oy0 + oy < p.H && ox0 + ox < p.W)
                *(v4i *)(p.out + (((long)b * p.H + oy0 + oy) * p.W + ox0 + ox) * 64 + c16) = t2[f];
        }
    } else {
        __syncthreads();   // every wave is done reading the t1 tile: t2 takes its place, [output pixel][64 channels]
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            if (f == 1 && nfr != 2) continue;
            const int o = (wn * 2 + f) * 32 + l;
            *(v4i *)(T + o * TP + (wm * 2 + half) * 16) = t2[f];
        }
        __syncthreads();   // the t2 tile is complete

        if constexpr (REDUCE)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) fr[ks] = *(const v4i *)(p.wp + ((wave * 4 + ks) * 64 + lane) * 16);

        // ---- last 1x1 convolution + residual add: this wave's 32 output channels, all seven pixel fragments ----
        // Registers are short: one fragment at a time, its accumulators start from the bias in LDS, and the forms of the
        // requantisation with three constants a channel read those there as well.
        if (wave * 32 >= p.Cout_p) return;   // no barrier follows
        const AddConst ac = add_const<RQA>(p);
        const int m0 = wave * 32, c0 = m0 + 16 * half;   // the lane's 16 channels
        auto pixel = [&](int f) { return at_s[f * 32 + l].x; };
        // the fragments of one 1x1 convolution from 64 channels: operand(f, K half), then use(f, results of rq_conv)
        constexpr bool KEEP = rq_is_top(RQ) || RQ == RQ_PAIR;
        auto conv64 = [&](const v4i (&fa)[2], const auto &prm, int lo, auto first, auto end, auto operand, auto use) {
            asm volatile("" ::: "memory");
            int mm[16], ch[16], ss[16];
            auto constants = [&]() {
#pragma unroll
                for (int i = 0; i < 16; ++i) { mm[i] = prm[1][c0 + i]; ch[i] = prm[2][c0 + rq_chi_at<RQ>(i)]; ss[i] = prm[3][c0 + i]; }
            };
            const RqLayer L = rq_layer<RQ>(prm[2][0], prm[3][0]);
            if constexpr (KEEP) constants();
#pragma unroll
            for (int f = decltype(first)::value; f < decltype(end)::value; ++f) {
                asm volatile("" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
                v16i a;
#pragma unroll
                for (int i = 0; i < 16; ++i) a[i] = prm[0][c0 + i];
#pragma unroll
                for (int ksub = 0; ksub < 2; ++ksub) a = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[ksub], operand(f, ksub), a, 0, 0, 0);
                if constexpr (!KEEP) constants();
                int q[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) q[i] = rq_conv<RQ>(a[i], mm[i], ch[i], ss[i], lo, L);
                use(f, q, L);
            }
        };
        if constexpr (PROJ) {
            // projection shortcut first: r = clamp(requant(Wp x)), kept packed; x at the lane's pixel is fetched a fragment
            // ahead (pixels outside the image read pixel 0: in bounds, unused)
            v4i xn[2], x[2];
            auto fetch = [&](int f) {
                const uint32_t px = pixel(f);
#pragma unroll
                for (int ksub = 0; ksub < 2; ++ksub) xn[ksub] = *(const v4i *)(p.in + (uint64_t)(px != ~0u ? px : 0) * 64 + ksub * 32 + half * 16);
            };
            fetch(0);
            conv64(fp, prmp, p.lop, Frag<0>{}, Frag<NP_FR>{}, [&](int f, int ksub) {
                if (ksub == 0) {
                    x[0] = xn[0]; x[1] = xn[1];
                    if (f + 1 < NP_FR) fetch(f + 1);
                }
                return x[ksub];
            }, [&](int f, const int (&q)[16], const RqLayer &L) {
                resid[f] = rq_pack16<RQ>(q, L);
                asm volatile("" : "+v"(resid[f]));   // packed: the compiler would keep the sixteen values
            });
        }
        auto t2_operand = [&](int f, int ksub) {
            return *(const v4i *)(T + (f * 32 + l) * TP + (ksub * 2 + half) * 16);
        };
        auto sum = [&](int f, const int (&q)[16], const RqLayer &L) {
            v4i y;
#pragma unroll
            for (int i = 0; i < 4; ++i) y[i] = (int)rq_add4<RQ, RQA>(q[4 * i], q[4 * i + 1], q[4 * i + 2], q[4 * i + 3], (uint32_t)resid[f][i], ac, L);
            return y;
        };
        if constexpr (!REDUCE) {
            conv64(f3, prm3, p.lo3, Frag<0>{}, Frag<NP_FR>{}, t2_operand, [&](int f, const int (&q)[16], const RqLayer &L) {
                const v4i y = sum(f, q, L);
                const uint32_t px = pixel(f);
                if (px != ~0u) *(v4i *)(p.out + c0 + (uint64_t)px * (uint32_t)p.Cout_p) = y;
            });
        } else {
            // The sum goes to memory (only its even pixels where nothing but a stride-2 projection reads it) and, three, two
            // and two fragments at a time, into LDS: [pixel][256 channels], chunk c of pixel p at c ^ (p & 15), in the space of
            // the 3x3 weights.  After a barrier each wave makes 16 of the next convolution's channels of those pixels
            // while the others go on to the next fragments, which have a region of their own.
            const RqLayer Lr = rq_layer<RQ>(prmr[2][0], prmr[3][0]);
            auto group = [&](auto first, auto end, int region) {
                constexpr int F0 = decltype(first)::value, F1 = decltype(end)::value;
                const int ln = lane & 15, g = lane >> 4, oc = wave * 16 + 4 * g;
                conv64(f3, prm3, p.lo3, first, end, t2_operand, [&](int f, const int (&q)[16], const RqLayer &L) {
                    const v4i y = sum(f, q, L);
                    const uint32_t px = pixel(f);
                    const int i = (f - F0) * 32 + l;
                    if (f == 0)   // no wait for a store behind them
#pragma unroll
                        for (int ks = 0; ks < 4; ++ks) asm volatile("" : "+v"(fr[ks]));
                    *(v4i *)(&Ls[region + i * 256 + (((2 * wave + half) ^ (i & 15)) << 4)]) = y;
                    if (px != ~0u) *(v4i *)(p.out + c0 + (uint64_t)px * 256) = y;
                });
                int bias[4], mm[4], ch[4], ss[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) { bias[i] = prmr[0][oc + i]; mm[i] = prmr[1][oc + i]; ch[i] = prmr[2][oc + rq_chi_at<RQ>(i)]; ss[i] = prmr[3][oc + i]; }
                lds_barrier();   // the group's sums are complete
                const bool full = oy0 + TH <= p.H && ox0 + TW <= p.W;
#pragma unroll
                for (int nb = 0; nb < 2 * (F1 - F0); ++nb) {
                    v4acc a = {bias[0], bias[1], bias[2], bias[3]};
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks)
                        a = __builtin_amdgcn_mfma_i32_16x16x64_i8(fr[ks], *(const v4i *)(&Ls[region + (16 * nb + ln) * 256 + (((4 * ks + g) ^ ln) << 4)]), a, 0, 0, 0);
                    int q[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) q[i] = rq_conv<RQ>(a[i], mm[i], ch[i], ss[i], p.lop, Lr);
                    // sixteen pixels of the tile from a constant one on: they lie in one row or in two
                    const int cy = (F0 * 32 + 16 * nb) / TW, cx = (F0 * 32 + 16 * nb) % TW;
                    const bool wrap = cx + ln >= TW;
                    const uint32_t at = (uint32_t)((b * p.H + oy0 + cy) * p.W + ox0 + cx) + (uint32_t)(ln + (wrap ? p.W - TW : 0));
                    if (full || (oy0 + cy + wrap < p.H && ox0 + cx + ln - (wrap ? TW : 0) < p.W))
                        *(uint32_t *)(p.out2 + (at * RN + (uint32_t)oc)) = rq_pack<RQ>(q[0], q[1], q[2], q[3], Lr);
                }
            };
            static_assert(5 * 32 * 256 <= FRONT && 3 + 2 + 2 == NP_FR, "regions");
            group(Frag<0>{}, Frag<3>{}, 0);
            group(Frag<3>{}, Frag<5>{}, 3 * 32 * 256);
            group(Frag<5>{}, Frag<7>{}, 0);   // every wave is done with the first group: it has passed the second's barrier
        }
    }
}

}  // namespace

// Geometry with a kernel: first convolution 1x1 (stride 1) from a multiple of 64 stored channels
// into 64; second 3x3 stride 1 pad 1, 64 -> 64; optional tail 1x1 from 64 back to the input's
// channel count (at most 256) with the block input as residual.
bool bottleneck_supported(int cin_p, int cmid_p, int cout_p, int tail) {
    if (cin_p % 64 != 0 || cin_p < 64 || cin_p > 1024 || cmid_p != 64) return false;
    if (tail == 2) return cin_p == 64 && cout_p % 64 == 0 && cout_p >= 64 && cout_p <= 256;   // projection shortcut from 64 channels
    return !tail || (cout_p == cin_p && cout_p <= 256);
}

hipError_t launch_bottleneck(const BneckParams &p, hipStream_t st) {
    if (p.B <= 0) return hipSuccess;
    if (!p.in || !p.out || !p.w1 || !p.w2 || !p.zpad || p.H < 1 || p.W < 1 ||
        !bottleneck_supported(p.Cin_p, 64, p.Cout_p, p.tail ? (p.proj ? 2 : 1) : 0) || (p.tail && !p.w3) ||
        ((p.proj || p.reduce) && (!p.tail || !p.wp || !p.biasp || !p.m0sp || !p.chip || !p.shm1p)) ||
        (p.reduce && (p.proj || !p.out2 || p.Cout_p != 256 || (p.sparse && (p.H & 1)))))
        return hipErrorInvalidValue;
    const long tiles = (long)p.B * ((p.H + TH - 1) / TH) * ((p.W + TW - 1) / TW);
    if (tiles > 0x7fffffffL || (long)p.B * p.H * p.W * (p.Cin_p > 64 ? p.Cin_p : 64) >= (1L << 31)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)tiles), block(512);
    const int mode = p.tail ? (p.proj ? 2 : p.reduce ? 3 : 1) : 0;
    // Resident workgroups keep the weights, but their time goes in rounds of 256 tiles, that of this file's kernel with the tiles.  The lines lie where a
    // round just begun costs no more, or hardly.  us, this file's / resident, at 5.03, 6.02, 8.04, 10.01, 12.03, 16.02 and 36.5 rounds:
    //   identity block  RQ_PAIR      55.0/53.4  63.1/59.4  77.7/72.1    97.7/84.9    114/101  149/129  329/288
    //                   RQ_TOP       55.5/55.0  64.2/62.0  79.3/75.3    100/88.4     114/103  149/131  310/279
    //                   RQ_TIE_FREE  64.5/61.4  76.2/69.0  92.7/85.5    116/99.7     135/117  175/153  393/338
    //                   RQ_ANY       71.8/69.1  83.1/76.8  108/98.9     128/116      149/135  191/175  433/390
    //                   RQ_TOP_TIES  64.4/64.9  74.5/72.3  94.8/92.1    113/108      130/126  167/162  371/357
    //   first block     RQ_PAIR      48.6/49.7  56.6/56.2  72.6/68.8    85.3/81.7    101/95   134/124  319/278
    //                   RQ_TIE_FREE  67.3/64.8  77.2/74.1  98.8/93.1    119/112      139/131  182/171  426/385
    //                   RQ_ANY       76.6/75.9  88.6/86.4  116/110      136/131      161/155  207/196  484/448
    //                   RQ_TOP_TIES  69.2/69.8  79.7/79.6  101.5/101.4  121/120      145/142  187/180  425/411
    //                   RQ_TOP       52.5/56.4  61.2/63.2  77.0/78.2    90.2/93.1    107/109  140/140  322/307
    //                     (an add with exact halves: 57.0/60.2, 82.9/84.6, 97.8/100, 116/119, 153/152, 347/335)
    // (at 3.3 rounds 39.0/39.1, 39.2/40.6, 46.6/45.1, 50.7/50.2, 46.1/47.2; 37.3/38.1, 48.9/47.5, 54.7/55.0, 49.8/50.4, 39.0/42.3)
    const int form = p.rq & p.add_rq & RQ_PAIR ? (int)RQ_PAIR : p.rq & ~RQ_PAIR;
    const int rounds = p.proj ? (form == RQ_TOP ? 16 : form == RQ_TOP_TIES ? 9 : 6) : form == RQ_TOP_TIES ? 6 : 5;
    if (((mode == 1 && p.Cin_p == 256) || (mode == 2 && p.Cout_p == 256)) && tiles >= 256 * rounds && (long)p.B * p.H * p.W * 256 < (1L << 31))
        return launch_bottleneck_stream(p, (int)tiles, st);
    static const char *const names[4][2] = {{"bottleneck_kernel<head, false>", "bottleneck_kernel<head, true>"},
                                            {"bottleneck_kernel<block, false>", "bottleneck_kernel<block, true>"},
                                            {"bottleneck_kernel<block + projection, false>", "bottleneck_kernel<block + projection, true>"},
                                            {"bottleneck_kernel<block + next, false>", "bottleneck_kernel<block + next, true>"}};
    set_kernel_name(names[mode][(p.rq & RQ_TIE_FREE) && (mode == 0 || p.add_rq != RQ_ANY)]);
    with_rq(p.rq, p.add_rq, [&](auto rq, auto rqa) {
        constexpr int RQ = decltype(rq)::value, RQA = decltype(rqa)::value;
        if (mode == 3) hipLaunchKernelGGL((bottleneck_kernel<3, RQ, RQA>), grid, block, 0, st, p);
        else if (mode == 2) hipLaunchKernelGGL((bottleneck_kernel<2, RQ, RQA>), grid, block, 0, st, p);
        else if (mode == 1 && p.Cin_p == 256) hipLaunchKernelGGL((bottleneck_kernel<4, RQ, RQA>), grid, block, 0, st, p);
        else if (mode == 1) hipLaunchKernelGGL((bottleneck_kernel<1, RQ, RQA>), grid, block, 0, st, p);
        else hipLaunchKernelGGL((bottleneck_kernel<0, RQ, RQA>), grid, block, 0, st, p);
    });
    return hipGetLastError();
}

}  // namespace isr
