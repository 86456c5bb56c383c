// First layer fused with the max pooling that follows it: 7x7 stride-2 convolution
// (pad 3) of the noisy NHWC4 image into 64 channels, then 3x3 stride-2 max pooling
// (pad 1, in-bounds taps only), then requantisation + clamp -- in that order: for a
// positive multiplier the requantisation z + RHA(acc M0, s) and the clamp are
// non-decreasing in acc, so the maximum over a window of requantised values equals
// the requantised maximum of the int32 accumulators.  Pooling the accumulators first
// requantises a quarter of the values and nothing but the pooled tensor leaves the CU.
//
// A wave makes 32 of the 64 channels of 4 pooled rows x 31 pooled columns; 8 waves (both channel halves of 2 row groups x 2
// column strips, or of 4 row groups for images of at most 31 pooled columns) share in LDS
//   * the 64 x 256-byte weight matrix (K = (ky, kx padded to 8, channel padded to 4)),
//   * the input rows of their band, shifted right by 3 pixels and padded with the input
//     zero-point, so that the 16 K-bytes of an MFMA fragment lane -- 4 horizontally
//     adjacent taps x 4 channels -- are 16 contiguous, 8-byte aligned LDS bytes.
// Per convolution row the wave computes one MFMA fragment of the 32 even columns
// 2 px and one of the odd columns 2 px - 1 (v_mfma_i32_32x32x32_i8, one K step per
// kernel row, both operands from LDS, no global gather); the horizontal maximum of a
// pooled pixel is then lane-local but for the right neighbour, fetched with a DPP
// wave shift, and the vertical maximum runs in registers over the 9 rows.
//
// Bound by the issue of integer arithmetic, half of it the noise.  Bands of 8 pooled rows draw 39 rows of noise for 32 (bands of
// 4: 23 for 16), waves of 4 pooled rows compute 9 convolution rows for 8 (waves of 2: 5 for 4), the bias joins the maxima
// and not the accumulators, and a column outside the image is replaced by one of the same window instead of being masked:
// 668 copies of 224 x 224 303 -> 269 us by the bands, the waves and the bias, 291 -> 246 us with the columns as well (each pair
// on a card of its own).  Even columns read as 16 bytes a lane (two reads of 8, 16 bytes apart from lane to lane, take half of the
// banks each: conflicts were 41 % of the cycles) and the neighbour's maximum in the DPP operand: 256 -> 239.5 us.
#include <climits>

#include "conv_device.h"
#include "noise_device.h"

namespace isr {

namespace {

constexpr int SP_WMAX = 224;            // widest input row held in LDS
constexpr int SP_K = 7, SP_KP = 256;    // kernel size; padded K bytes per output channel
constexpr int SP_STRIP = 31;            // pooled columns per wave
constexpr int SP_ROWS = 4;              // pooled rows per wave
constexpr int SP_NT = 512;
// input band: 39 rows of up to 232 pixels (two strips) or 71 rows of up to 132 (one strip)
constexpr int SP_IN_BYTES = 71 * (4 * SP_STRIP + 8) * 4;
static_assert(39 * (SP_WMAX + 8) * 4 <= SP_IN_BYTES, "two-strip band fits");
// pooled rows per workgroup
constexpr int sp_band(int nstrips) { return SP_ROWS * (SP_NT / 64 / 2) / nstrips; }

template <int RQ>
__global__ __launch_bounds__(SP_NT, 4) void stem_pool_kernel(const StemPoolParams p) {
    __shared__ __attribute__((aligned(16))) int8_t Wl[64 * SP_KP];
    __shared__ __attribute__((aligned(16))) int8_t In[SP_IN_BYTES];
    __shared__ __attribute__((aligned(16))) int prm[4][64];
    __shared__ __attribute__((aligned(16))) NoiseLds ntab;                 // the sampler's table when the kernel draws its own input

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nstrips = (p.Wp + SP_STRIP - 1) / SP_STRIP;       // 1 or 2 (checked by the launcher)
    const int P = sp_band(nstrips);
    const int nbands = (p.Hp + P - 1) / P;
    const int b = blockIdx.x / nbands, p0 = (blockIdx.x % nbands) * P;
    const int cy0 = 2 * p0 - 1;               // first convolution row of the band (may be -1)
    const int iy0 = 2 * cy0 - 3;              // first input row of the band
    const int IR = 4 * P + 7;                 // input rows of the band
    const int PW = p.W + 8;                   // patch row stride in pixels
    const uint32_t zb = (uint32_t)(p.zp_in & 0xFF) * 0x01010101u;

    // weights, constants and the sampler's table are all on their way before any of them is waited for
    v4i wv[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) wv[j] = *(const v4i *)(p.w + (long)(tid + SP_NT * j) * 16);
    const RqRaw raw = rq_fetch(p.bias, p.m0s, p.chi, p.shm1, tid & 63);
    const uint8_t *xim = nullptr;
    const DeviceNoiseTable *tab = nullptr;
    uint32_t image_id = 0;
    SlotUse use{};
    if (p.fused_noise) {
        use = resolve_noise_source(p.noise, b, xim, tab, image_id);
        store_noise_table<SP_NT>(ntab, fetch_noise_table<SP_NT>(tab, tid), tid);
    }
    // weights: row r, 16-byte chunk c at chunk position c ^ (r & 15)
    static_assert(64 * (SP_KP / 16) == 2 * SP_NT, "two chunks a thread");
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int r = (tid + SP_NT * j) >> 4, c = tid & 15;
        *(v4i *)(&Wl[r * SP_KP + ((c ^ (r & 15)) << 4)]) = wv[j];
    }
    if (tid < 64) rq_store<RQ>(prm, raw, tid);
    // input band: pixel (row r, input column x) at patch column x + 3
    const int wchunks = p.W >> 2;             // 16-byte chunks (4 pixels) per input row
    if (p.fused_noise) {
        // the noisy rows are drawn here instead of being read back from memory: the stream is counter-based,
        // so the rows that neighbouring bands share are simply drawn again, bit for bit the same
        const NoiseSampler smp = tab->s;
        __syncthreads();
        const int dr = SP_NT / wchunks, dc = SP_NT - dr * wchunks;
        for (int r = tid / wchunks, c = tid - r * wchunks; r < IR;) {
            const int iy = iy0 + r;
            uint32_t v[4] = {zb, zb, zb, zb};
            if ((unsigned)iy < (unsigned)p.H)
                noisy_quad(ntab, smp, tab, xim, p.noise.C, p.H, p.W, iy, c, use.sample, image_id, use.phase, p.noise.key0, p.noise.key1, v);
            int *dst = (int *)(&In[(r * PW + 3 + 4 * c) * 4]);
            dst[0] = (int)v[0]; dst[1] = (int)v[1]; dst[2] = (int)v[2]; dst[3] = (int)v[3];
            r += dr;
            c += dc;
            if (c >= wchunks) { c -= wchunks; ++r; }
        }
    } else {
        for (int i = tid; i < IR * wchunks; i += SP_NT) {
            const int r = i / wchunks, c = i - r * wchunks, iy = iy0 + r;
            v4i v = {(int)zb, (int)zb, (int)zb, (int)zb};
            if ((unsigned)iy < (unsigned)p.H) v = *(const v4i *)(p.in + (((long)b * p.H + iy) * p.W + 4 * c) * 4);
            int *dst = (int *)(&In[(r * PW + 3 + 4 * c) * 4]);
            dst[0] = v[0]; dst[1] = v[1]; dst[2] = v[2]; dst[3] = v[3];
        }
    }
    for (int i = tid; i < IR * 8; i += SP_NT) {   // 3 columns left, 5 right of the image
        const int r = i >> 3, c = i & 7;
        *(int *)(&In[(r * PW + (c < 3 ? c : p.W + c)) * 4]) = (int)zb;
    }
    __syncthreads();

    // ---- this wave: channels 32 fm .. 32 fm + 31 of pooled rows py0 .. py0 + 3, pooled columns px0 .. px0 + 30 ----
    const int fm = wave & 1, strip = (wave >> 1) % nstrips, rg = (wave >> 1) / nstrips;
    const int py0 = p0 + SP_ROWS * rg, px0 = strip * SP_STRIP;
    if (py0 >= p.Hp) return;                  // wave-uniform; no barrier follows
    const int l = lane & 31, half = lane >> 5;
    const int px = px0 + l;
    const bool pxok = l < SP_STRIP && px < p.Wp;
    const int oxe = pxok ? 2 * px : 0;                         // even fragment: column 2 px
    // odd fragment: column 2 px - 1 (left neighbour, and right neighbour of the lane before); outside the image the nearest
    // column, which is the centre of the window that wants it and leaves its maximum as it is
    const int oxo_raw = 2 * (px0 + l) - 1, oxo = oxo_raw < 0 ? 0 : oxo_raw < p.Wo ? oxo_raw : p.Wo - 1;
    const int8_t *srce = &In[(2 * oxe + 4 * half) * 4], *srco = &In[(2 * oxo + 4 * half) * 4];
    const int rowbytes = PW * 4;
    const int lo = p.relu ? p.zp_out : -128;

    const int oc = fm * 32 + 16 * half;       // first of the 16 channels this lane holds
    v4i fa[SP_K];
#pragma unroll
    for (int ky = 0; ky < SP_K; ++ky) {
        const int r = fm * 32 + l, c = ky * 2 + half;
        fa[ky] = *(const v4i *)(&Wl[r * SP_KP + ((c ^ (r & 15)) << 4)]);
    }
    int v[16];                                // running maxima of the current pooled row, bias not yet added
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = INT_MIN;
    const RqLayer L = rq_layer<RQ>(prm[2][0], prm[3][0]);
    auto emit = [&](int py) {
        if (!pxok) return;
        int q[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) q[i] = rq_conv<RQ>(v[i] + prm[0][oc + i], prm[1][oc + i], prm[2][oc + rq_chi_at<RQ>(i)], prm[3][oc + i], lo, L);
        *(v4i *)(p.out + ((((long)b * p.Hp + py) * p.Wp + px) << 6) + oc) = rq_pack16<RQ>(q, L);
    };
    // pooled row j takes convolution rows 2 j, 2 j + 1, 2 j + 2 of the wave's nine
#pragma unroll
    for (int r = 0; r < 2 * SP_ROWS + 1; ++r) {
        const int cyl = 2 * SP_ROWS * rg + r, cy = cy0 + cyl;   // convolution row: local, global
        const bool inside = (unsigned)cy < (unsigned)p.Ho;       // rows outside the image never win the max
        int h[16];
        if (inside) {
            v16i ae = {}, ao = {};
#pragma unroll
            for (int ky = 0; ky < SP_K; ++ky) {
                const int off = (2 * cyl + ky) * rowbytes;
                const long long o0 = *(const long long *)(srco + off), o1 = *(const long long *)(srco + off + 8);
                const v4i fe = *(const v4i *)(srce + off);   // a row is a multiple of 16 bytes, an even column at one
                const v4i fo = {(int)o0, (int)(o0 >> 32), (int)o1, (int)(o1 >> 32)};
                ae = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[ky], fe, ae, 0, 0, 0);
                ao = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[ky], fo, ao, 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                // lane + 1 holds column 2 px + 1 (wave_shl:1 reads the next lane; the last one, which has none, makes no pixel)
                const int right = __builtin_amdgcn_mov_dpp(ao[i], 0x130, 0xf, 0xf, true);
                if (r % 2) {
                    int m = max(v[i], max(ae[i], ao[i]));
                    asm("" : "+v"(m));   // three operands in one instruction and the neighbour in the next, which reads it by DPP
                    v[i] = max(m, right);
                } else {
                    h[i] = max(max(ae[i], ao[i]), right);
                    v[i] = max(v[i], h[i]);
                }
            }
        }
        if (r >= 2 && r % 2 == 0) {
            const int py = py0 + r / 2 - 1;
            emit(py);
            if (py + 1 >= p.Hp) return;
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = inside ? h[i] : INT_MIN;
        }
    }
}

}  // namespace

bool stem_pool_supported(int k, int stride, int pad, int cout_p, int H, int W, int fast_requant, int pool_k,
                         int pool_stride, int pool_pad) {
    return k == SP_K && stride == 2 && pad == 3 && cout_p == 64 && fast_requant && pool_k == 3 && pool_stride == 2 &&
           pool_pad == 1 && W % 4 == 0 && W >= 8 && W <= SP_WMAX && H >= 1;
}

hipError_t launch_stem_pool(const StemPoolParams &p, hipStream_t st) {
    if (p.B <= 0) return hipSuccess;
    // geometry the kernel assumes: 7x7/2 pad 3 then 3x3/2 pad 1, at most two strips of pooled columns
    if (p.W % 4 != 0 || p.W < 8 || p.W > SP_WMAX || p.Ho != (p.H - 1) / 2 + 1 || p.Wo != (p.W - 1) / 2 + 1 ||
        p.Hp != (p.Ho - 1) / 2 + 1 || p.Wp != (p.Wo - 1) / 2 + 1 || p.Wp > 2 * SP_STRIP || !p.out || !p.w)
        return hipErrorInvalidValue;
    if (p.fused_noise) {
        const NoiseSource &ns = p.noise;
        if (!ns.x || !ns.table || ns.C < 1 || ns.C > 3 || ns.H != p.H || ns.W != p.W || !valid_slots(ns.slots)) return hipErrorInvalidValue;
    } else if (!p.in) {
        return hipErrorInvalidValue;
    }
    const int nstrips = (p.Wp + SP_STRIP - 1) / SP_STRIP, P = sp_band(nstrips);
    if ((4 * P + 7) * (p.W + 8) * 4 > SP_IN_BYTES) return hipErrorInvalidValue;
    const long blocks = (long)p.B * ((p.Hp + P - 1) / P);
    if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
    set_kernel_name(p.fused_noise ? "stem_pool_kernel (+noise)" : "stem_pool_kernel");
    with_rq(p.rq, [&](auto rq) { hipLaunchKernelGGL((stem_pool_kernel<decltype(rq)::value>), dim3((unsigned)blocks), dim3(SP_NT), 0, st, p); });
    return hipGetLastError();
}

}  // namespace isr
