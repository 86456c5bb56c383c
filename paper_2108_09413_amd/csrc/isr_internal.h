// Internal declarations shared by the host code and the kernel launchers.
#ifndef ISR_INTERNAL_H
#define ISR_INTERNAL_H

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <memory>
#include <string>
#include <vector>

#include "isr.h"

namespace isr {

// ---- noise table -----------------------------------------------------------
// The threshold table T (2R ascending 64-bit values, T[2R - 1 - i] = ~T[i]) in the form of the device samplers.  A uniform
// u left of the centre draws #{i < R : T[i] <= u} - R, one right of it the mirrored value of ~u.  So with x the high
// word of u or ~u, whichever is below 2^31, one word of a guide table indexed by the exponent and the leading mantissa bits
// of float(x) tells the count: buckets get narrower towards the tail with the thresholds, and none holds two.
//   guide word = lowest index bit (31) | mantissa bits below the index of the bucket's threshold (all ones: none), left-aligned
//                below it | R - count before the threshold = |draw| left of it (bits 0 .. 13)
// A mantissa equal to the threshold's, or x below `lo`, is decided by the 64-bit thresholds themselves.
constexpr uint32_t NOISE_DRAW_MASK = 0x3FFF;  // sigma 1024: R = 8690
constexpr uint32_t NOISE_HALF_MAX = 256;      // pixels: thresholds of draws -255 .. -1 (saturation makes the rest meet 0 or 255)
constexpr uint32_t NOISE_GUIDE_MAX = 1920;    // words of a pixel table's guide
struct NoiseSampler {
    uint32_t shift, mask;       // byte offset of the guide word = (bits of float(x) >> shift) & mask
    uint32_t key_shift;         // lowest index bit and the mantissa bits below it, left-aligned = bits << key_shift
    uint32_t reach;             // thresholds in use: draws are -reach .. reach
    float lo, hi;               // float(x) is clamped to these
};
struct DeviceNoiseTable {
    NoiseSampler s;
    uint32_t hi[NOISE_HALF_MAX], lo[NOISE_HALF_MAX];   // high and low words of the thresholds
    alignas(16) uint32_t guide[NOISE_GUIDE_MAX];
};

bool build_noise_table(uint32_t sigma, std::vector<uint64_t> &T, uint32_t &R);
struct NoiseTable {
    std::vector<uint64_t> T;   // 2R ascending thresholds
    uint32_t R = 0;
};
// Shared, immutable table of a sigma (built on first use); null for sigma outside 1..1024.
std::shared_ptr<const NoiseTable> cached_noise_table(uint32_t sigma);
// Table of the stored-noise generator as one block of 32-bit words: guide table, n = R high words, n low words.
bool build_bank_table(uint32_t sigma, std::vector<uint32_t> &words, uint32_t &n_out, uint32_t &R_out);
struct NoiseBankParams;
// The table arguments of a launch from such a block in device memory (16-byte aligned).
void set_bank_table(NoiseBankParams &p, const uint32_t *dev, size_t words, uint32_t R);
// The guide words of a block into the form that noise_bank_kernel reads: |draw| left of the bucket's threshold << 16 | the 16 lowest
// float bits of the threshold.
void bank_guide(std::vector<uint32_t> &words, uint32_t R);
// Records the hipError_t that isr_last_device_error() reports on this thread.
void set_last_device_error(int hip_error);
bool build_device_table(uint32_t sigma, DeviceNoiseTable &out);

// One (image, sigma) pair of a batched call.
struct NoiseItem {
    uint32_t image;          // index into the array of clean images
    uint32_t table_slot;     // index into the array of noise tables
    uint32_t image_id;       // counter word of the random stream
};

// The copies of a call are one list of slots: n[0] samples of phase `phase` for each (image, sigma) pair, one pair after the
// other, then n[1] samples of the next phase likewise.  A launch works on the slots from `begin` on.
struct Slots {
    uint64_t begin;
    uint64_t split;                  // pairs * n[0]: the first slot of the second phase
    uint32_t n[2];
    uint32_t pairs, phase, first;    // first: sample index of a pair's first slot
};
// What the copy in a slot is: its random stream (phase, sample) and the tally row of its vote, [phases][pairs].
struct SlotUse {
    uint32_t phase, pair, sample, row;
};
#ifdef __HIPCC__
__host__ __device__
#endif
inline SlotUse slot_use(const Slots &l, uint64_t copy) {
    uint64_t s = l.begin + copy;
    const uint32_t second = s >= l.split;
    if (second) s -= l.split;
    uint32_t pair = 0;
    if (l.pairs > 1) {
        const uint32_t n = second ? l.n[1] : l.n[0];
        pair = (uint32_t)(s / n);
        s -= (uint64_t)pair * n;
    }
    return {l.phase + second, pair, l.first + (uint32_t)s, second * l.pairs + pair};
}

inline bool valid_slots(const Slots &l) { return l.pairs == 1 || (l.pairs > 1 && l.n[0] > 0); }

// Where the copies of a launch draw from.  Single pair: the call's own image and table; batch mode (items != null): the
// pair's of the slot.
struct NoiseSource {
    const uint8_t *x;                // [C][H][W] clean image ([images][C][H][W] in batch mode)
    const DeviceNoiseTable *table;   // the table (batch mode: table 0 of the array indexed by table_slot)
    const NoiseItem *items;
    uint32_t key0, key1, image;
    int32_t C, H, W;
    Slots slots;
};

// ---- parsed model (host) ---------------------------------------------------
enum OpType : int32_t { OP_CONV = 1, OP_ADD = 2, OP_MAXPOOL = 3, OP_GAP = 4, OP_FC = 5 };

struct TensorDesc {
    int32_t C, H, W, zp;
    int32_t Cp;          // channels as stored on the device (multiple of 16; 4 for the input)
};

struct HostOp {
    OpType type;
    int32_t a = -1, b = -1, out = -1;
    int32_t k = 0, stride = 1, pad = 0, relu = 0;
    int32_t Ma = 0, Mb = 0, sh = 0;
    std::vector<int8_t> w;                  // CONV: OIHW, FC: [Cout][Cin]
    std::vector<int32_t> bias, M0, shift;
};

struct ParsedModel {
    int32_t C = 0, H = 0, W = 0, classes = 0;
    std::vector<TensorDesc> tensors;
    std::vector<HostOp> ops;
};

// Returns ISR_OK / ISR_ERR_FORMAT / ISR_ERR_UNSUPPORTED; `why` gets a short reason.
int parse_model(const void *blob, size_t bytes, ParsedModel &out, std::string &why);

// ---- device-side op descriptors -------------------------------------------
// Forms of the requantisation and of the residual add (conv_device.h).  The class of a layer or an add is one of the first
// five values, with RQ_PAIR set beside it where that form serves it too.
enum Rq : int { RQ_ANY = 0, RQ_TIE_FREE = 1, RQ_TOP_TIES = 2, RQ_TOP = 3, RQ_TOP_WIDE = 4, RQ_PAIR = 8 };
constexpr int rq_form(int rq) { return rq & RQ_PAIR ? (int)RQ_PAIR : rq; }   // the form that a class takes
constexpr bool rq_is_top(int rq) { return rq >= RQ_TOP_TIES && rq <= RQ_TOP_WIDE; }
struct AddConst { int32_t ms, mr, c0, k, sh, lo; };   // constants of a residual add in its form

struct ConvParams {
    const int8_t *in;        // [B][H][W][Cin_p]
    int8_t *out;             // [B][Ho][Wo][Cout_p]
    const int8_t *w;         // [Mp][Kp] rows in MFMA row order, K = (tap, channel)
    const int32_t *bias;     // [Mp] bias - z_in * sum(w)
    const uint32_t *m0x2;    // [Mp] M0 << 1
    const uint32_t *rnd_lo;  // [Mp] low / high word of 2^(31 + shift)
    const uint32_t *rnd_hi;
    const uint32_t *shift;   // [Mp]
    const int32_t *m0s;      // [Mp] M0                                  } single-multiply path,
    const int32_t *chi;      // [Mp] 2^(shift-2) + z_out * 2^(shift-1)   } valid when every
    const int32_t *shm1;     // [Mp] shift - 1                           } shift is in [2, 22]
    int32_t fast_requant;
    // 1: no output channel can meet a negative acc * M0 = (odd) * 2^(30 + shift) within its accumulator range and above its
    // clamp, so that the sign correction of the rounding term changes nothing: the kernel then
    // takes (mulhi(acc, M0) + chi) >> (shift - 1) (decided per layer when the model is loaded)
    int32_t tie_free;
    int32_t rq;              // Rq class of this convolution's requantisation (conv_device.h)
    // residual add folded into the epilogue (fuse_add != 0): with q the int8 result above,
    //   v = q * add_mul_self + res * add_mul_res + add_c0            (= (q-z)Ms + (res-zr)Mr)
    //   out = clamp((v + add_k + (v >> 31)) >> add_sh, add_lo, 127)  (add_k = 2^(sh-1) + z_o 2^sh)
    const int8_t *res;       // [B][Ho][Wo][Cout_p] other input of the add
    int32_t fuse_add, add_mul_self, add_mul_res, add_c0, add_k, add_sh, add_lo;
    int32_t add_rq;          // Rq class of the add
    int32_t add_tie_free;    // 1: no pair of int8 inputs makes v a negative exact half above the clamp: out = clamp((v + add_k) >> add_sh)
    // fuse_add == 2: the residual is itself the output of a 1x1 stride-1 convolution (same pixels, same
    // channels) that has no other reader; the kernel computes it first, keeps it in registers and never
    // stores it.  Its operands:
    const int8_t *in2;       // [B][Ho][Wo][Cin2_p]
    const int8_t *w2;        // [Mp][Cin2_p] rows in MFMA row order
    const int32_t *bias2, *m0s2, *chi2, *shm12;   // as bias / m0s / chi / shm1
    int32_t Cin2_p, lo2, tie_free2, rq2;              // lo2: lower clamp of the residual tensor
    const uint32_t *ktab;    // [Kp/16] per 16-byte K chunk: ky | kx<<8, 0xFFFFFFFF = padding chunk; null = plain GEMM
    const int32_t *ktoff;    // [Kp/16] byte offset (ky*W + kx)*Cin_p + channel of the chunk
    const int8_t *zpad;      // 16 bytes of z_in: source of out-of-image taps for loads that go straight to LDS
    // 1x1 layers of the shapes expand_reduce.hip serves: the weights once more, one 1 KB block per MFMA operand
    // fragment (64 lanes x 16 bytes in lane order); null elsewhere
    const int8_t *wfrag;
    const int8_t *wfrag2;    // fuse_add == 2: the same of the residual convolution (w2)
    int32_t H, W, Cin_p, Ho, Wo, Cout_p;
    int32_t k, stride, pad, Kp, Mp;   // k: kernel size (k x k taps)
    int32_t force_tile;      // 0: the launcher picks the output tile; 1..7: 128x128, 128x256, 256x128, 256x256, 256x256 with 128x128 / 128x64 per wave, 256x256 of conv_patch.hip
    int32_t kb;              // K bytes per step of the kernel (64 or 128); Kp is a multiple of it
    int32_t zp_in, zp_out, relu;
    int32_t npix;            // B * Ho * Wo
    int32_t c4;              // 1: input is NHWC4 and a K chunk is 4 horizontal taps
};

// First convolution (7x7 stride 2 pad 3 on the NHWC4 image, 64 stored output channels)
// fused with the 3x3 stride-2 pad-1 max pooling that follows it.
struct StemPoolParams {
    const int8_t *in;        // [B][H][W][4] noisy image
    int8_t *out;             // [B][Hp][Wp][64] pooled activations
    const int8_t *w;         // [>= 64][256] rows in MFMA row order, K = (ky, kx padded to 8, channel padded to 4)
    const int32_t *bias, *m0s, *chi, *shm1;   // as in ConvParams (single-multiply requantisation)
    int32_t H, W, Ho, Wo, Hp, Wp;
    int32_t zp_in, zp_out, relu, rq, B;
    // fused_noise != 0: `in` is unused; the kernel draws the noisy input rows of its band itself (the
    // sampler of the noise stage on the same counter-based stream), copy b of the launch from `noise`
    int32_t fused_noise;
    NoiseSource noise;
};

// First convolution of the narrow small-image nets: 3x3 stride 1 pad 1 on the NHWC4 image
// into 16 stored channels (stem16.hip).
struct Stem16Params {
    const int8_t *in;        // [B][H][W][4]
    int8_t *out;             // [B][H][W][16]
    const int8_t *w;         // [16][64], K = (ky, kx padded to 4, channel padded to 4)
    const int32_t *bias, *m0s, *chi, *shm1;
    int32_t H, W, B, zp_in, lo, tie_free;
};

// The nets on 32 x 32 images with 16 / 32 / 64 channels at 32 / 16 / 8 pixels, one launch per stage, or of few copies one for all (narrow_net.hip).
// Per-channel constants come packed, int32 [4][C]: bias, M0, chi, shift-1.
struct NarrowBlock {         // identity residual block, stored in device memory
    const int8_t *w1, *w2;   // [>= C][Kp] each, K = (tap, channel), Kp = 9 C rounded up to 64
    const int32_t *prm1, *prm2;
    int32_t zp_x, zp_t;      // zero-points of the block input and of the middle tensor
    int32_t lo1, lo2;        // lower clamps of the two convolutions
    int32_t form;            // 0: RQ_PAIR, add RQ_PAIR; 1: RQ_PAIR, add RQ_ANY; 2: RQ_ANY, add RQ_ANY
    AddConst add;
    int32_t pad_;
};
// Counters of a call whose last workgroup sends the tallies, zero before and after: votes and, in the last launch, finished workgroups of
// every sixteenth workgroup, and how many of these parts are complete.  Additions to 64 bytes come through 10 to 15 ns apart, whichever
// workgroups make them.
constexpr uint32_t TALLY_PARTS = 16, SENT_TALLIES = 256, SENT_COPIES = 4096;   // most tallies, and copies of a net with blocks, of such a call
struct TallyParts {
    struct { uint32_t finished, unused[31], votes[SENT_TALLIES]; } part[TALLY_PARTS];
    uint32_t complete;
};
struct NarrowParams {
    const int8_t *in;        // [B][S][S][C], or the NHWC4 image [B][S][S][4] (stem != 0)
    int8_t *out;             // [B][S][S][C]; tail != 0: [B][S/2][S/2][2C]; unused with a head
    int32_t B;
    // first layer, 3x3 into 16 channels; with fused_noise the kernel draws its own input
    int32_t stem, fused_noise, zp_in, lo0, form0;   // form0: as NarrowBlock::form
    const int8_t *w0;
    const int32_t *prm0;
    NoiseSource noise;
    // chain of identity blocks
    int32_t nblocks;
    const NarrowBlock *blocks;
    NarrowBlock first;       // blocks[0], which a kernel then has without a load of its descriptor
    // tail 1: down-sampling block t = conv3x3/2(x), u = conv3x3(t), r = conv1x1/2(x), y = add(r, u); 2: t alone
    int32_t tail, tform;     // form as above
    const int8_t *tw1, *tw2, *twp;
    const int32_t *tprm;     // [3][4][2C]: t, u, r
    int32_t tzp_x, tzp_t, tlo1, tlo2, tlop;
    AddConst tadd;           // "self" is the projection r
    // head: global average pooling of the last tensor, fully connected layer, votes
    int32_t head, gap_zp_in, gap_zp_out, gap_M0, gap_sh;
    const int8_t *fc_w;
    const int32_t *fc_bias;
    int32_t classes, classes_p;
    int32_t *logits, *argmax;
    uint32_t *counts;        // votes are added here, or each goes to
    uint64_t *votes;         // the host's memory, by its place in the list: class, and `seq` in the high word
    uint32_t seq;
    // with counts: votes go to `parts`, where given, instead; in the last launch of such a call the last workgroup to finish sends the
    // `tallies` sums of these and the counters to `tally_host`, leaves zeros in their place and stores `seq` to `flag`.  0: none
    uint32_t tallies;
    uint32_t *tally_host, *flag;
    TallyParts *parts;
    Slots slots;             // of the votes
};
constexpr uint64_t DIRECT_VOTES = 256;   // most votes of a call that go to the host one by one

// Bottleneck block in one kernel: conv1x1 -> conv3x3 [-> conv1x1 + residual add with the block input
// when tail != 0]; 64 middle channels (bottleneck.hip) or 128 (bottleneck128.hip, tail only).
struct BneckParams {
    const int8_t *in;        // [B][H][W][Cin_p] block input x (also the residual of the tail)
    int8_t *out;             // tail: [B][H][W][Cout_p]; else the 3x3 output [B][H][W][64]
    const int8_t *w1;        // [>= Cmid][Cin_p] rows in MFMA row order
    const int8_t *w2;        // [>= Cmid][9 Cmid], K = (tap, channel)
    const int8_t *w3;        // [>= Cout_p][Cmid] (tail)
    const int32_t *bias1, *m0s1, *chi1, *shm11;   // as in ConvParams, per convolution
    const int32_t *bias2, *m0s2, *chi2, *shm12;
    const int32_t *bias3, *m0s3, *chi3, *shm13;
    // proj != 0 (with tail): the residual is not x but clamp(requant(conv1x1_p(x))), a projection shortcut
    // from 64 input channels computed in the same kernel; its weights [>= Cout_p][64] and constants:
    const int8_t *wp;
    const int32_t *biasp, *m0sp, *chip, *shm1p;
    int32_t proj, lop;       // lop: lower clamp of the projection's int8 result
    // reduce != 0 (identity block of 256 channels): out2 = clamp(requant(conv1x1(out))), [B][H][W][128], computed from the
    // sums in LDS; its weights (fragment-major, ConvParams::wfrag), constants and lower clamp in wp .. lop.  sparse: nothing
    // else needs odd rows or columns of `out`, which are not written.
    int32_t reduce, sparse;
    int8_t *out2;
    const int8_t *zpad;      // 16 readable bytes (source of halo pixels outside the image)
    int32_t Cin_p, Cout_p, H, W, B, tail;
    int32_t zp_t1;           // zero-point of the first convolution's output (padding value of the 3x3)
    int32_t lo1, lo2, lo3;   // lower clamps of the three int8 results
    int32_t add_mul_self, add_mul_res, add_c0, add_k, add_sh, add_lo;   // as in ConvParams
    int32_t rq, add_rq;      // Rq class (conv_device.h) of every convolution of the block together; that of the add
};

// Closing 1x1 convolution + residual add of one bottleneck block and the opening 1x1 convolution of the next
// in one kernel (expand_reduce.hip): y = add(requant(W3 t2), x), t1n = requant(W1n y); 128 -> 512 -> 128 channels.
struct XrParams {
    const int8_t *t2;        // [npix][128] input of the expanding convolution
    const int8_t *x;         // [npix][512] residual
    int8_t *y;               // [npix][512] the sum (the next block's input and residual)
    int8_t *t1n;             // [npix][128] output of the reducing convolution
    const int8_t *a1, *a2;   // fragment-major weight copies (ConvParams::wfrag) of the two convolutions
    // in2 != null: the residual is not x but clamp(requant(Wp in2)), a projection from 256 channels computed in the kernel
    const int8_t *in2;       // [npix][256]
    const int8_t *ap;        // fragment-major copy of the projection weights
    const int32_t *biasp, *m0sp, *chip, *shm1p;   // [512]
    int32_t lop;             // lower clamp of the projection's int8 result
    int32_t Hin, Win, Ho, Wo, pstride;   // the projection reads pixel (pstride y, pstride x) of its Hin x Win input for output pixel (y, x)
    const int32_t *bias1, *m0s1, *chi1, *shm11;   // as in ConvParams, expanding convolution [512]
    const int32_t *bias2, *m0s2, *chi2, *shm12;   // reducing convolution [128]
    int32_t lo1, lo2;        // lower clamps of the two convolutions' int8 results
    int32_t add_mul_self, add_mul_res, add_c0, add_k, add_sh, add_lo;   // as in ConvParams
    int32_t rq, add_rq;      // Rq class of all convolutions together (at least tie-free); that of the add
    int32_t npix;
    int32_t n2;              // output channels of the reducing convolution: 128, or 256 (stored residual only)
    int32_t k1;              // input channels of the expanding convolution: 128 (512 block channels) or 256 (1024; stored residual, n2 = 256)
};

struct AddParams {
    const int8_t *a, *b;
    int8_t *out;
    int32_t za, zb, zo, Ma, Mb, sh, relu;
    int64_t n16;             // number of 16-byte groups
};

struct PoolParams {
    const int8_t *in;
    int8_t *out;
    int32_t H, W, Cp, Ho, Wo, k, stride, pad;
    int32_t B;
};

struct GapParams {
    const int8_t *in;        // [B][HW][Cp]
    int8_t *out;             // [B][Cp]
    int32_t HW, Cp, zp_in, zp_out, M0, sh, B;
};

struct FcParams {
    const int8_t *in;        // [B][Kp]
    const int8_t *w;         // [Kp / 16][classes_p][16]: 16-byte K chunks, class-contiguous
    const int32_t *bias;     // [classes], bias - z_in * sum(w)
    int32_t Kp, classes, classes_p, B;   // classes_p: classes rounded up to a multiple of 4
    int32_t *logits;         // [B][classes] or null
    int32_t *argmax;         // [B] or null
    uint32_t *counts;        // [phases][pairs][classes] (accumulated) or null
    Slots slots;             // of the votes
};

struct NoiseParams {
    const uint8_t *x;        // [C][H][W] clean image ([images][C][H][W] in batch mode)
    const DeviceNoiseTable *table;   // the table (batch mode: table 0 of the array indexed by table_slot)
    int8_t *out;             // [B][H][W][4]
    int32_t C, H, W;
    uint32_t key0, key1, image, phase, sample_begin, count;
    // batch mode (items != null): copy s of the chunk is slot slot_begin + s; item i owns slots
    // [i * n_per_item, (i + 1) * n_per_item) and sample index = slot - i * n_per_item; the
    // launch covers items item_first .. item_first + item_count - 1 (one grid row each)
    const NoiseItem *items;
    uint32_t n_per_item, item_first, item_count;
    uint64_t slot_begin;
};

// Stored-noise generator: count tensors of d draws each, int16.
struct NoiseBankParams {
    const uint32_t *thi, *tlo;   // [s.reach] high / low words of the ascending thresholds below the centre (device)
    const uint32_t *guide;       // guide table (device)
    uint32_t guide_words;
    NoiseSampler s;
    int16_t *out;                // [count][d]
    uint32_t d;                  // draws per tensor, a multiple of 4
    uint32_t key0, key1, bank, first, count;
};

// ---- floating-point comparison systems (float_path.hip) ------------------------------------
// Continuous Gaussian noise: copy s, logical element p = (c*H + y)*W + x gets x[p] + sigma z with z the
// standard-normal draw of counter (p >> 2, sample_begin + s, image, 8 + phase), element p & 3.
struct FloatNoiseParams {
    const uint8_t *x;        // [C][H][W] clean image
    void *out;               // quant: int8 [B][H][W][4], clamp(round(v), 0, 255) - 128; else float [B][H][W][4], v - center
    int32_t C, H, W;
    uint32_t key0, key1, image, phase, sample_begin, count;
    float sigma, center;
    int32_t quant;
};

// fp32 convolution as an implicit GEMM on the fp32 MFMA, NHWC activations:
//   t = act((bias + sum over in-bounds taps of in * w) * scale);  out = res ? act_add(ma * t + mb * res) : t
struct FConvParams {
    const float *in;         // [B][H][W][Cin_p]
    float *out;              // [B][Ho][Wo][Cout_p]
    const float *res;        // [B][Ho][Wo][Cout_p] or null
    const uint16_t *w;       // bfloat16 [Kq / 8][Cout_pp][32]: step s holds k = 32 s .. + 31 of K = (tap, channel); rows in MFMA row order per 32 channels
    const float *zeros;      // 16 bytes of zeros: source of out-of-image taps
    const float *bias, *scale;   // [Cout_pp], by channel
    const int32_t *ktab;     // [Kq]: dy << 24 | dx << 16 | channel offset of the quad; -1 = padding quad
    int32_t H, W, Cin_p, Ho, Wo, Cout_p, Cout_pp, k, stride, pad, Kq;   // k x k taps; Kq quads of K, a multiple of 8
    int32_t npix;            // B * Ho * Wo
    int32_t relu, add_relu;
    float ma, mb;
    // in2 != null: the residual is not stored but another 1x1 convolution's result, computed in the kernel (this one is 1x1 as well)
    const float *in2;        // [B][H2][W2][Cin2_p]
    const uint16_t *w2;
    const float *bias2, *scale2;
    int32_t H2, W2, Cin2_p, stride2, relu2;
};
struct FAddParams { const float *a, *b; float *out; float ma, mb; int32_t relu; int64_t n4; };
struct FPoolParams { const float *in; float *out; int32_t H, W, Cp, Ho, Wo, k, stride, pad, B; };
struct FGapParams { const float *in; float *out; int32_t HW, Cp, B; float scale; };
struct FVoteParams { const float *logits; int32_t classes, stride, B; int32_t *argmax; uint32_t *counts; };
hipError_t launch_float_noise(const FloatNoiseParams &p, hipStream_t st);
hipError_t launch_fconv(const FConvParams &p, hipStream_t st);
bool fconv_pair_supported(const FConvParams &p, const FConvParams &q);   // q's result as p's residual in one kernel ...
bool fconv_pair_wanted(const FConvParams &p);                            // ... for this number of pixels
bool fexpand_supported(const FConvParams &p, const FConvParams &q);      // p with its add, and q that reads the sum, in one kernel ...
bool fexpand_wanted(const FConvParams &p, const FConvParams &q);         // ... for this number of pixels
hipError_t launch_fexpand(const FConvParams &p, const FConvParams &q, hipStream_t st);
bool fstem_pool_supported(const FConvParams &p, const FPoolParams &q);   // p and the pooling q of its result in one kernel
hipError_t launch_fstem_pool(const FConvParams &p, const FPoolParams &q, hipStream_t st);   // p.out and q.in are not used
int fconv_tile_m(int cout_p);   // channels per output tile chosen for a layer (Cout_pp is a multiple of it)
hipError_t launch_fadd(const FAddParams &p, hipStream_t st);
hipError_t launch_fmaxpool(const FPoolParams &p, hipStream_t st);
hipError_t launch_fgap(const FGapParams &p, hipStream_t st);
hipError_t launch_fvote(const FVoteParams &p, hipStream_t st);

// Name of the kernel instance the last launcher call on this thread enqueued (template arguments
// included, as a profiler prints them); the per-kernel timing report is keyed by it.
void set_kernel_name(const char *name);
const char *last_kernel_name();

// Kernel launchers (kernels.hip / conv_igemm.hip).  All asynchronous on `st`.
hipError_t launch_noise_bank(const NoiseBankParams &p, hipStream_t st);
hipError_t launch_noise(const NoiseParams &p, hipStream_t st);
hipError_t launch_conv(const ConvParams &p, hipStream_t st);
bool conv_patch_supported(const ConvParams &p);
hipError_t launch_conv_patch(const ConvParams &p, hipStream_t st);   // deep 3x3 layers, pixel rows staged once per channel slice (conv_patch.hip)
hipError_t launch_conv_deep(const ConvParams &p, hipStream_t st);   // 256 x 256 tiles, 128 x 128 per wave (conv_deep.hip)
hipError_t launch_stem_pool(const StemPoolParams &p, hipStream_t st);
bool stem_pool_supported(int k, int stride, int pad, int cout_p, int H, int W, int fast_requant, int pool_k,
                         int pool_stride, int pool_pad);
hipError_t launch_stem16(const Stem16Params &p, hipStream_t st);
bool stem16_supported(int k, int stride, int pad, int cout_p, int H, int W, int fast_requant);
hipError_t launch_narrow(const NarrowParams &p, int channels, hipStream_t st);   // narrow_net.hip
bool narrow_chain_wanted(int copies);   // all three stages in one launch
bool narrow_short(const NarrowParams &p);   // a whole net of two convolutions, from the image to the votes
hipError_t launch_narrow_chain(const NarrowParams &s16, const NarrowParams &s32, const NarrowParams &s64, hipStream_t st);
bool basic_block_supported(int channels, int size);
hipError_t launch_bottleneck(const BneckParams &p, hipStream_t st);
hipError_t launch_bottleneck_stream(const BneckParams &p, int ntiles, hipStream_t st);   // blocks of 256 channels in launches of many tiles (bottleneck_stream.hip)
bool bottleneck_supported(int cin_p, int cmid_p, int cout_p, int tail);
hipError_t launch_bottleneck128(const BneckParams &p, hipStream_t st);
bool expand_reduce_supported(const ConvParams &expand, const ConvParams &reduce);
void expand_reduce_params(const ConvParams &expand, const ConvParams &reduce, const int8_t *a, const int8_t *b, int8_t *y,
                          int8_t *t1n, int32_t copies, XrParams &xp);
hipError_t launch_expand_reduce(const XrParams &p, hipStream_t st);   // expand_reduce.hip   // 128 middle channels, identity blocks (bottleneck128.hip)
bool bottleneck128_supported(int cin_p, int cmid_p, int cout_p);
bool trans_block_supported(int cout, int size_out);
hipError_t launch_add(const AddParams &p, hipStream_t st);
hipError_t launch_maxpool(const PoolParams &p, hipStream_t st);
hipError_t launch_gap(const GapParams &p, hipStream_t st);
hipError_t launch_fc(const FcParams &p, hipStream_t st);
// flag != null (at most PUBLISH_WATCHED tallies): `seq` is stored there when the tallies are on the host
constexpr size_t PUBLISH_WATCHED = 2560;
hipError_t launch_publish(uint32_t *counts, uint32_t *host, size_t n, uint32_t *flag, uint32_t seq, hipStream_t st);
hipError_t launch_fill_u32(uint32_t *p, uint32_t value, size_t n, hipStream_t st);
// Tile geometry of the convolution kernel chosen for (Cout_p): rows per M tile.
int conv_tile_m(int cout_p);
// K bytes per step chosen for a layer (see conv_igemm.hip).
int conv_k_step(int kreal, int cin_p, int cout_p, int fast_requant);

}  // namespace isr

#endif
