// Device helpers shared by the convolution kernels: LDS swizzle, requantisation,
// clamp and byte packing.
#ifndef ISR_CONV_DEVICE_H
#define ISR_CONV_DEVICE_H

#include <type_traits>

#include "isr_internal.h"

namespace isr {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v4acc __attribute__((ext_vector_type(4)));   // result of a 16x16 MFMA
typedef int v16i __attribute__((ext_vector_type(16)));

// 16-byte chunk swizzle inside an LDS row of CPR chunks (64 or 128 bytes): spreads equal chunk indices of
// neighbouring rows over different banks for the 128-bit fragment reads.  The LDS serves such a read 16
// consecutive lanes at a time from 64 banks of 4 bytes, so 16 consecutive rows reading one logical chunk must
// cover 256 bytes exactly once: the rows that share a 256-byte line (4 rows of 64 bytes, 2 of 128) keep the
// chunk, each next group of rows moves it on by one (measured: as fast as contiguous reads; XOR with the
// low row bits instead costs 13-14 % of the read rate).
template <int CPR>
__device__ __forceinline__ int swz(int row) { return CPR == 4 ? ((row >> 2) & 3) : ((row >> 1) & 7); }

// RHA(acc * M0, 31 + shift) on magnitude and sign, 32x32->64 multiply-add:
//   |acc| * (M0 << 1) + 2^(31+shift) = 2 * (|acc| * M0 + 2^(30+shift)),
// so the rounded quotient is the high word shifted right by `shift`.
__device__ __forceinline__ int requant(int acc, uint32_t m0x2, uint32_t rnd_lo, uint32_t rnd_hi, uint32_t sh) {
    uint32_t mag = (uint32_t)(acc < 0 ? -acc : acc);
    uint64_t prod = (uint64_t)mag * (uint64_t)m0x2 + (((uint64_t)rnd_hi << 32) | rnd_lo);
    int r = (int)((uint32_t)(prod >> 32) >> sh);
    return acc < 0 ? -r : r;
}

// Same result from one signed 32x32+64 multiply-add when 2 <= shift <= 22:
//   z_out + RHA(v, s) = floor((v + 2^(s-1) - [v<0] + z_out 2^s) / 2^s),  v = acc M0, s = 31 + shift.
// 2^(s-1) + z_out 2^s is a multiple of 2^32 (chi holds its high word), and
// subtracting [v<0] turns the 64-bit addend into (chi + m : m) with m = acc >> 31.
__device__ __forceinline__ int requant_fast(int acc, int m0, int chi, int shm1) {
    int m = acc >> 31;
    long addend = (long)(((unsigned long)(uint32_t)(chi + m) << 32) | (uint32_t)m);
    long w = (long)acc * (long)m0 + addend;
    return (int)(w >> 32) >> shm1;
}

// The same again for a layer whose products acc * M0 are never a negative exact half above the clamp
// (ConvParams::tie_free): with the low word of the rounding term gone only the high
// word of the product is needed.
__device__ __forceinline__ int requant_tie_free(int acc, int m0, int chi, int shm1) {
    return (__mulhi(acc, m0) + chi) >> shm1;
}

template <bool TIE_FREE>
__device__ __forceinline__ int requant_q(int acc, int m0, int chi, int shm1) {
    if constexpr (TIE_FREE) return requant_tie_free(acc, m0, chi, shm1);
    else return requant_fast(acc, m0, chi, shm1);
}

// clamp(v, lo, hi) for lo <= hi in one instruction
__device__ __forceinline__ int clamp3(int v, int lo, int hi) {
    int r;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(v), "v"(lo), "v"(hi));
    return r;
}

// Residual add on the int8 result q of the convolution and the int8 residual r8 (second
// requantisation): v = q Ms + r8 Mr + c0, out = clamp((v + k + (v >> 31)) >> sh, lo, 127)
// with k = 2^(sh-1) + z_out 2^sh; 24-bit multiplies: |q|, |r8| <= 2^7, |multipliers| < 2^23.
template <bool TIE_FREE>
__device__ __forceinline__ int fused_add(int q, int r8, const ConvParams &p) {
    if constexpr (TIE_FREE) {
        const int v = __mul24(q, p.add_mul_self) + (p.add_c0 + p.add_k) + __mul24(r8, p.add_mul_res);
        return clamp3(v >> p.add_sh, p.add_lo, 127);
    }
    const int v = __mul24(q, p.add_mul_self) + p.add_c0 + __mul24(r8, p.add_mul_res);
    return clamp3((v + p.add_k + (v >> 31)) >> p.add_sh, p.add_lo, 127);
}

// low bytes of four registers -> one dword (3 byte-permutes)
__device__ __forceinline__ uint32_t pack4(int a, int b, int c, int d) {
    uint32_t lo = __builtin_amdgcn_perm((uint32_t)b, (uint32_t)a, 0x0c0c0400u);
    uint32_t hi = __builtin_amdgcn_perm((uint32_t)d, (uint32_t)c, 0x0c0c0400u);
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}

// How a layer's requantisation and its fused residual add are computed; chosen per layer when the model is loaded.
//   RQ_ANY       any layer of the single-multiply form
//   RQ_TIE_FREE  no accumulator value meets an exact half whose rounding would show (ConvParams::tie_free): rectified layers, and
//                nearly all others
//   RQ_TOP       tie-free, lower clamp -128, and every intermediate fits (plan.cpp): the int8 result is kept in the TOP
//                byte of a word, where int32 saturation is its clamp.  w = mulhi(acc, M0) fits 24 bits, so
//                  sat32(w * 2^(24 - shm1) + (2^23 + z_out 2^24))
//                is floor((w + chi) / 2^shm1), clamped to [-128, 127], times 2^24 plus a fraction: add, shift and clamp
//                become one v_mad_i32_i24 with the clamp bit, and the packing is two byte permutes and an or.  Issue
//                cycles of a wave per output, from the measured rates (add, shift, and, or 2.5 - 2.8; multiplies, clamp,
//                permute 4.3 - 4.5): 12 instead of 17, with a residual add 29 instead of 37.  ResNet-50, 668 copies:
//                identity block at 56 x 56 409 -> 349 us, expand + reduce at 28 x 28 160 -> 138, at 14 x 14 120 -> 108.
//   RQ_TOP_TIES  the same with ties (a 64-bit multiply-add instead of the multiply)
//   RQ_PAIR      tie-free, lower clamp -128, ONE shift for all channels of the layer (networks quantised per tensor have one; the
//                multipliers may differ).  w = high word of acc * M0 + chi 2^32 is one v_mad_i64_i32, and v_ashr_pk_i8_i32
//                shifts, saturates and packs two of them: 9.0 issue cycles an output against 12.3 of RQ_TOP, 27 against 31 with an
//                add (measured, a wave instruction: v_mad_i64_i32, v_mul_hi, v_mad_i32_i24, 24-bit multiplies, v_add3, v_perm 4.65,
//                v_ashr_pk_i8_i32 8.6, v_or 2.55).  No bound on the range of w, which int32 holds.  Certification of ResNet-50, n = 10 000: 65.4 -> 63.7 ms, of the
//                110-layer net, n = 100 000: 26.71 -> 25.68 ms, ResNet-20 5.24 -> 5.12.
// An add is RQ_ANY, RQ_TIE_FREE, RQ_TOP, RQ_TOP_WIDE (two signed operands, whose sum may leave int32 and saturates) or RQ_PAIR.
// The forms of several convolutions combine with & (Rq).
// v_mad_i32_i24 with the clamp bit: sat32(a * b + c), a and b in 24 bits (no builtin reaches the clamp bit)
__device__ __forceinline__ int mad24_sat(int a, int b, int c) {
    int r;
    asm("v_mad_i32_i24 %0, %1, %2, %3 clamp" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// The per-channel constants as the kernels stage them: in the top form `chi` becomes the addend (the same for every
// channel of a layer, padding channels included) and `shm1` the multiplier.
template <int RQ>
__device__ __forceinline__ int rq_chi(int chi, int shm1) { return rq_is_top(RQ) ? chi << (24 - shm1) : chi; }
template <int RQ>
__device__ __forceinline__ int rq_sh(int shm1) { return rq_is_top(RQ) ? 1 << (24 - shm1) : shm1; }
// index of channel i's addend
template <int RQ>
__device__ __forceinline__ constexpr int rq_chi_at(int i) { return rq_is_top(RQ) || RQ == RQ_PAIR ? 0 : i; }
// four channels' addends (one value for a whole layer where the form has one)
template <int RQ>
__device__ __forceinline__ v4i rq_chi4(const int *c) {
    if constexpr (rq_chi_at<RQ>(1) == 0) return v4i{c[0], c[0], c[0], c[0]};
    else return *(const v4i *)c;
}

// RQ_PAIR: a layer's addend and shift, in scalar registers; the other forms have theirs per channel.
struct RqLayer {
    long add;   // chi 2^32
    int sh;
};
// from the staged constants of any real channel
template <int RQ>
__device__ __forceinline__ RqLayer rq_layer(int chi, int sh) {
    if constexpr (RQ == RQ_PAIR) {
        long add = (long)((unsigned long)(uint32_t)__builtin_amdgcn_readfirstlane(chi) << 32);
        asm("" : "+s"(add));   // a low word known to be zero would make a multiply and an add of the multiply-add
        return {add, __builtin_amdgcn_readfirstlane(sh)};
    } else {
        return {0, 0};
    }
}

// requantise + clamp to [lo, 127]: the value, in the top form a word with the value in its top byte, in the pair form one
// that rq_pack shifts and clamps
template <int RQ>
__device__ __forceinline__ int rq_conv(int acc, int m0, int chi, int sh, int lo, const RqLayer &layer) {
    if constexpr (RQ == RQ_PAIR) {
        return (int)(((long)acc * (long)m0 + layer.add) >> 32);
    } else if constexpr (RQ == RQ_TOP) {
        return mad24_sat(__mulhi(acc, m0), sh, chi);
    } else if constexpr (RQ == RQ_TOP_TIES) {
        const long w = (long)acc * (long)m0 + (long)(acc >> 31);   // v - [v < 0], as requant_fast
        return mad24_sat((int)(w >> 32), sh, chi);
    } else {
        return clamp3(requant_q<RQ == RQ_TIE_FREE>(acc, m0, chi, sh), lo, 127);
    }
}

// sat8(v >> sh) of four words -> one dword.  Each instruction writes one half of the register and keeps the other; a vector
// instruction right behind a write of the upper half must not read it (the wait state at the end).
__device__ __forceinline__ uint32_t pack_shifted(int a, int b, int c, int d, int sh) {
    uint32_t r;
    asm("v_ashr_pk_i8_i32 %0, %1, %2, %5\n\tv_ashr_pk_i8_i32 %0, %3, %4, %5 op_sel:[0,0,0,1]\n\ts_nop 0"
        : "=&v"(r) : "v"(a), "v"(b), "v"(c), "v"(d), "s"(sh));
    return r;
}

// four results of rq_conv -> one dword of int8
template <int RQ>
__device__ __forceinline__ uint32_t rq_pack(int a, int b, int c, int d, const RqLayer &layer) {
    if constexpr (RQ == RQ_PAIR) {
        return pack_shifted(a, b, c, d, layer.sh);
    } else if constexpr (rq_is_top(RQ)) {
        const uint32_t lo = __builtin_amdgcn_perm((uint32_t)b, (uint32_t)a, 0x0c0c0703u);
        const uint32_t hi = __builtin_amdgcn_perm((uint32_t)d, (uint32_t)c, 0x07030c0cu);
        return lo | hi;
    } else {
        return pack4(a, b, c, d);
    }
}
template <int RQ>
__device__ __forceinline__ v4i rq_pack16(const int (&q)[16], const RqLayer &layer) {
    return v4i{(int)rq_pack<RQ>(q[0], q[1], q[2], q[3], layer), (int)rq_pack<RQ>(q[4], q[5], q[6], q[7], layer),
               (int)rq_pack<RQ>(q[8], q[9], q[10], q[11], layer), (int)rq_pack<RQ>(q[12], q[13], q[14], q[15], layer)};
}

// Constants of the residual add.  Top form: everything times 2^(23 - add_sh); the saturating double of the sum has the
// int8 result in the top byte.
template <int RQA, class P>
__host__ __device__ __forceinline__ AddConst add_const(const P &p) {
    if constexpr (RQA == RQ_PAIR) {
        return {p.add_mul_self, p.add_mul_res, p.add_c0 + p.add_k, 0, p.add_sh, 0};
    } else if constexpr (rq_is_top(RQA)) {
        const int s = 23 - p.add_sh;
        return {p.add_mul_self << s, p.add_mul_res << s, (p.add_c0 + p.add_k) << s, 0, 0, 0};
    } else {
        return {p.add_mul_self, p.add_mul_res, p.add_c0, p.add_k, p.add_sh, p.add_lo};
    }
}

// Residual add of the int8 value q and the int8 value r8: the value, or a word as rq_conv<RQA> returns.
// 24-bit multiplies: |q|, |r| <= 2^7, |multipliers| < 2^23.
template <int RQA>
__device__ __forceinline__ int rq_add_value(int q, int r8, const AddConst &a) {
    if constexpr (RQA == RQ_PAIR) {
        return __mul24(q, a.ms) + __mul24(r8, a.mr) + a.c0;
    } else if constexpr (RQA == RQ_TOP) {
        const int v = __mul24(q, a.ms) + __mul24(r8, a.mr) + a.c0;
        return __builtin_elementwise_add_sat(v, v);
    } else if constexpr (RQA == RQ_TOP_WIDE) {
        const int v = mad24_sat(q, a.ms, __mul24(r8, a.mr) + a.c0);
        return __builtin_elementwise_add_sat(v, v);
    } else if constexpr (RQA == RQ_TIE_FREE) {
        const int v = __mul24(q, a.ms) + (a.c0 + a.k) + __mul24(r8, a.mr);
        return clamp3(v >> a.sh, a.lo, 127);
    } else {
        const int v = __mul24(q, a.ms) + a.c0 + __mul24(r8, a.mr);
        return clamp3((v + a.k + (v >> 31)) >> a.sh, a.lo, 127);
    }
}
// Four channels: q as rq_conv<RQ> returns them, the residuals the bytes of rword (the byte selections fold into the
// multiplies); the sums as one dword of int8.
template <int RQ, int RQA>
__device__ __forceinline__ uint32_t rq_add4(int q0, int q1, int q2, int q3, uint32_t rword, const AddConst &a, const RqLayer &layer) {
    static_assert(RQA == RQ_ANY || RQA == RQ_TIE_FREE || (RQA == RQ_PAIR ? RQ == RQ_PAIR : rq_is_top(RQ)), "a form of the add next to one of the convolution");
    int q[4] = {q0, q1, q2, q3}, v[4];
    uint32_t qword = 0;
    if constexpr (RQ == RQ_PAIR) qword = rq_pack<RQ>(q0, q1, q2, q3, layer);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int qj = RQ == RQ_PAIR ? (int)(int8_t)(qword >> (8 * j)) : rq_is_top(RQ) ? q[j] >> 24 : q[j];
        v[j] = rq_add_value<RQA>(qj, (int)(int8_t)(rword >> (8 * j)), a);
    }
    return rq_pack<RQA>(v[0], v[1], v[2], v[3], RqLayer{0, a.sh});
}

// Calls f with the compile-time forms <RQ of the convolutions, RQ of the add> that serve layers of these classes.
template <class F>
void with_rq(int rq, int rqa, F f) {
    using std::integral_constant;
    if (rq & rqa & RQ_PAIR) {
        f(integral_constant<int, RQ_PAIR>{}, integral_constant<int, RQ_PAIR>{});
        return;
    }
    rq &= ~RQ_PAIR;
    rqa &= ~RQ_PAIR;
    if (rq == RQ_TOP && rqa == RQ_TOP) f(integral_constant<int, RQ_TOP>{}, integral_constant<int, RQ_TOP>{});
    else if (rq == RQ_TOP && rqa == RQ_TOP_WIDE) f(integral_constant<int, RQ_TOP>{}, integral_constant<int, RQ_TOP_WIDE>{});
    else if (rq == RQ_TOP) f(integral_constant<int, RQ_TOP>{}, integral_constant<int, RQ_ANY>{});
    else if (rq == RQ_TOP_TIES) f(integral_constant<int, RQ_TOP_TIES>{}, integral_constant<int, RQ_ANY>{});
    else if (rq == RQ_TIE_FREE && rqa != RQ_ANY) f(integral_constant<int, RQ_TIE_FREE>{}, integral_constant<int, RQ_TIE_FREE>{});
    else f(integral_constant<int, RQ_ANY>{}, integral_constant<int, RQ_ANY>{});
}
// the same for a kernel without an add
template <class F>
void with_rq(int rq, F f) {
    using std::integral_constant;
    if (rq & RQ_PAIR) f(integral_constant<int, RQ_PAIR>{});
    else if (rq == RQ_TOP) f(integral_constant<int, RQ_TOP>{});
    else if (rq == RQ_TOP_TIES) f(integral_constant<int, RQ_TOP_TIES>{});
    else if (rq == RQ_TIE_FREE) f(integral_constant<int, RQ_TIE_FREE>{});
    else f(integral_constant<int, RQ_ANY>{});
}

// One channel's requantisation constants as the model holds them, fetched before and stored to LDS in a kernel's form
// after the loads that a workgroup starts with: a store waits for its loads, and the loads behind it start that much later.
struct RqRaw {
    int bias, m0s, chi, shm1;
};
__device__ __forceinline__ RqRaw rq_fetch(const int *bias, const int *m0s, const int *chi, const int *shm1, int c) {
    return {bias[c], m0s[c], chi[c], shm1[c]};
}
template <int RQ, class Prm>
__device__ __forceinline__ void rq_store(Prm &prm, const RqRaw &r, int c) {
    prm[0][c] = r.bias; prm[1][c] = r.m0s; prm[2][c] = rq_chi<RQ>(r.chi, r.shm1); prm[3][c] = rq_sh<RQ>(r.shm1);
}

// 16 bytes per lane from global memory into LDS: lane l of the wave writes bytes
// [16 l, 16 l + 16) after the wave-uniform LDS address `lptr`.
#define ISR_GLOBAL_TO_LDS16(gptr, lptr)                                                             \
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(gptr),        \
                                     (__attribute__((address_space(3))) void *)(lptr), 16, 0, 0)

// Wave-uniform LDS byte address of `p` as a plain integer, and a direct-to-LDS load that takes its destination
// from one: the compiler then cannot tie the load to the array and puts no vmcnt(0) in front of every later
// read of that array (which would serialise refill and compute); the kernel's own waits and barriers order them.
__device__ __forceinline__ uint32_t lds_address(const void *p) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)(uintptr_t)(const __attribute__((address_space(3))) void *)p);
}
#define ISR_GLOBAL_TO_LDS16_AT(gptr, lds_u32)                                                       \
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(gptr),        \
                                     (__attribute__((address_space(3))) void *)(uintptr_t)(lds_u32), 16, 0, 0)

// The compiler does not order LDS reads after loads that write LDS; this wait does.
template <int N>
__device__ __forceinline__ void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
// The workgroup's barrier for tiles in LDS; loads from memory stay in flight.  This wave's LDS operations are complete before it, not
// only issued: others may overwrite behind it what this wave has read, be it with stores or with loads straight into LDS.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

}  // namespace isr

#endif
