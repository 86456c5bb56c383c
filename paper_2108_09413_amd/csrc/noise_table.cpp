// Inverse-CDF threshold table of the discrete Gaussian N_Z(0, sigma^2)
// (Def. 3.3 with location 0), integer arithmetic only, and the compact form
// of it the device sampler reads.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <vector>

#include "isr.h"
#include "isr_internal.h"

namespace isr {

typedef unsigned __int128 u128;

static inline uint64_t mul_q62(uint64_t a, uint64_t b) { return (uint64_t)(((u128)a * b) >> 62); }

// Thresholds T[i] = floor(2^64 * P[delta <= i - R]), i in [0, 2R).
// Unnormalised masses exp(-k^2 / (2 sigma^2)) are carried in Q62 fixed point:
// e1 = exp(-1/D), D = 2 sigma^2, from its alternating power series, then
// mass(k+1) = mass(k) * ratio(k), ratio(k+1) = ratio(k) * e1^2.  Masses are
// truncated by 10 bits so that their total fits 64 bits; R is the last k whose
// truncated mass is non-zero.
bool build_noise_table(uint32_t sigma, std::vector<uint64_t> &T, uint32_t &R) {
    if (sigma < 1 || sigma > 1024) return false;
    const uint64_t one = 1ull << 62;
    const uint64_t D = 2ull * sigma * sigma;
    uint64_t e1 = one, term = one;
    for (uint64_t j = 1; (term /= D * j) != 0; ++j) e1 = (j & 1) ? e1 - term : e1 + term;
    const uint64_t e2 = mul_q62(e1, e1);
    std::vector<uint64_t> mass;   // mass[k] for k >= 0, already truncated
    uint64_t cur = one, ratio = e1;
    while ((cur >> 10) != 0) {
        mass.push_back(cur >> 10);
        cur = mul_q62(cur, ratio);
        ratio = mul_q62(ratio, e2);
    }
    R = (uint32_t)mass.size() - 1;
    u128 total = mass[0];
    for (uint32_t k = 1; k <= R; ++k) total += 2 * (u128)mass[k];
    if (total >> 64) return false;
    T.assign(2 * (size_t)R, 0);
    u128 below = 0;  // sum of masses of all values <= current one
    for (uint32_t i = 0; i < 2 * R; ++i) {
        uint32_t dist = i < R ? R - i : i - R;
        below += mass[dist];
        T[i] = (uint64_t)((below << 64) / total);
    }
    return true;
}

// The table of a sigma is a pure function of sigma: built once per process and shared
// (the certification decision looks its quantile up in it on every call).
std::shared_ptr<const NoiseTable> cached_noise_table(uint32_t sigma) {
    static std::mutex mu;
    static std::map<uint32_t, std::shared_ptr<const NoiseTable>> cache;
    std::lock_guard<std::mutex> lock(mu);
    auto it = cache.find(sigma);
    if (it != cache.end()) return it->second;
    auto t = std::make_shared<NoiseTable>();
    if (!build_noise_table(sigma, t->T, t->R)) return nullptr;
    if (cache.size() >= 64) cache.clear();   // bounds the memory held (at most 147 KB per sigma)
    cache[sigma] = t;
    return t;
}

namespace {

uint32_t float_bits(uint32_t x) {
    const float f = (float)x;   // to nearest, as the device converts
    uint32_t b;
    std::memcpy(&b, &f, 4);
    return b;
}

// Guide tables: `mant` leading mantissa bits and the low `expo` exponent bits make the index; the exponent of the
// largest x is 157 and `first`, that of the lowest buckets, differs from it in those bits only.
struct GuideShape {
    uint32_t mant, expo, first, most;   // most: the largest sigma up to which no bucket holds two thresholds
    size_t words() const { return (size_t)((157u & ((1u << expo) - 1)) + 1) << mant; }
};
// More buckets per octave as sigma grows.  Five exponent bits put x below `lo` at 2^-21 of the draws; tables of the large
// sigmas keep to four (57 KB of LDS at sigma 1024, x below 2^18 in 2^-13 of the draws).  At least 2^7 buckets: the 16 lowest bits
// of a float then hold all below its bucket (bank_guide).
const GuideShape BANK_SHAPES[] = {{7, 5, 137, 169}, {8, 5, 137, 332}, {9, 4, 145, 661}, {10, 4, 145, 1024}};
// Pixels need the thresholds of draws within 255 only: a large sigma has none far out in the tail.
const GuideShape PIXEL_SHAPES[] = {{6, 5, 137, 86}, {7, 4, 144, 169}, {8, 3, 152, 332}, {9, 2, 156, 782}, {10, 0, 157, 1024}};

// By sigma: filling one shape after the other until one takes the thresholds makes a build up to twenty times as long (sigma
// 256: 44 us instead of 8 for the bank's table, 16 instead of 1 for the pixels'; sigma 1000: 138 / 26 and 22 / 1).
template <size_t N>
const GuideShape &shape_of(const GuideShape (&shapes)[N], uint32_t sigma) {
    size_t k = 0;
    while (k + 1 < N && sigma > shapes[k].most) ++k;
    return shapes[k];
}

// The largest float below the lowest buckets' exponent: x below them is clamped to it.  Where there are thresholds down
// there, its guide word holds a threshold of the same mantissa, and the draw is looked up.
float floor_of(const GuideShape &g) { return std::nextafter(std::ldexp(1.0f, (int)g.first - 127), 0.0f); }
bool has_below(const GuideShape &g, const uint64_t *T, uint32_t reach) {
    return reach && float_bits((uint32_t)(T[0] >> 32)) < g.first << 23;
}

NoiseSampler sampler_of(const GuideShape &g, uint32_t reach, bool below) {
    NoiseSampler s;
    s.shift = 21 - g.mant;
    s.mask = ((1u << (g.mant + g.expo)) - 1) << 2;
    s.key_shift = 8 + g.mant;
    s.reach = reach;
    s.lo = below ? floor_of(g) : std::ldexp(1.0f, (int)g.first - 127);
    s.hi = std::nextafter(std::ldexp(1.0f, 31), 0.0f);
    return s;
}

// From threshold to threshold, into words that hold zeros; false: two thresholds in one bucket.
bool fill_guide(const GuideShape &g, const uint64_t *T, uint32_t reach, uint32_t *guide) {
    const uint32_t rest = 23 - g.mant, index_mask = (1u << (g.mant + g.expo)) - 1, ones = (1u << rest) - 1, end = 158u << g.mant;
    auto put = [&](uint32_t from, uint32_t to, uint32_t thr, uint32_t count) {   // buckets [from, to): consecutive words
        uint32_t *word = guide + (from & index_mask);
        const uint32_t key = thr << (8 + g.mant) | (reach - count);
#pragma clang loop vectorize(disable) unroll(disable)   // most runs are a bucket or two
        for (uint32_t b = from; b < to; ++b) *word++ = b << 31 | key;
    };
    uint32_t j = 0, next = g.first << g.mant;
    while (j < reach && float_bits((uint32_t)(T[j] >> 32)) < g.first << 23) ++j;
    if (j) {   // the bucket of floor_of
        if (((next - 1) & index_mask) >= g.words()) return false;
        put(next - 1, next, ones, j - 1);
    }
    for (; j < reach; ++j) {
        const uint32_t bits = float_bits((uint32_t)(T[j] >> 32)), b = bits >> rest;
        if (b < next || b >= end) return false;
        put(next, b, ones, j);
        put(b, b + 1, bits & ones, j);
        next = b + 1;
    }
    put(next, end, ones, reach);
    return true;
}

}  // namespace

// Device form.  Pixels lie in [0, 255], so after saturation only
// clamp(delta, -255, 255) matters: keep the thresholds between -255 and 255.
bool build_device_table(uint32_t sigma, DeviceNoiseTable &out) {
    const auto tab = cached_noise_table(sigma);
    if (!tab) return false;
    const uint32_t reach = tab->R < 255 ? tab->R : 255;
    const uint64_t *T = tab->T.data() + (tab->R - reach);
    std::memset(&out, 0, sizeof(out));
    for (uint32_t j = 0; j < reach; ++j) { out.hi[j] = (uint32_t)(T[j] >> 32); out.lo[j] = (uint32_t)T[j]; }
    const GuideShape &g = shape_of(PIXEL_SHAPES, sigma);
    if (g.words() > NOISE_GUIDE_MAX || !fill_guide(g, T, reach, out.guide)) return false;
    out.s = sampler_of(g, reach, has_below(g, T, reach));
    return true;
}

bool build_bank_table(uint32_t sigma, std::vector<uint32_t> &words, uint32_t &n_out, uint32_t &R_out) {
    const auto tab = cached_noise_table(sigma);
    if (!tab) return false;
    const uint64_t *T = tab->T.data();
    const size_t R = tab->R;
    const GuideShape &g = shape_of(BANK_SHAPES, sigma);
    words.assign(2 * R + g.words(), 0);
    if (!fill_guide(g, T, (uint32_t)R, words.data())) return false;
    uint32_t *hi = words.data() + g.words(), *lo = hi + R;
    for (size_t j = 0; j < R; ++j) { hi[j] = (uint32_t)(T[j] >> 32); lo[j] = (uint32_t)T[j]; }
    n_out = R_out = (uint32_t)R;
    return true;
}

void bank_guide(std::vector<uint32_t> &words, uint32_t R) {
    const size_t n = words.size() - 2 * (size_t)R;
    for (const GuideShape &g : BANK_SHAPES)
        if (g.words() == n) {
            const uint32_t rest = 23 - g.mant, ones = (1u << rest) - 1, key_shift = 8 + g.mant;
            for (uint32_t i = 0; i < n; ++i)   // a word holds one of its index bits: the others are where it stands
                words[i] = (words[i] & NOISE_DRAW_MASK) << 16 | ((i << rest | (words[i] >> key_shift & ones)) & 0xFFFF);
        }
}

void set_bank_table(NoiseBankParams &p, const uint32_t *dev, size_t words, uint32_t R) {
    p.guide = dev;
    p.guide_words = (uint32_t)(words - 2 * (size_t)R);
    p.thi = dev + p.guide_words;
    p.tlo = p.thi + R;
    p.s = {};
    for (const GuideShape &g : BANK_SHAPES)
        if (g.words() == p.guide_words) p.s = sampler_of(g, R, true);   // the lowest thresholds are below all buckets
}

}  // namespace isr

extern "C" int isr_noise_table(uint32_t sigma, uint64_t *T_host, size_t cap, uint32_t *R_out) {
    if (!R_out || (cap && !T_host)) return ISR_ERR_ARG;
    const auto tab = isr::cached_noise_table(sigma);
    if (!tab) return ISR_ERR_ARG;
    *R_out = tab->R;
    for (size_t i = 0; i < cap && i < tab->T.size(); ++i) T_host[i] = tab->T[i];
    return ISR_OK;
}

// Inverse cdf of the discrete law by lookup in the same table (Thm 3.2, proof steps 2 and 3).
extern "C" int isr_discrete_quantile(uint32_t sigma, double p_lower, int32_t *t_out, uint64_t *radius_sq_out) {
    if (sigma < 1 || sigma > 1024 || !(p_lower >= 0.0 && p_lower <= 1.0)) return ISR_ERR_ARG;
    const auto tab = isr::cached_noise_table(sigma);
    if (!tab) return ISR_ERR_ARG;
    // floor(2^64 p): exact for a double below 1 (53 significant bits, scaled by a power of two)
    const uint64_t u = p_lower >= 1.0 ? ~0ull : (uint64_t)std::ldexp(p_lower, 64);
    // thresholds ascend: the number of entries <= u by binary search
    const int64_t below = std::upper_bound(tab->T.begin(), tab->T.end(), u) - tab->T.begin();
    const int64_t t = -(int64_t)tab->R - 1 + below;
    if (t_out) *t_out = (int32_t)t;
    if (radius_sq_out) *radius_sq_out = t > 0 ? (uint64_t)(t * t) : 0;
    return ISR_OK;
}

