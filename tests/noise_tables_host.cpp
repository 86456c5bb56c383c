// The sampler's tables of every sigma, read on the host the way the kernels read them (noise_device.h) at both sides of
// every threshold and of every bucket edge, against the thresholds themselves; and what building them costs beside
// building the thresholds.  Built and run by tests/test_noise_tables_host.py.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <vector>

#include "isr_internal.h"

using namespace isr;

static uint32_t bits_of(float f) { uint32_t b; std::memcpy(&b, &f, 4); return b; }

// the draw of (u, ulo) clamped to +-reach
static int looked_up(const uint32_t *guide, const uint32_t *hi, const uint32_t *lo, const NoiseSampler &s, uint32_t u, uint32_t ulo) {
    const bool right = (int32_t)u < 0;
    const uint32_t x = right ? ~u : u;
    const float f = std::min(std::max((float)x, s.lo), s.hi);
    const uint32_t bits = bits_of(f), e = guide[((bits >> s.shift) & s.mask) >> 2], t = e - (bits << s.key_shift);
    int a;
    if (t > NOISE_DRAW_MASK) {
        const int m = (int)(e & NOISE_DRAW_MASK) + ((int32_t)t >> 31);
        return right ? m : -m;
    }
    uint32_t from = (float)x <= s.lo ? 0 : s.reach - (e & NOISE_DRAW_MASK), to = s.reach - (e & NOISE_DRAW_MASK) + 1;
    if (to > s.reach) to = s.reach;
    a = (int)(std::lower_bound(hi + from, hi + to, x) - hi);
    if (right) ulo = ~ulo;
    while (a < (int)s.reach && hi[a] == x && (right ? lo[a] < ulo : lo[a] <= ulo)) ++a;
    const int d = a - (int)s.reach;
    return right ? -d : d;
}

// by the thresholds alone
static int drawn(const std::vector<uint64_t> &T, int R, uint32_t u, uint32_t ulo) {
    const uint64_t w = (uint64_t)u << 32 | ulo;
    return (int)(std::upper_bound(T.begin(), T.end(), w) - T.begin()) - R;
}

template <class F>
static double microseconds(F f) {
    double best = 1e9;
    for (int r = 0; r < 9; ++r) {
        const auto t = std::chrono::steady_clock::now();
        for (int i = 0; i < 20; ++i) f();
        best = std::min(best, std::chrono::duration<double>(std::chrono::steady_clock::now() - t).count() / 20 * 1e6);
    }
    return best;
}

int main() {
    static DeviceNoiseTable t;
    std::vector<uint32_t> words;
    long checked = 0;
    for (uint32_t sigma = 1; sigma <= 1024; ++sigma) {
        uint32_t n = 0, R = 0;
        const auto tab = cached_noise_table(sigma);
        if (!tab || !build_device_table(sigma, t) || !build_bank_table(sigma, words, n, R)) { std::printf("no table: sigma %u\n", sigma); return 1; }
        NoiseBankParams bank{};
        set_bank_table(bank, words.data(), words.size(), R);
        auto check = [&](uint32_t x) {
            for (uint32_t u : {x, ~x})
                for (uint32_t ulo : {0u, ~0u}) {
                    const int want = drawn(tab->T, (int)tab->R, u, ulo);
                    const int stored = looked_up(bank.guide, bank.thi, bank.tlo, bank.s, u, ulo);
                    const int pixel = looked_up(t.guide, t.hi, t.lo, t.s, u, ulo);
                    const int reach = (int)t.s.reach;
                    ++checked;
                    if (stored != want || pixel != std::max(-reach, std::min(reach, want))) {
                        std::printf("sigma %u, word %08x %08x: %d, stored %d, pixel %d\n", sigma, u, ulo, want, stored, pixel);
                        return false;
                    }
                }
            return true;
        };
        for (uint32_t j = 0; j < tab->R; ++j)
            for (int d = -1; d <= 1; ++d)
                if (!check((uint32_t)std::min<int64_t>(std::max<int64_t>((int64_t)(tab->T[j] >> 32) + d, 0), 0x7FFFFFFF))) return 1;
        for (uint32_t b = 127u << 11; b < 158u << 11; b += sigma % 16 ? 13 : 1) {   // edges of the finest buckets and of coarser ones
            float f;
            const uint32_t bits = b << 12;
            std::memcpy(&f, &bits, 4);
            const uint32_t x = (uint32_t)f;
            if (!check(x) || !check(x - 1)) return 1;
        }
        if (!check(0) || !check(1) || !check(0x7FFFFFFF)) return 1;
    }
    std::printf("checked %ld\n", checked);
    for (uint32_t sigma : {256u, 1000u}) {
        std::vector<uint64_t> T;
        uint32_t n, R;
        const double thresholds = microseconds([&] { build_noise_table(sigma, T, R); });
        const double pixel = microseconds([&] { build_device_table(sigma, t); });
        const double stored = microseconds([&] { std::vector<uint32_t> w; build_bank_table(sigma, w, n, R); });
        std::printf("sigma %u pixel %.3f stored %.3f\n", sigma, pixel / thresholds, stored / thresholds);
    }
    return 0;
}
