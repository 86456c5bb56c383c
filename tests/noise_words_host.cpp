// The stored-noise generator's guide words in the form its kernel reads (bank_guide), looked up as it does -- one subtraction, and
// zeros below it where the draw is open, which the search from the word's upper half then decides -- around every threshold and at
// the first and last values of buckets, against the thresholds themselves.  Built and run by tests/test_noise_words_host.py.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <vector>

#include "isr_internal.h"

using namespace isr;

static uint32_t bits_of(float f) { uint32_t b; std::memcpy(&b, &f, 4); return b; }

// the draw of the high word u where it decides; false: open
static bool looked_up(const std::vector<uint32_t> &guide, uint32_t words, const NoiseSampler &s, uint32_t u, int &draw, uint32_t &base) {
    const int right = (int32_t)u >> 31;
    const float f = std::min(std::max((float)(u ^ (uint32_t)right), s.lo), s.hi);
    const uint32_t at = ((bits_of(f) >> s.shift) & s.mask) >> 2;
    if (at >= words) { std::printf("word %u outside the table\n", at); std::exit(1); }
    const uint32_t t = guide[at] - (bits_of(f) & 0xFFFF);
    const int m = (int16_t)(t >> 16);
    draw = right - (m ^ right);
    base = s.reach - (guide[at] >> 16);
    return (uint16_t)t != 0;
}

// of an open one: the steps of noise_draw_slow (noise_device.h), with the low word given
static int searched(const uint32_t *thi, const uint32_t *tlo, const NoiseSampler &s, uint32_t u, uint32_t ulo, uint32_t base) {
    const bool right = (int32_t)u < 0;
    const uint32_t x = right ? ~u : u, y = right ? ~ulo : ulo;
    uint32_t a = (float)x <= s.lo ? 0 : base, e = std::min(base + 1, s.reach);
    while (a < e) {
        const uint32_t mid = (a + e) >> 1;
        if (thi[mid] < x) a = mid + 1; else e = mid;
    }
    while (a < s.reach && thi[a] == x && (right ? tlo[a] < y : tlo[a] <= y)) ++a;
    const int d = (int)a - (int)s.reach;
    return right ? -d : d;
}

int main() {
    std::vector<uint32_t> words;
    long checked = 0, open = 0;
    for (uint32_t sigma = 1; sigma <= 1024; ++sigma) {
        uint32_t n = 0, R = 0;
        const auto tab = cached_noise_table(sigma);
        if (!tab || !build_bank_table(sigma, words, n, R)) return 1;
        NoiseBankParams bank{};
        set_bank_table(bank, words.data(), words.size(), R);
        bank_guide(words, R);
        const std::vector<uint64_t> &T = tab->T;
        // the word and its mirror image, with the ends of the low words and, where it meets threshold `at`, around that one's
        auto check = [&](int64_t value, uint32_t at = 0, bool meets = false) {
            const uint32_t x = (uint32_t)std::min<int64_t>(std::max<int64_t>(value, 0), 0x7FFFFFFF);
            for (uint32_t u : {x, ~x}) {
                const uint32_t own = (uint32_t)T[u == x ? at : 2 * R - 1 - at], lows[] = {0u, ~0u, own - 1, own, own + 1};
                for (int i = 0; i < (meets ? 5 : 2); ++i) {
                    const uint32_t ulo = lows[i];
                    const int want = (int)(std::upper_bound(T.begin(), T.end(), (uint64_t)u << 32 | ulo) - T.begin()) - (int)R;
                    int got = 0;
                    uint32_t base = 0;
                    const bool decided = looked_up(words, bank.guide_words, bank.s, u, got, base);
                    if (!decided) got = searched(bank.thi, bank.tlo, bank.s, u, ulo, base);
                    ++checked;
                    open += !decided;
                    if (got != want) {
                        std::printf("sigma %u, word %08x %08x: %d instead of %d\n", sigma, u, ulo, got, want);
                        std::exit(1);
                    }
                }
            }
        };
        for (uint32_t j = 0; j < R; ++j) {
            const int64_t x = (int64_t)(T[j] >> 32);
            const int64_t ulp = std::max<int64_t>(1, x >> 24);   // of float(x): neighbours in the table's resolution too
            for (int64_t d : {-2 * ulp, -ulp, (int64_t)-1, (int64_t)0, (int64_t)1, ulp, 2 * ulp}) check(x + d, j, d == 0);
        }
        for (uint32_t b = 127u << 7; b < 158u << 7; ++b)   // first and last floats of the coarsest buckets
            for (uint32_t bits : {b << 16, b << 16 | 0xFFFFu, b << 16 | 0xFFFEu}) {
                float f;
                std::memcpy(&f, &bits, 4);
                check((int64_t)f);
            }
        for (int64_t x : {0, 1, 0x7FFFFFBF, 0x7FFFFFC0, 0x7FFFFFFF}) check(x);
    }
    std::printf("checked %ld open %ld\n", checked, open);
    return 0;
}
