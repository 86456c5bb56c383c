// What a call does with the words that it watches for in host memory, on both word sizes: there already, stored while it waits, stored by the
// time the stream has ended, not even then (an earlier call's word in its place), and a stream that ends in an error.
// Built and run by tests/test_host_watch.py.
#include <cstdio>
#include <thread>

#include "host_watch.h"

using clk = std::chrono::steady_clock;

template <class Word>
static int run(const char *size) {
    const int high = 8 * (sizeof(Word) - 4);
    const Word vote = high ? 5 : 0, before = (Word)6 << high | vote, now = (Word)7 << high | vote;
    const auto soon = clk::now(), later = clk::now() + std::chrono::seconds(60);
    Word word = now;
    auto check = [&](const char *what, int got, int want, bool there) {
        if (got == want && (word == now) == there) return 0;
        std::printf("%s, %s: status %d instead of %d\n", size, what, got, want);
        return 1;
    };
    auto never = [] { return (int)ISR_ERR_ARG; };
    int bad = check("there already", isr::watch(&word, 7, soon, never), ISR_OK, true);
    word = before;
    std::thread kernel([&] {
        std::this_thread::sleep_for(std::chrono::milliseconds(20));
        __atomic_store_n(&word, now, __ATOMIC_RELEASE);
    });
    bad += check("stored meanwhile", isr::watch(&word, 7, later, never), ISR_OK, true);
    kernel.join();
    word = before;
    bad += check("there at the stream's end", isr::watch(&word, 7, soon, [&] { word = now; return (int)ISR_OK; }), ISR_OK, true);
    word = before;
    bad += check("not there at the stream's end", isr::watch(&word, 7, soon, [] { return (int)ISR_OK; }), ISR_ERR_DEVICE, false);
    bad += check("the stream ends in an error", isr::watch(&word, 7, soon, [] { return (int)ISR_ERR_WORKSPACE; }), ISR_ERR_WORKSPACE, false);
    return bad;
}

int main() { return run<uint32_t>("32 bits") + run<uint64_t>("64 bits") ? 1 : 0; }
