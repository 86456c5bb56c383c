// Waiting on the host for a word that a kernel stores into host memory.  Plain C++: tests/host_watch_host.cpp runs it.
#pragma once
#include <chrono>
#include <cstdint>

#include "isr.h"

namespace isr {

// Does *word's high part say `seq` (of a word of 32 bits: the word itself)?
template <class Word>
inline bool arrived(const Word *word, uint32_t seq) {
    return (uint32_t)(__atomic_load_n(word, __ATOMIC_ACQUIRE) >> (8 * (sizeof(Word) - 4))) == seq;
}

// Waits until it does.  After `patience` the rest is left to `stream_end`, behind which the word has to be there: whatever an earlier
// call has left in it is never taken for this call's.
template <class Word, class StreamEnd>
int watch(const Word *word, uint32_t seq, std::chrono::steady_clock::time_point patience, StreamEnd stream_end) {
    for (uint32_t spins = 1; !arrived(word, seq); ++spins) {
        if (spins % 64 == 0 && std::chrono::steady_clock::now() > patience) {
            const int rc = stream_end();
            return rc != ISR_OK ? rc : arrived(word, seq) ? ISR_OK : ISR_ERR_DEVICE;
        }
        __builtin_ia32_pause();
    }
    return ISR_OK;
}

}  // namespace isr
