// The model object behind the C ABI's opaque handle, shared by the files that implement entry points.
#ifndef ISR_MODEL_H
#define ISR_MODEL_H

#include <map>
#include <string>
#include <vector>

#include "isr_internal.h"
#include "plan.h"

namespace isr {
constexpr int TABLE_SLOTS = 8;
struct FloatNet;   // float_api.cpp: the float network of the FloatRS-fp comparison system, built on first use
void free_float_net(FloatNet *net);
}  // namespace isr

using isr::Plan; using isr::DevOp; using isr::ParsedModel; using isr::DeviceNoiseTable; using isr::NoiseItem;
using isr::TABLE_SLOTS;

struct isr_model {
    ParsedModel pm;
    std::vector<DevOp> ops;             // one descriptor per op of the blob
    Plan plan[3];                       // [0] op by op, [1] with the fusions that pay, [2] with every fusion the kernels cover
    int use_fused = 1;
    int conv_tile = 0;                  // forced conv output tile (0 = automatic)
    uint8_t *dconst = nullptr;          // weights and per-channel tables; dtables and dcounts are in the same allocation
    DeviceNoiseTable *dtables = nullptr;  // TABLE_SLOTS entries
    DeviceNoiseTable *htables = nullptr;  // pinned staging, TABLE_SLOTS entries; hcounts is in the same allocation
    uint32_t table_sigma[TABLE_SLOTS] = {0};
    int table_next = 0;
    uint32_t *dcounts = nullptr;        // 2 * classes
    isr::TallyParts *dparts = nullptr;  // in the same allocation
    uint32_t *hcounts = nullptr, *hcounts_dev = nullptr;   // pinned, 2 * classes, and its address for kernels
    uint32_t *hflag = nullptr, *hflag_dev = nullptr;       // one word in the same pinned allocation: number of the last call whose tallies arrived
    uint64_t *hvotes = nullptr, *hvotes_dev = nullptr;     // DIRECT_VOTES words in the same pinned allocation: votes that go to the host one by one
    uint32_t published = 0;                                // number of the last call that had its tallies or votes sent
    isr::Slots direct{};                // of the running call's votes that go one by one; direct_votes of them, 0: none
    uint32_t direct_votes = 0;
    uint32_t sent_tallies = 0;          // of the running call's tallies, by its last stage kernel itself; 0: none
    hipEvent_t end = nullptr;           // recorded behind tallies whose arrival the host watches
    uint32_t launches = 0;              // of the call that is running
    bool staging_busy = false;          // copies out of htables or hitems may be under way
    bool counts_clean = false, counts_b_clean = false, parts_clean = false;   // dcounts, dcounts_b, dparts hold zeros
    // batched calls: item descriptors and per-item vote counters, grown on demand
    NoiseItem *ditems = nullptr, *hitems = nullptr;
    uint32_t *dcounts_b = nullptr, *hcounts_b = nullptr, *hcounts_b_dev = nullptr;   // 2 * items_cap * classes each
    uint32_t items_cap = 0;
    // workspace
    uint8_t *ws = nullptr;
    size_t ws_bytes = 0;
    uint32_t chunk = 0;
    hipStream_t stream = nullptr;
    // per-kernel timing
    uint32_t profile_every = 0;
    uint64_t chunk_counter = 0;
    std::vector<hipEvent_t> events;
    std::map<std::string, isr_kernel_stat> stats;   // per kernel instance (name as a profiler prints it)
    // floating-point comparison systems
    float quant_sigma = -1.f;           // >= 0 while a FloatRS-quant call runs: the noise stage draws continuous Gaussian noise and rounds it
    isr::FloatNet *fnet = nullptr;
};

namespace isr {
// What the copies of a call are drawn from (NoiseSource without the launch's place in the list).
struct Draw {
    const uint8_t *x;
    const DeviceNoiseTable *table;
    const NoiseItem *items;
    uint64_t seed;
    uint32_t image;
    Slots slots;
};
inline Slots one_phase(uint32_t phase, uint32_t first, uint32_t n) { return Slots{0, n, {n, 0}, 1, phase, first}; }

// The integer path's Monte-Carlo loop with the input stage of FloatRS-quant (api.cpp): noisy copies are
// clamp(round(x + sigma z)) with continuous z instead of discrete-Gaussian draws; everything after is the int8 network.
int run_quant(isr_model *m, const uint8_t *x, float sigma, uint64_t seed, uint32_t image, const Slots &slots,
              int32_t *logits_host, int32_t *argmax_host, uint32_t *dcounts, int stop_tensor);
// The vote counters m->dcounts before a call's first vote: zero; and after its last: on the host in m->hcounts.
int open_counts(isr_model *m);
int close_counts(isr_model *m, uint32_t phases);
}  // namespace isr

#endif
