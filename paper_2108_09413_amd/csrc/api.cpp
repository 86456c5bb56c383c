// C ABI: model loading, workspace planning and the Monte-Carlo driver that
// enqueues noise -> layers -> vote kernels for chunks of sample indices.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>

#include "host_watch.h"
#include "isr_internal.h"
#include "model.h"
#include "plan.h"

using namespace isr;

namespace {

thread_local int g_last_hip_error = 0;

#define HIP_TRY(expr)                                     \
    do {                                                  \
        hipError_t e_ = (expr);                           \
        if (e_ != hipSuccess) {                           \
            g_last_hip_error = (int)e_;                   \
            return ISR_ERR_DEVICE;                        \
        }                                                 \
    } while (0)

}  // namespace

void isr::set_last_device_error(int hip_error) { g_last_hip_error = hip_error; }

namespace { thread_local const char *g_kernel_name = ""; }
void isr::set_kernel_name(const char *name) { g_kernel_name = name; }
const char *isr::last_kernel_name() { return g_kernel_name; }


namespace {

// The pinned staging memory before it is written anew: copies out of it of an earlier call have ended.  Published tallies say so;
// after a call that published none, or failed on its way, the stream's end does.  A stream that is being captured is refused, here
// as by the synchronisation: a copy that is only recorded would leave its table marked as resident.
int free_staging(isr_model *m) {
    if (m->staging_busy) {
        HIP_TRY(hipStreamSynchronize(m->stream));
    } else {
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        HIP_TRY(hipStreamIsCapturing(m->stream, &capture));
        if (capture != hipStreamCaptureStatusNone) HIP_TRY(hipErrorStreamCaptureUnsupported);
    }
    m->staging_busy = false;
    return ISR_OK;
}

int get_table(isr_model *m, uint32_t sigma, const DeviceNoiseTable **out) {
    int rc;
    for (int i = 0; i < TABLE_SLOTS; ++i)
        if (m->table_sigma[i] == sigma) { *out = m->dtables + i; return ISR_OK; }
    int slot = m->table_next;
    m->table_next = (slot + 1) % TABLE_SLOTS;
    if ((rc = free_staging(m)) != ISR_OK) return rc;
    if (!build_device_table(sigma, m->htables[slot])) return ISR_ERR_ARG;
    m->staging_busy = true;
    HIP_TRY(hipMemcpyAsync(m->dtables + slot, m->htables + slot, sizeof(DeviceNoiseTable), hipMemcpyHostToDevice, m->stream));
    m->table_sigma[slot] = sigma;
    *out = m->dtables + slot;
    return ISR_OK;
}

// Device tables of isr_noise_bank: a call has one to itself until its stream is synchronised and hands it back; the next call
// on the GPU with the same sigma finds it filled.  At most BANK_TABLES wait for the next call, the others are freed, and
// all are when the process ends (registered after the HIP runtime's own handlers, so run before them).
constexpr size_t BANK_TABLE_BYTES = 128 * 1024;   // sigma 1024 takes 126 840
constexpr size_t BANK_TABLES = 4;
struct BankTable {
    int device = -1;
    uint32_t sigma = 0, R = 0;                // of the contents; 0: none
    size_t words = 0;
    uint32_t *dev = nullptr, *host = nullptr; // host: pinned staging
    void free() { if (dev) (void)hipFree(dev); if (host) (void)hipHostFree(host); dev = host = nullptr; }
};
class BankTables {
  public:
    hipError_t take(uint32_t sigma, BankTable &t) {
        int device = 0;
        hipError_t e = hipGetDevice(&device);
        if (e != hipSuccess) return e;
        {
            std::lock_guard<std::mutex> lock(mu_);
            int best = -1;
            for (size_t i = 0; i < idle_.size(); ++i)
                if (idle_[i].device == device && (best < 0 || idle_[i].sigma == sigma)) best = (int)i;
            if (best >= 0 && (idle_[best].sigma == sigma || idle_.size() == BANK_TABLES)) {
                t = idle_[best];
                idle_.erase(idle_.begin() + best);
                return hipSuccess;
            }
        }
        t = BankTable();
        t.device = device;
        e = hipMalloc((void **)&t.dev, BANK_TABLE_BYTES);
        if (e == hipSuccess) e = hipHostMalloc((void **)&t.host, BANK_TABLE_BYTES, hipHostMallocDefault);
        if (e != hipSuccess) t.free();
        return e;
    }
    void give_back(BankTable &t) {
        if (!t.dev) return;
        BankTable oldest;
        {
            std::lock_guard<std::mutex> lock(mu_);
            static const int at_exit = std::atexit([] { all().clear(); });
            (void)at_exit;
            idle_.push_back(t);
            if (idle_.size() > BANK_TABLES) { oldest = idle_.front(); idle_.erase(idle_.begin()); }
        }
        oldest.free();
    }
    void clear() {
        std::lock_guard<std::mutex> lock(mu_);
        for (BankTable &t : idle_) t.free();
        idle_.clear();
    }
    static BankTables &all() { static BankTables &t = *new BankTables; return t; }   // outlives static destruction

  private:
    std::mutex mu_;
    std::vector<BankTable> idle_;   // oldest first
};

// Room that the constants of the narrow-net ops need at most: in either plan each convolution's once (three times where a
// kernel stages as many), one descriptor per op.
size_t narrow_ops_room(const std::vector<DevOp> &ops) {
    size_t bytes = 512;
    for (const DevOp &d : ops) bytes += 2 * (sizeof(NarrowBlock) + (d.type == OP_CONV ? (size_t)3 * 4 * 4 * d.conv.Cout_p : 0));
    return bytes;
}

// The constant arguments of the narrow-net ops of the fused plans: block descriptors and per-channel constants packed
// in the form the kernel stages them, appended to `arena`, the host image of the constants at m->dconst.
int build_narrow_ops(isr_model *m, ConstArena &arena, size_t limit) {
    std::vector<NarrowBlock> blocks;
    std::vector<int32_t> consts;
    auto host = [&](const int32_t *dev) { return (const int32_t *)(arena.host.data() + ((const uint8_t *)dev - m->dconst)); };
    auto form_of = [](int rq, int add_rq) { return !(rq & RQ_PAIR) ? 2 : add_rq & RQ_PAIR ? 0 : 1; };
    auto pack = [&](const ConvParams &c) {   // [4][C], returns its offset
        const size_t off = consts.size();
        const int C = c.Cout_p;
        consts.resize(off + 4 * C);
        int32_t *k = consts.data() + off;
        for (int i = 0; i < C; ++i) {
            k[i] = host(c.bias)[i];
            k[C + i] = host(c.m0s)[i];
            k[2 * C + i] = host(c.chi)[i];
            k[3 * C + i] = host(c.shm1)[i];
        }
        return off;
    };
    auto add_of = [](const ConvParams &c, bool pair) {   // as add_const of the kernels
        return pair ? AddConst{c.add_mul_self, c.add_mul_res, c.add_c0 + c.add_k, 0, c.add_sh, 0}
                    : AddConst{c.add_mul_self, c.add_mul_res, c.add_c0, c.add_k, c.add_sh, c.add_lo};
    };
    auto lo_of = [](const ConvParams &c) { return c.relu ? c.zp_out : -128; };
    for (int pi = 1; pi <= 2; ++pi)
        for (DevOp &d : m->plan[pi].ops) {
            if (!d.narrow) continue;
            NarrowParams &np = d.np;
            // offsets now (+ 1: 0 stays "none"), pointers after the upload
            for (const DevOp &q : d.parts) {
                const ConvParams &c1 = q.conv, &c2 = q.conv2, &cp = q.conv3;
                if (q.stem16) {
                    np.stem = 1;
                    np.form0 = form_of(c1.rq, RQ_PAIR);
                    np.w0 = c1.w; np.zp_in = c1.zp_in; np.lo0 = lo_of(c1);
                    np.prm0 = (const int32_t *)(pack(c1) + 1);
                } else if (q.block) {
                    np.nblocks = (int32_t)q.chain.size();
                    np.blocks = (const NarrowBlock *)(blocks.size() + 1);
                    for (const auto &blk : q.chain) {
                        const ConvParams &a = blk.first, &b = blk.second;
                        NarrowBlock nb{};
                        nb.form = form_of(a.rq & b.rq, b.add_rq);
                        nb.w1 = a.w; nb.w2 = b.w;
                        nb.prm1 = (const int32_t *)pack(a);
                        nb.prm2 = (const int32_t *)pack(b);
                        nb.zp_x = a.zp_in; nb.zp_t = a.zp_out; nb.lo1 = lo_of(a); nb.lo2 = lo_of(b);
                        nb.add = add_of(b, nb.form == 0);
                        blocks.push_back(nb);
                    }
                } else if (q.trans) {
                    np.tail = 1;
                    np.tform = form_of(c1.rq & c2.rq & cp.rq, cp.add_rq);
                    np.tw1 = c1.w; np.tw2 = c2.w; np.twp = cp.w;
                    np.tprm = (const int32_t *)(pack(c1) + 1);
                    pack(c2);
                    pack(cp);
                    np.tzp_x = c1.zp_in; np.tzp_t = c1.zp_out;
                    np.tlo1 = lo_of(c1); np.tlo2 = lo_of(c2); np.tlop = lo_of(cp);
                    np.tadd = add_of(cp, np.tform == 0);
                } else if (q.type == OP_CONV) {
                    np.tail = 2;
                    np.tform = form_of(c1.rq, RQ_PAIR);
                    np.tw1 = c1.w;
                    np.tprm = (const int32_t *)(pack(c1) + 1);
                    consts.resize(consts.size() + 2 * 4 * c1.Cout_p);   // the kernel stages three convolutions' constants
                    np.tzp_x = c1.zp_in; np.tzp_t = c1.zp_out; np.tlo1 = lo_of(c1);
                } else if (q.type == OP_GAP) {
                    np.head = 1;
                    np.gap_zp_in = q.gap.zp_in; np.gap_zp_out = q.gap.zp_out; np.gap_M0 = q.gap.M0; np.gap_sh = q.gap.sh;
                } else {
                    np.fc_w = q.fc.w; np.fc_bias = q.fc.bias; np.classes = q.fc.classes; np.classes_p = q.fc.classes_p;
                }
            }
        }
    if (blocks.empty() && consts.empty()) return ISR_OK;
    const size_t block_bytes = (blocks.size() * sizeof(NarrowBlock) + 255) & ~(size_t)255;
    uint8_t *dnarrow = m->dconst + arena.host.size();   // the end of the constants on the device too
    if (arena.host.size() + block_bytes + consts.size() * 4 > limit) return ISR_ERR_UNSUPPORTED;   // cannot happen: narrow_ops_room
    const int32_t *dconsts = (const int32_t *)(dnarrow + block_bytes);
    for (NarrowBlock &nb : blocks) { nb.prm1 = dconsts + (size_t)nb.prm1; nb.prm2 = dconsts + (size_t)nb.prm2; }
    for (int pi = 1; pi <= 2; ++pi)
        for (DevOp &d : m->plan[pi].ops) {
            NarrowParams &np = d.np;
            if (!d.narrow) continue;
            if (np.prm0) np.prm0 = dconsts + (size_t)np.prm0 - 1;
            if (np.tprm) np.tprm = dconsts + (size_t)np.tprm - 1;
            if (np.blocks) {
                np.first = blocks[(size_t)np.blocks - 1];
                np.blocks = (const NarrowBlock *)dnarrow + (size_t)np.blocks - 1;
            }
        }
    const size_t at = arena.host.size();
    arena.host.resize(at + block_bytes + consts.size() * 4);
    std::memcpy(arena.host.data() + at, blocks.data(), blocks.size() * sizeof(NarrowBlock));
    std::memcpy(arena.host.data() + at + block_bytes, consts.data(), consts.size() * 4);
    return ISR_OK;
}

// Enqueues the Monte-Carlo loop over the slots of a call.  Optional outputs: per-sample logits / argmax (device
// buffers inside the workspace, copied to the host pointers chunk by chunk) and the device vote counters,
// [phases][pairs][classes].  stop_tensor >= 0 ends each forward right after that tensor.  Chunks are cut from the slot list
// without regard to the boundaries of pairs and phases, so short runs still fill the device.
int run_slots(isr_model *m, const Plan &pl, const Draw &draw, int32_t *logits_host, int32_t *argmax_host, uint32_t *dcounts,
              int stop_tensor) {
    const ParsedModel &pm = m->pm;
    uint8_t *ws = m->ws;
    Slots slots = draw.slots;
    const uint64_t count = slots.split + (uint64_t)slots.pairs * slots.n[1];
    // bytes of one copy of a tensor: copies are contiguous, so a range of copies of a chunk is a sub-chunk
    auto tptr = [&](int t, uint32_t first_copy) -> uint8_t * {
        const TensorDesc &d = pm.tensors[t];
        return ws + pl.toff[t] + (size_t)first_copy * d.H * d.W * d.Cp;
    };
    // a plan that takes more copies than asked for gets equal chunks, so that no short one is left over
    uint64_t per_chunk = pl.chunk;
    if (pl.chunk > m->chunk && count > pl.chunk) {
        const uint64_t chunks = (count + pl.chunk - 1) / pl.chunk;
        per_chunk = (count + chunks - 1) / chunks;
    }
    // votes of few copies in one chunk go to the host one by one where the last op is a stage kernel
    const bool heads = dcounts && stop_tensor < 0 && !pl.ops.empty() && pl.ops.back().narrow && pl.ops.back().head;
    const bool direct = heads && count <= DIRECT_VOTES && count <= per_chunk;
    // and the few tallies of more by that kernel's last workgroup.  Calls of ResNet-20 are 0.8 us shorter for it (narrow_head,
    // narrow_net.hip); above 4096 copies, without the pause that a kernel of one workgroup is, 10 100 copies one call after the other ran
    // at a lower clock, 609 us instead of 599, on one of two cards.  Nets of two convolutions end this way whatever the number: added to
    // one place, their votes are what bounds the call (narrow_head).
    const uint64_t words = (uint64_t)(slots.n[1] ? 2 : 1) * slots.pairs * pm.classes;
    const bool sends = heads && !direct && words <= SENT_TALLIES && (count <= SENT_COPIES || narrow_short(pl.ops.back().np)) &&
                       (dcounts == m->dcounts || dcounts == m->dcounts_b);
    if (direct) {
        ++m->published;
        m->direct = slots;
        m->direct_votes = (uint32_t)count;
    }
    for (uint64_t done = 0; done < count;) {
        uint32_t cnt = (uint32_t)std::min<uint64_t>(per_chunk, count - done);
        const bool timed = m->profile_every && (m->chunk_counter++ % m->profile_every) == 0;
        size_t ev = 0;
        auto mark = [&]() -> int {   // event before a launch / after the last one
            ++m->launches;
            if (!timed) return ISR_OK;
            if (ev == m->events.size()) {
                hipEvent_t e;
                HIP_TRY(hipEventCreate(&e));
                m->events.push_back(e);
            }
            HIP_TRY(hipEventRecord(m->events[ev++], m->stream));
            return ISR_OK;
        };
        struct Work { const char *kernel; int conv; double ops, bytes; };
        std::vector<Work> ev_work;   // per timed launch: the kernel instance and its algorithmic work
        int prc;

        // where the copies from j0 on are in the list, and draw their noise
        auto slots_at = [&](uint32_t j0) { Slots l = slots; l.begin = done + j0; return l; };
        auto noise_source = [&](uint32_t j0) {
            NoiseSource ns{};
            ns.x = draw.x; ns.table = draw.table; ns.items = draw.items;
            ns.key0 = (uint32_t)draw.seed; ns.key1 = (uint32_t)(draw.seed >> 32); ns.image = draw.image;
            ns.C = pm.C; ns.H = pm.H; ns.W = pm.W;
            ns.slots = slots_at(j0);
            return ns;
        };
        // copies [j0, j0 + bn) of the chunk through the noise stage, for plans that have it as a launch of its own
        auto run_noise = [&](uint32_t j0, uint32_t bn) -> int {
            for (uint32_t j = j0; j < j0 + bn;) {
                // one phase, and at most one grid row per pair
                const uint64_t slot = done + j;
                const uint32_t second = slot >= slots.split, n = slots.n[second];
                const uint64_t s0 = second ? slot - slots.split : slot;
                uint64_t bm = std::min<uint64_t>(j0 + bn - j, second ? count - slot : slots.split - slot);
                if (slots.pairs > 1) bm = std::min<uint64_t>(bm, (uint64_t)n * 65534);
                NoiseParams np;
                np.x = draw.x; np.table = draw.table; np.out = (int8_t *)tptr(0, j);
                np.C = pm.C; np.H = pm.H; np.W = pm.W;
                np.key0 = (uint32_t)draw.seed; np.key1 = (uint32_t)(draw.seed >> 32);
                np.image = draw.image; np.phase = slots.phase + second; np.sample_begin = slots.first + (uint32_t)s0; np.count = (uint32_t)bm;
                np.items = draw.items; np.n_per_item = 0; np.item_first = 0; np.item_count = 0; np.slot_begin = 0;
                if (draw.items) {
                    np.n_per_item = n; np.slot_begin = s0;
                    np.item_first = (uint32_t)(s0 / n);
                    np.item_count = (uint32_t)((s0 + bm - 1) / n) - np.item_first + 1;
                }
                if ((prc = mark()) != ISR_OK) return prc;
                if (m->quant_sigma >= 0.f) {   // FloatRS-quant: continuous noise rounded onto the pixel grid (single pair only)
                    FloatNoiseParams fp{};
                    fp.x = draw.x; fp.out = np.out; fp.C = pm.C; fp.H = pm.H; fp.W = pm.W;
                    fp.key0 = np.key0; fp.key1 = np.key1; fp.image = np.image; fp.phase = np.phase;
                    fp.sample_begin = np.sample_begin; fp.count = np.count; fp.sigma = m->quant_sigma; fp.center = 0.f; fp.quant = 1;
                    HIP_TRY(launch_float_noise(fp, m->stream));
                } else {
                    HIP_TRY(launch_noise(np, m->stream));
                }
                if (timed) ev_work.push_back({last_kernel_name(), 0, 0.0, (double)bm * pm.H * pm.W * 4});
                j += (uint32_t)bm;
            }
            return ISR_OK;
        };
        auto narrow_params = [&](const DevOp &d, uint32_t j0, uint32_t bn) {
            NarrowParams np = d.np;
            np.in = (const int8_t *)tptr(d.a, j0);
            np.out = d.head ? nullptr : (int8_t *)tptr(d.out, j0);
            np.B = (int32_t)bn;
            np.fused_noise = d.noise_fused && m->quant_sigma < 0.f;
            if (np.fused_noise) np.noise = noise_source(j0);
            if (d.head) {
                np.logits = logits_host ? (int32_t *)(ws + pl.logits_off) + (size_t)j0 * pm.classes : nullptr;
                np.argmax = argmax_host ? (int32_t *)(ws + pl.argmax_off) + j0 : nullptr;
                np.counts = direct ? nullptr : dcounts;
                np.votes = direct ? m->hvotes_dev : nullptr;
                np.seq = m->published;
                np.slots = slots_at(j0);
                if (sends) {
                    np.parts = m->dparts;
                    m->parts_clean = false;
                }
                if (sends && done + j0 + bn == count) {   // the call's last launch
                    const bool batch = dcounts == m->dcounts_b;
                    np.seq = ++m->published;
                    np.tallies = m->sent_tallies = (uint32_t)words;
                    np.tally_host = batch ? m->hcounts_b_dev : m->hcounts_dev;
                    np.flag = m->hflag_dev;
                }
            }
            return np;
        };
        // copies [j0, j0 + bn) of the chunk through the three stages of a net on 32x32 images, one launch
        auto run_chain = [&](const DevOp *d, uint32_t j0, uint32_t bn) -> int {
            if ((prc = mark()) != ISR_OK) return prc;
            HIP_TRY(launch_narrow_chain(narrow_params(d[0], j0, bn), narrow_params(d[1], j0, bn), narrow_params(d[2], j0, bn), m->stream));
            if (timed)
                ev_work.push_back({last_kernel_name(), 1, (d[0].ops_per_sample + d[1].ops_per_sample + d[2].ops_per_sample) * bn,
                                   (d[0].bytes_per_sample + d[1].bytes_per_sample + d[2].bytes_per_sample) * bn});
            return ISR_OK;
        };
        // copies [j0, j0 + bn) of the chunk through one op of the plan
        auto run_op = [&](const DevOp &d, uint32_t j0, uint32_t bn) -> int {
            if ((prc = mark()) != ISR_OK) return prc;
            set_kernel_name("");
            switch (d.type) {
            case OP_CONV: {
                if (d.stem_pool) {
                    const TensorDesc &to = pm.tensors[d.out];
                    StemPoolParams sp;
                    sp.in = (const int8_t *)tptr(d.a, j0);
                    sp.out = (int8_t *)tptr(d.out, j0);
                    sp.w = d.conv.w; sp.bias = d.conv.bias; sp.m0s = d.conv.m0s; sp.chi = d.conv.chi; sp.shm1 = d.conv.shm1;
                    sp.H = d.conv.H; sp.W = d.conv.W; sp.Ho = d.conv.Ho; sp.Wo = d.conv.Wo; sp.Hp = to.H; sp.Wp = to.W;
                    sp.zp_in = d.conv.zp_in; sp.zp_out = d.conv.zp_out; sp.relu = d.conv.relu; sp.rq = d.conv.rq; sp.B = (int32_t)bn;
                    sp.fused_noise = d.noise_fused && m->quant_sigma < 0.f;
                    sp.noise = sp.fused_noise ? noise_source(j0) : NoiseSource{};
                    HIP_TRY(launch_stem_pool(sp, m->stream));
                    break;
                }
                if (d.stem16) {
                    const ConvParams &c = d.conv;
                    Stem16Params sp;
                    sp.in = (const int8_t *)tptr(d.a, j0);
                    sp.out = (int8_t *)tptr(d.out, j0);
                    sp.w = c.w; sp.bias = c.bias; sp.m0s = c.m0s; sp.chi = c.chi; sp.shm1 = c.shm1;
                    sp.H = c.H; sp.W = c.W; sp.B = (int32_t)bn; sp.zp_in = c.zp_in;
                    sp.lo = c.relu ? c.zp_out : -128; sp.tie_free = c.tie_free;
                    HIP_TRY(launch_stem16(sp, m->stream));
                    break;
                }
                if (d.narrow) {
                    HIP_TRY(launch_narrow(narrow_params(d, j0, bn), d.narrow, m->stream));
                    break;
                }
                if (d.bneck) {
                    const ConvParams &c1 = d.conv, &c2 = d.conv2, &c3 = d.conv3;
                    BneckParams bp{};
                    bp.in = (const int8_t *)tptr(d.a, j0);
                    bp.out = (int8_t *)tptr(d.out, j0);
                    bp.w1 = c1.w; bp.bias1 = c1.bias; bp.m0s1 = c1.m0s; bp.chi1 = c1.chi; bp.shm11 = c1.shm1;
                    bp.w2 = c2.w; bp.bias2 = c2.bias; bp.m0s2 = c2.m0s; bp.chi2 = c2.chi; bp.shm12 = c2.shm1;
                    bp.zpad = c1.zpad;
                    bp.Cin_p = c1.Cin_p; bp.H = c1.H; bp.W = c1.W; bp.B = (int32_t)bn; bp.tail = d.bneck >= 2;
                    bp.zp_t1 = c1.zp_out;
                    bp.lo1 = c1.relu ? c1.zp_out : -128;
                    bp.lo2 = c2.relu ? c2.zp_out : -128;
                    bp.rq = c1.rq & c2.rq; bp.add_rq = RQ_TOP | RQ_PAIR;
                    if (bp.tail) {
                        // the closing 1x1 convolution; with a projection shortcut (bneck == 4) conv3 carries two
                        // convolutions, and either of them may be the one that reads the block input
                        const bool swap = d.bneck == 4 && d.proj_is_main;
                        bp.w3 = swap ? c3.w2 : c3.w; bp.bias3 = swap ? c3.bias2 : c3.bias; bp.m0s3 = swap ? c3.m0s2 : c3.m0s;
                        bp.chi3 = swap ? c3.chi2 : c3.chi; bp.shm13 = swap ? c3.shm12 : c3.shm1;
                        bp.Cout_p = c3.Cout_p;
                        const int lo_main = c3.relu ? c3.zp_out : -128;
                        bp.lo3 = swap ? c3.lo2 : lo_main;
                        bp.add_mul_self = swap ? c3.add_mul_res : c3.add_mul_self;   // "self" in the kernel = the closing convolution
                        bp.add_mul_res = swap ? c3.add_mul_self : c3.add_mul_res;
                        bp.add_c0 = c3.add_c0; bp.add_k = c3.add_k; bp.add_sh = c3.add_sh; bp.add_lo = c3.add_lo;
                        bp.rq &= c3.rq & (d.bneck == 4 ? c3.rq2 : ~0);
                        bp.add_rq = c3.add_rq;
                        if (d.bneck == 4) {
                            bp.proj = 1;
                            bp.wp = swap ? c3.w : c3.w2; bp.biasp = swap ? c3.bias : c3.bias2; bp.m0sp = swap ? c3.m0s : c3.m0s2;
                            bp.chip = swap ? c3.chi : c3.chi2; bp.shm1p = swap ? c3.shm1 : c3.shm12;
                            bp.lop = swap ? lo_main : c3.lo2;
                        }
                    }
                    if (d.reduce) {
                        const ConvParams &c4 = d.conv4;
                        bp.reduce = 1; bp.sparse = d.sparse;
                        bp.out2 = (int8_t *)tptr(d.out2, j0);
                        bp.wp = c4.wfrag; bp.biasp = c4.bias; bp.m0sp = c4.m0s; bp.chip = c4.chi; bp.shm1p = c4.shm1;
                        bp.lop = c4.relu ? c4.zp_out : -128;
                        bp.rq &= c4.rq;
                    }
                    if (d.bneck == 3) HIP_TRY(launch_bottleneck128(bp, m->stream));
                    else HIP_TRY(launch_bottleneck(bp, m->stream));
                    break;
                }
                if (d.xr) {
                    XrParams xp;
                    expand_reduce_params(d.conv, d.conv2, (const int8_t *)tptr(d.a, j0), (const int8_t *)tptr(d.b, j0),
                                         (int8_t *)tptr(d.out, j0), (int8_t *)tptr(d.out2, j0), (int32_t)bn, xp);
                    HIP_TRY(launch_expand_reduce(xp, m->stream));
                    break;
                }
                ConvParams c = d.conv;
                c.in = (const int8_t *)tptr(d.a, j0);
                c.out = (int8_t *)tptr(d.out, j0);
                c.res = c.fuse_add == 1 ? (const int8_t *)tptr(d.b, j0) : nullptr;
                c.in2 = c.fuse_add == 2 ? (const int8_t *)tptr(d.b, j0) : nullptr;
                c.npix = (int32_t)(bn * c.Ho * c.Wo);
                c.force_tile = m->conv_tile;
                HIP_TRY(launch_conv(c, m->stream));
                break; }
            case OP_ADD: {
                AddParams a = d.add;
                const TensorDesc &t = pm.tensors[d.out];
                a.a = (const int8_t *)tptr(d.a, j0);
                a.b = (const int8_t *)tptr(d.b, j0);
                a.out = (int8_t *)tptr(d.out, j0);
                a.n16 = (int64_t)bn * t.H * t.W * t.Cp / 16;
                HIP_TRY(launch_add(a, m->stream));
                break; }
            case OP_MAXPOOL: {
                PoolParams p = d.pool;
                p.in = (const int8_t *)tptr(d.a, j0);
                p.out = (int8_t *)tptr(d.out, j0);
                p.B = (int32_t)bn;
                HIP_TRY(launch_maxpool(p, m->stream));
                break; }
            case OP_GAP: {
                GapParams g = d.gap;
                g.in = (const int8_t *)tptr(d.a, j0);
                g.out = (int8_t *)tptr(d.out, j0);
                g.B = (int32_t)bn;
                HIP_TRY(launch_gap(g, m->stream));
                break; }
            case OP_FC: {
                FcParams f = d.fc;
                f.in = (const int8_t *)tptr(d.a, j0);
                f.B = (int32_t)bn;
                f.logits = logits_host ? (int32_t *)(ws + pl.logits_off) + (size_t)j0 * pm.classes : nullptr;
                f.argmax = argmax_host ? (int32_t *)(ws + pl.argmax_off) + j0 : nullptr;
                f.counts = dcounts;
                f.slots = slots_at(j0);
                HIP_TRY(launch_fc(f, m->stream));
                break; }
            }
            if (timed) ev_work.push_back({last_kernel_name(), d.type == OP_CONV ? 1 : 0, d.ops_per_sample * bn, d.bytes_per_sample * bn});
            return ISR_OK;
        };

        // The plan is walked in segments (plan.h): the ops of a segment run back to back on one
        // sub-chunk of copies after the other, so that what an op writes is still in the caches
        // when the next op of the segment reads it.  Segment 0 starts with the noise stage.
        size_t nops = pl.ops.size();
        if (stop_tensor == 0) nops = 0;
        else if (stop_tensor > 0)
            for (size_t i = 0; i < pl.ops.size(); ++i)
                if (pl.ops[i].out == stop_tensor || pl.ops[i].out2 == stop_tensor) { nops = i + 1; break; }
        size_t op0 = 0;
        bool noise_done = false;
        for (size_t sg = 0; sg <= pl.segments.size() && (op0 < nops || !noise_done); ++sg) {
            // ops [op0, op1) in sub-chunks of `sub` copies; past the last segment: the rest, whole chunk
            size_t op1 = nops;
            uint32_t sub = cnt;
            if (sg < pl.segments.size()) {
                op1 = std::min(nops, pl.segments[sg].end);
                sub = std::max<uint32_t>(1, std::min(cnt, pl.segments[sg].sub));
            }
            if (op1 < op0) op1 = op0;
            // no noise launch when the first op of the plan draws its own input (and runs at all)
            const bool own_noise = nops > 0 && !pl.ops.empty() && pl.ops[0].noise_fused && m->quant_sigma < 0.f;
            for (uint32_t j0 = 0; j0 < cnt; j0 += sub) {
                const uint32_t bn = std::min(sub, cnt - j0);
                if (!noise_done && !own_noise && (prc = run_noise(j0, bn)) != ISR_OK) return prc;
                for (size_t i = op0; i < op1; ++i) {
                    const DevOp *d = &pl.ops[i];
                    const bool chain = op1 - i >= 3 && d[0].narrow == 16 && d[1].narrow == 32 && d[2].narrow == 64 && d[0].np.tail == 1 && d[1].np.tail == 1 &&
                                       d[1].a == d[0].out && d[2].a == d[1].out && narrow_chain_wanted((int)bn) && images_apart(pm, pl, i);
                    if ((prc = chain ? run_chain(d, j0, bn) : run_op(*d, j0, bn)) != ISR_OK) return prc;
                    if (chain) i += 2;
                }
            }
            noise_done = true;
            op0 = op1;
        }
        if (timed) {
            if ((prc = mark()) != ISR_OK) return prc;
            HIP_TRY(hipStreamSynchronize(m->stream));
            for (size_t i = 0; i + 1 < ev && i < ev_work.size(); ++i) {
                float ms = 0.f;
                HIP_TRY(hipEventElapsedTime(&ms, m->events[i], m->events[i + 1]));
                isr_kernel_stat &st = m->stats[ev_work[i].kernel];
                if (st.launches == 0) {
                    std::strncpy(st.name, ev_work[i].kernel, sizeof(st.name) - 1);
                    st.is_conv = ev_work[i].conv;
                }
                st.launches += 1;
                st.total_ms += ms;
                st.alg_ops += ev_work[i].ops;
                st.alg_bytes += ev_work[i].bytes;
            }
        }
        if (logits_host) {
            HIP_TRY(hipMemcpyAsync(logits_host + (size_t)done * pm.classes, ws + pl.logits_off,
                                   (size_t)cnt * pm.classes * 4, hipMemcpyDeviceToHost, m->stream));
        }
        if (argmax_host) {
            HIP_TRY(hipMemcpyAsync(argmax_host + done, ws + pl.argmax_off, (size_t)cnt * 4,
                                   hipMemcpyDeviceToHost, m->stream));
        }
        if (logits_host || argmax_host) HIP_TRY(hipStreamSynchronize(m->stream));
        done += cnt;
    }
    return ISR_OK;
}

}  // namespace

int isr::run_quant(isr_model *m, const uint8_t *x, float sigma, uint64_t seed, uint32_t image, const Slots &slots,
                   int32_t *logits_host, int32_t *argmax_host, uint32_t *dcounts, int stop_tensor) {
    m->quant_sigma = sigma;
    const int rc = run_slots(m, m->plan[m->use_fused], Draw{x, nullptr, nullptr, seed, image, slots}, logits_host, argmax_host, dcounts, stop_tensor);
    m->quant_sigma = -1.f;
    return rc;
}

// The counters are zero between calls: the last kernel of a call leaves them so.  After a call that failed on its way (and, of a batch,
// in new memory) they are cleared here.
static int open_call(isr_model *m) {
    if (!m->parts_clean) HIP_TRY(launch_fill_u32((uint32_t *)m->dparts, 0, sizeof(TallyParts) / 4, m->stream));
    m->parts_clean = true;
    m->launches = m->direct_votes = m->sent_tallies = 0;
    return ISR_OK;
}
int isr::open_counts(isr_model *m) {
    if (!m->counts_clean) HIP_TRY(launch_fill_u32(m->dcounts, 0, 2 * (size_t)m->pm.classes, m->stream));
    m->counts_clean = false;
    return open_call(m);
}
// Tallies to the host and zeros on the device, by the last kernel of a call: nothing that the call was given is in use when its
// flag has arrived, only the kernel's own end is still to come.  Waits of more than 2 ms, and what goes wrong, are the runtime's.
//
// The event behind the kernel has the stream's end on its way while the host watches; without it whoever synchronises next only
// then asks for it, and waits longer than the flag has saved.  Behind more than five launches and this one a synchronisation
// that comes after the end takes 28 us, whatever they are, where one that waits for the end takes 2, so such a call waits for the stream
// itself.  us of calls in a row / of a call and a synchronisation of the device behind it, prediction with 100 copies or
// (two-convolution net, one launch) certification with 1000:
//                                    stream's end      flag alone       flag and event
//   two-convolution net              38.7 / 41.1       34.8 / 45.0      34.6 / 39.0
//   ResNet-20                        47.0 / 49.5       42.6 / 53.0      42.1 / 46.5
//   ResNet-50, 36 launches            956 /  960        948 /  981       947 /  980
//   two-convolution net, 5 launches   81.6 / 83.8                        77.2 / 81.6
//   two-convolution net, 6 launches   94.3 / 96.7                        90.0 / 118.4
//   ResNet-20, 5 launches           179.6 / 181.4                      174.6 / 178.9
//   ResNet-20, 6 launches           210.6 / 213.0                      205.9 / 233.9
//   20 pairs of 10 classes           58.7 / 60.7       62.9 / 63.7      54.5 / 56.5
//   256 pairs of 10 classes         265.8 / 268.1     274.7 / 270.8    260.6 / 262.3
constexpr uint32_t WATCHED_LAUNCHES = 5;
// Up to 256 votes (a launch whose workgroups all run at once) are not even tallied on the device: the host watches for each of them in
// its memory and no launch stands behind the last one (prediction of ResNet-20 with 100 copies 42.2 -> 39.7 us).  More are tallied
// there: stores of single words to the host are 20 ns apart.  Up to 256 tallies of up to 4096 copies of such a net (of two convolutions: of
// any number) are sent by the last workgroup of its last kernel, with no launch of their own either.
static int publish(isr_model *m, uint32_t *counts, uint32_t *host, uint32_t *host_dev, size_t n) {
    const auto patience = std::chrono::steady_clock::now() + std::chrono::milliseconds(2);
    auto stream_end = [m]() -> int {
        HIP_TRY(hipStreamSynchronize(m->stream));
        return ISR_OK;
    };
    int rc;
    if (m->direct_votes) {
        HIP_TRY(hipEventRecord(m->end, m->stream));
        std::fill(host, host + n, 0u);
        for (uint32_t i = 0; i < m->direct_votes; ++i) {
            if ((rc = watch(&m->hvotes[i], m->published, patience, stream_end)) != ISR_OK) return rc;
            host[(size_t)slot_use(m->direct, i).row * m->pm.classes + (uint32_t)m->hvotes[i]] += 1;
        }
    } else if (m->sent_tallies) {
        if (m->sent_tallies != n) return ISR_ERR_ARG;   // cannot happen: the counters of all phases and pairs
        if (m->launches <= WATCHED_LAUNCHES + 1) {
            HIP_TRY(hipEventRecord(m->end, m->stream));
            if ((rc = watch(m->hflag, m->published, patience, stream_end)) != ISR_OK) return rc;
        } else {
            HIP_TRY(hipStreamSynchronize(m->stream));
            if (!arrived(m->hflag, m->published)) return ISR_ERR_DEVICE;
        }
        m->parts_clean = true;
    } else if (n <= PUBLISH_WATCHED && m->launches <= WATCHED_LAUNCHES) {
        HIP_TRY(launch_publish(counts, host_dev, n, m->hflag_dev, ++m->published, m->stream));
        HIP_TRY(hipEventRecord(m->end, m->stream));
        if ((rc = watch(m->hflag, m->published, patience, stream_end)) != ISR_OK) return rc;
    } else {
        HIP_TRY(launch_publish(counts, host_dev, n, nullptr, 0, m->stream));
        HIP_TRY(hipStreamSynchronize(m->stream));
    }
    m->staging_busy = false;
    return ISR_OK;
}
int isr::close_counts(isr_model *m, uint32_t phases) {
    const int rc = publish(m, m->dcounts, m->hcounts, m->hcounts_dev, (size_t)phases * m->pm.classes);
    if (rc != ISR_OK) return rc;
    m->counts_clean = true;
    return ISR_OK;
}

namespace {

// Makes the tables of every sigma in `sigmas` resident at once (at most TABLE_SLOTS
// distinct values) and returns the slot of each.  The staging memory is free (free_staging).
int get_tables(isr_model *m, const std::vector<uint32_t> &sigmas, std::vector<uint32_t> &slots) {
    std::vector<uint32_t> distinct;
    for (uint32_t s : sigmas)
        if (std::find(distinct.begin(), distinct.end(), s) == distinct.end()) distinct.push_back(s);
    if ((int)distinct.size() > TABLE_SLOTS) return ISR_ERR_ARG;
    for (uint32_t s : distinct) {
        bool have = false;
        for (int i = 0; i < TABLE_SLOTS; ++i) have = have || m->table_sigma[i] == s;
        if (have) continue;
        int slot = -1;   // a slot whose table this batch does not need
        for (int k = 0; k < TABLE_SLOTS && slot < 0; ++k) {
            const int c = (m->table_next + k) % TABLE_SLOTS;
            if (std::find(distinct.begin(), distinct.end(), m->table_sigma[c]) == distinct.end()) slot = c;
        }
        if (slot < 0) return ISR_ERR_ARG;   // cannot happen: fewer needed tables than slots
        m->table_next = (slot + 1) % TABLE_SLOTS;
        if (!build_device_table(s, m->htables[slot])) return ISR_ERR_ARG;
        m->staging_busy = true;
        HIP_TRY(hipMemcpyAsync(m->dtables + slot, m->htables + slot, sizeof(DeviceNoiseTable), hipMemcpyHostToDevice, m->stream));
        m->table_sigma[slot] = s;
    }
    slots.resize(sigmas.size());
    for (size_t i = 0; i < sigmas.size(); ++i)
        for (int k = 0; k < TABLE_SLOTS; ++k)
            if (m->table_sigma[k] == sigmas[i]) slots[i] = (uint32_t)k;
    return ISR_OK;
}

// Validates a batch, uploads its item descriptors and sees to clean vote counters.
int prepare_batch(isr_model *m, const void *x, uint32_t n_images, const isr_item *items, uint32_t n_items, double alpha) {
    if (!m || !x || !items || n_images == 0 || n_items == 0) return ISR_ERR_ARG;
    if (!(alpha > 0.0 && alpha < 1.0)) return ISR_ERR_ARG;
    if (!m->ws || m->chunk == 0) return ISR_ERR_WORKSPACE;
    std::vector<uint32_t> sigmas(n_items), slots;
    for (uint32_t i = 0; i < n_items; ++i) {
        if (items[i].image >= n_images || items[i].sigma < 1 || items[i].sigma > 1024) return ISR_ERR_ARG;
        sigmas[i] = items[i].sigma;
    }
    const size_t C = (size_t)m->pm.classes;
    if (n_items > m->items_cap) {
        HIP_TRY(hipStreamSynchronize(m->stream));
        if (m->ditems) (void)hipFree(m->ditems);
        if (m->hitems) (void)hipHostFree(m->hitems);
        if (m->dcounts_b) (void)hipFree(m->dcounts_b);
        if (m->hcounts_b) (void)hipHostFree(m->hcounts_b);
        m->ditems = m->hitems = nullptr;
        m->dcounts_b = m->hcounts_b = nullptr;
        m->items_cap = 0;
        const uint32_t cap = std::max<uint32_t>(n_items, 64);
        HIP_TRY(hipMalloc((void **)&m->ditems, sizeof(NoiseItem) * cap));
        HIP_TRY(hipHostMalloc((void **)&m->hitems, sizeof(NoiseItem) * cap, hipHostMallocDefault));
        HIP_TRY(hipMalloc((void **)&m->dcounts_b, sizeof(uint32_t) * 2 * cap * C));
        HIP_TRY(hipHostMalloc((void **)&m->hcounts_b, sizeof(uint32_t) * 2 * cap * C, hipHostMallocCoherent));
        HIP_TRY(hipHostGetDevicePointer((void **)&m->hcounts_b_dev, m->hcounts_b, 0));
        m->items_cap = cap;
        m->counts_b_clean = false;
    }
    int rc = free_staging(m);
    if (rc != ISR_OK || (rc = get_tables(m, sigmas, slots)) != ISR_OK) return rc;
    for (uint32_t i = 0; i < n_items; ++i) m->hitems[i] = NoiseItem{items[i].image, slots[i], items[i].image_id};
    m->staging_busy = true;
    HIP_TRY(hipMemcpyAsync(m->ditems, m->hitems, sizeof(NoiseItem) * n_items, hipMemcpyHostToDevice, m->stream));
    if (!m->counts_b_clean) HIP_TRY(launch_fill_u32(m->dcounts_b, 0, (size_t)2 * m->items_cap * C, m->stream));
    m->counts_b_clean = false;
    return open_call(m);
}

// The tallies of a batched call on the host, zeros on the device (as close_counts).
int finish_batch(isr_model *m, size_t words) {
    const int rc = publish(m, m->dcounts_b, m->hcounts_b, m->hcounts_b_dev, words);
    if (rc != ISR_OK) return rc;
    m->counts_b_clean = true;
    return ISR_OK;
}

int check_call(const isr_model *m, const void *x, uint32_t sigma, double alpha, bool need_alpha) {
    if (!m || !x) return ISR_ERR_ARG;
    if (sigma < 1 || sigma > 1024) return ISR_ERR_ARG;
    if (need_alpha && !(alpha > 0.0 && alpha < 1.0)) return ISR_ERR_ARG;
    if (!m->ws || m->chunk == 0) return ISR_ERR_WORKSPACE;
    return ISR_OK;
}

}  // namespace

extern "C" {

int isr_load_model(const void *blob_host, size_t bytes, isr_model **out) {
    if (!blob_host || !out) return ISR_ERR_ARG;
    *out = nullptr;
    isr_model *m = new (std::nothrow) isr_model();
    if (!m) return ISR_ERR_ARG;
    std::string why;
    int rc = parse_model(blob_host, bytes, m->pm, why);
    if (rc != ISR_OK) { delete m; return rc; }
    ConstArena arena;
    arena.put(nullptr, 256);  // offset 0 is never a valid table
    rc = build_device_ops(m->pm, m->ops, arena);
    if (rc != ISR_OK) { delete m; return rc; }
    auto cleanup = [&](int code) { isr_free_model(m); return code; };
    // one device allocation: [constants][room for those of the narrow-net ops][counters][noise tables], and one pinned one
    auto round_256 = [](size_t b) { return (b + 255) & ~(size_t)255; };
    const size_t narrow_off = round_256(arena.host.size()), counts_off = round_256(narrow_off + narrow_ops_room(m->ops));
    const size_t counts_bytes = sizeof(uint32_t) * 2 * m->pm.classes, parts_off = round_256(counts_off + counts_bytes);
    const size_t tables_off = round_256(parts_off + sizeof(TallyParts)), tables_bytes = round_256(sizeof(DeviceNoiseTable) * TABLE_SLOTS);
    hipError_t e = hipMalloc((void **)&m->dconst, tables_off + tables_bytes);
    const size_t flag_off = round_256(tables_bytes + counts_bytes);
    if (e == hipSuccess) e = hipHostMalloc((void **)&m->htables, flag_off + 64 + DIRECT_VOTES * 8, hipHostMallocCoherent);   // the host watches flag and votes while a kernel runs
    if (e == hipSuccess) {
        m->dtables = (DeviceNoiseTable *)(m->dconst + tables_off);
        m->dcounts = (uint32_t *)(m->dconst + counts_off);
        m->dparts = (TallyParts *)(m->dconst + parts_off);
        m->hcounts = (uint32_t *)((uint8_t *)m->htables + tables_bytes);
        m->hflag = (uint32_t *)((uint8_t *)m->htables + flag_off);
        *m->hflag = m->published;
        m->hvotes = (uint64_t *)((uint8_t *)m->htables + flag_off + 64);
        std::fill(m->hvotes, m->hvotes + DIRECT_VOTES, 0);
        e = hipHostGetDevicePointer((void **)&m->hcounts_dev, m->hcounts, 0);
        if (e == hipSuccess) e = hipHostGetDevicePointer((void **)&m->hflag_dev, m->hflag, 0);
        if (e == hipSuccess) e = hipHostGetDevicePointer((void **)&m->hvotes_dev, m->hvotes, 0);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&m->end, hipEventDisableTiming);
    }
    if (e != hipSuccess) { g_last_hip_error = (int)e; return cleanup(ISR_ERR_DEVICE); }
    rebase_device_ops(m->ops, m->dconst);
    m->plan[0].ops = m->ops;
    build_fused_plan(m->pm, m->ops, m->plan[1].ops, false);
    build_fused_plan(m->pm, m->ops, m->plan[2].ops, true);
    arena.host.resize(narrow_off);
    if ((rc = build_narrow_ops(m, arena, counts_off)) != ISR_OK) return cleanup(rc);
    arena.host.resize(tables_off);   // zeros in the counters
    m->counts_clean = m->parts_clean = true;
    e = hipMemcpy(m->dconst, arena.host.data(), arena.host.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) { g_last_hip_error = (int)e; return cleanup(ISR_ERR_DEVICE); }
    *out = m;
    return ISR_OK;
}

int isr_set_fusion(isr_model *m, int enable) {
    if (!m) return ISR_ERR_ARG;
    if (enable < 0 || enable > 2) return ISR_ERR_ARG;
    m->use_fused = enable;
    return ISR_OK;
}

int isr_noise_bank(uint32_t sigma, uint64_t seed, uint32_t bank_id, uint32_t first, uint32_t count, uint32_t d,
                   int16_t *out_device, void *hip_stream) {
    if (sigma < 1 || sigma > 1024 || !out_device || d == 0 || (d & 3) != 0) return ISR_ERR_ARG;
    if ((uint64_t)first + count > (1ull << 32)) return ISR_ERR_ARG;
    if (count == 0) return ISR_OK;
    hipStream_t st = (hipStream_t)hip_stream;
    BankTable t;
    hipError_t e = BankTables::all().take(sigma, t);
    if (e == hipSuccess && t.sigma != sigma) {
        std::vector<uint32_t> words;
        uint32_t n = 0;
        t.sigma = 0;
        if (!build_bank_table(sigma, words, n, t.R) || words.size() * 4 > BANK_TABLE_BYTES) {
            BankTables::all().give_back(t);
            return ISR_ERR_ARG;
        }
        t.words = words.size();
        bank_guide(words, t.R);
        std::memcpy(t.host, words.data(), t.words * 4);
        e = hipMemcpyAsync(t.dev, t.host, t.words * 4, hipMemcpyHostToDevice, st);
    }
    if (e == hipSuccess) {
        NoiseBankParams p;
        set_bank_table(p, t.dev, t.words, t.R);
        p.out = out_device; p.d = d;
        p.key0 = (uint32_t)seed; p.key1 = (uint32_t)(seed >> 32); p.bank = bank_id; p.first = first; p.count = count;
        e = launch_noise_bank(p, st);
    }
    const hipError_t done = hipStreamSynchronize(st);   // the table is handed back with this call
    if (e == hipSuccess) e = done;
    t.sigma = e == hipSuccess ? sigma : 0;
    BankTables::all().give_back(t);
    if (e != hipSuccess) { g_last_hip_error = (int)e; return ISR_ERR_DEVICE; }
    return ISR_OK;
}

int isr_set_conv_tile(isr_model *m, int tile) {
    if (!m || tile < 0 || tile > 7) return ISR_ERR_ARG;
    m->conv_tile = tile;
    return ISR_OK;
}

int isr_profile(isr_model *m, uint32_t every_chunks) {
    if (!m) return ISR_ERR_ARG;
    m->profile_every = every_chunks;
    m->chunk_counter = 0;
    m->stats.clear();
    return ISR_OK;
}

int isr_profile_read(const isr_model *m, isr_kernel_stat *out_host, uint32_t cap, uint32_t *n_out) {
    if (!m || !n_out || (cap && !out_host)) return ISR_ERR_ARG;
    uint32_t n = 0;
    for (const auto &kv : m->stats) {
        if (n < cap) out_host[n] = kv.second;
        ++n;
    }
    *n_out = n;
    return ISR_OK;
}

int isr_free_model(isr_model *m) {
    if (!m) return ISR_OK;
    for (hipEvent_t e : m->events) (void)hipEventDestroy(e);
    if (m->end) (void)hipEventDestroy(m->end);
    if (m->dconst) (void)hipFree(m->dconst);
    if (m->htables) (void)hipHostFree(m->htables);
    if (m->ditems) (void)hipFree(m->ditems);
    if (m->hitems) (void)hipHostFree(m->hitems);
    if (m->dcounts_b) (void)hipFree(m->dcounts_b);
    if (m->hcounts_b) (void)hipHostFree(m->hcounts_b);
    free_float_net(m->fnet);
    delete m;
    return ISR_OK;
}

int isr_model_info(const isr_model *m, int *C, int *H, int *W, int *num_classes) {
    if (!m) return ISR_ERR_ARG;
    if (C) *C = m->pm.C;
    if (H) *H = m->pm.H;
    if (W) *W = m->pm.W;
    if (num_classes) *num_classes = m->pm.classes;
    return ISR_OK;
}

size_t isr_workspace_bytes(const isr_model *m, uint32_t chunk_samples) {
    if (!m || chunk_samples == 0) return 0;
    size_t need = 0;
    for (int i = 0; i < 3; ++i) {
        Plan pl;
        pl.ops = m->plan[i].ops;
        if (i >= 1) plan_segments(m->pm, chunk_samples, pl);
        plan_workspace(m->pm, chunk_samples, pl);
        need = std::max(need, pl.bytes);
    }
    return need;
}

int isr_set_workspace(isr_model *m, void *workspace_device, size_t bytes, uint32_t chunk_samples, void *hip_stream) {
    if (!m || !workspace_device || chunk_samples == 0) return ISR_ERR_ARG;
    if ((uintptr_t)workspace_device % 256 != 0) return ISR_ERR_ARG;
    // pixel counts of a chunk are kept in 32 bits inside the kernels
    for (const TensorDesc &t : m->pm.tensors)
        if ((uint64_t)chunk_samples * t.H * t.W * std::max(t.Cp, 16) >= (1ull << 31)) return ISR_ERR_ARG;
    if (bytes < isr_workspace_bytes(m, chunk_samples)) return ISR_ERR_WORKSPACE;
    plan_segments(m->pm, chunk_samples, m->plan[1]);
    plan_segments(m->pm, chunk_samples, m->plan[2]);
    for (int i = 0; i < 3; ++i) plan_workspace(m->pm, i ? plan_copies(m->pm, chunk_samples, bytes, m->plan[i]) : chunk_samples, m->plan[i]);
    m->ws = (uint8_t *)workspace_device;
    m->ws_bytes = bytes;
    m->chunk = chunk_samples;
    m->stream = (hipStream_t)hip_stream;
    return ISR_OK;
}

int isr_certify(isr_model *m, const uint8_t *x_device, uint32_t sigma, uint32_t n0, uint32_t n, double alpha,
                uint64_t seed, uint32_t image_id, isr_result *out, uint32_t *counts0_host, uint32_t *counts1_host) {
    int rc = check_call(m, x_device, sigma, alpha, true);
    if (rc != ISR_OK) return rc;
    if (!out || n0 == 0 || n == 0) return ISR_ERR_ARG;
    const uint32_t C = (uint32_t)m->pm.classes;
    const DeviceNoiseTable *table = nullptr;
    if ((rc = get_table(m, sigma, &table)) != ISR_OK) return rc;
    if ((rc = open_counts(m)) != ISR_OK) return rc;
    const Draw draw{x_device, table, nullptr, seed, image_id, Slots{0, n0, {n0, n}, 1, 0, 0}};
    if ((rc = run_slots(m, m->plan[m->use_fused], draw, nullptr, nullptr, m->dcounts, -1)) != ISR_OK) return rc;
    if ((rc = close_counts(m, 2)) != ISR_OK) return rc;
    if (counts0_host) std::memcpy(counts0_host, m->hcounts, sizeof(uint32_t) * C);
    if (counts1_host) std::memcpy(counts1_host, m->hcounts + C, sizeof(uint32_t) * C);
    return isr_decide_certify(m->hcounts, m->hcounts + C, C, (double)sigma, n, alpha, out);
}

int isr_predict(isr_model *m, const uint8_t *x_device, uint32_t sigma, uint32_t n, double alpha, uint64_t seed,
                uint32_t image_id, isr_result *out, uint32_t *counts_host) {
    int rc = check_call(m, x_device, sigma, alpha, true);
    if (rc != ISR_OK) return rc;
    if (!out || n == 0) return ISR_ERR_ARG;
    const uint32_t C = (uint32_t)m->pm.classes;
    const DeviceNoiseTable *table = nullptr;
    if ((rc = get_table(m, sigma, &table)) != ISR_OK) return rc;
    if ((rc = open_counts(m)) != ISR_OK) return rc;
    const Draw draw{x_device, table, nullptr, seed, image_id, one_phase(0, 0, n)};
    if ((rc = run_slots(m, m->plan[m->use_fused], draw, nullptr, nullptr, m->dcounts, -1)) != ISR_OK) return rc;
    if ((rc = close_counts(m, 1)) != ISR_OK) return rc;
    if (counts_host) std::memcpy(counts_host, m->hcounts, sizeof(uint32_t) * C);
    return isr_decide_predict(m->hcounts, C, alpha, out);
}

int isr_certify_batch(isr_model *m, const uint8_t *x_device, uint32_t n_images, const isr_item *items_host,
                      uint32_t n_items, uint32_t n0, uint32_t n, double alpha, uint64_t seed, isr_result *out_host,
                      uint32_t *counts0_host, uint32_t *counts1_host) {
    if (!out_host || n0 == 0 || n == 0) return ISR_ERR_ARG;
    int rc = prepare_batch(m, x_device, n_images, items_host, n_items, alpha);
    if (rc != ISR_OK) return rc;
    const size_t C = (size_t)m->pm.classes, per_phase = (size_t)n_items * C;
    const Draw draw{x_device, m->dtables, m->ditems, seed, 0, Slots{0, (uint64_t)n_items * n0, {n0, n}, n_items, 0, 0}};
    if ((rc = run_slots(m, m->plan[m->use_fused], draw, nullptr, nullptr, m->dcounts_b, -1)) != ISR_OK) return rc;
    if ((rc = finish_batch(m, 2 * per_phase)) != ISR_OK) return rc;
    if (counts0_host) std::memcpy(counts0_host, m->hcounts_b, sizeof(uint32_t) * per_phase);
    if (counts1_host) std::memcpy(counts1_host, m->hcounts_b + per_phase, sizeof(uint32_t) * per_phase);
    for (uint32_t i = 0; i < n_items; ++i) {
        rc = isr_decide_certify(m->hcounts_b + i * C, m->hcounts_b + per_phase + i * C, (uint32_t)C, (double)items_host[i].sigma, n,
                                alpha, out_host + i);
        if (rc != ISR_OK) return rc;
    }
    return ISR_OK;
}

int isr_predict_batch(isr_model *m, const uint8_t *x_device, uint32_t n_images, const isr_item *items_host,
                      uint32_t n_items, uint32_t n, double alpha, uint64_t seed, isr_result *out_host,
                      uint32_t *counts_host) {
    if (!out_host || n == 0) return ISR_ERR_ARG;
    int rc = prepare_batch(m, x_device, n_images, items_host, n_items, alpha);
    if (rc != ISR_OK) return rc;
    const size_t C = (size_t)m->pm.classes, per_phase = (size_t)n_items * C;
    const Draw draw{x_device, m->dtables, m->ditems, seed, 0, Slots{0, (uint64_t)n_items * n, {n, 0}, n_items, 0, 0}};
    if ((rc = run_slots(m, m->plan[m->use_fused], draw, nullptr, nullptr, m->dcounts_b, -1)) != ISR_OK) return rc;
    if ((rc = finish_batch(m, per_phase)) != ISR_OK) return rc;
    if (counts_host) std::memcpy(counts_host, m->hcounts_b, sizeof(uint32_t) * per_phase);
    for (uint32_t i = 0; i < n_items; ++i) {
        rc = isr_decide_predict(m->hcounts_b + i * C, (uint32_t)C, alpha, out_host + i);
        if (rc != ISR_OK) return rc;
    }
    return ISR_OK;
}

int isr_debug_noisy(isr_model *m, const uint8_t *x_device, uint32_t sigma, uint64_t seed, uint32_t image_id,
                    uint32_t phase, uint32_t sample_begin, uint32_t count, int8_t *out_host) {
    int rc = check_call(m, x_device, sigma, 0.5, false);
    if (rc != ISR_OK) return rc;
    if (!out_host || count == 0 || count > m->chunk || phase > 1) return ISR_ERR_ARG;
    const DeviceNoiseTable *table = nullptr;
    if ((rc = get_table(m, sigma, &table)) != ISR_OK) return rc;
    if ((rc = run_slots(m, m->plan[m->use_fused], Draw{x_device, table, nullptr, seed, image_id, one_phase(phase, sample_begin, count)}, nullptr, nullptr, nullptr, 0)) != ISR_OK) return rc;
    const ParsedModel &pm = m->pm;
    const size_t hw = (size_t)pm.H * pm.W;
    std::vector<int8_t> tmp(count * hw * 4);
    HIP_TRY(hipMemcpyAsync(tmp.data(), m->ws + m->plan[m->use_fused].toff[0], tmp.size(), hipMemcpyDeviceToHost, m->stream));
    HIP_TRY(hipStreamSynchronize(m->stream));
    for (uint32_t s = 0; s < count; ++s)
        for (int c = 0; c < pm.C; ++c)
            for (size_t i = 0; i < hw; ++i) out_host[((size_t)s * pm.C + c) * hw + i] = tmp[((size_t)s * hw + i) * 4 + c];
    return ISR_OK;
}

int isr_debug_forward(isr_model *m, const uint8_t *x_device, uint32_t sigma, uint64_t seed, uint32_t image_id,
                      uint32_t phase, uint32_t sample_begin, uint32_t count, int32_t *logits_host,
                      int32_t *argmax_host, uint32_t *counts_host) {
    int rc = check_call(m, x_device, sigma, 0.5, false);
    if (rc != ISR_OK) return rc;
    if (count == 0 || phase > 1) return ISR_ERR_ARG;
    const uint32_t C = (uint32_t)m->pm.classes;
    const DeviceNoiseTable *table = nullptr;
    if ((rc = get_table(m, sigma, &table)) != ISR_OK) return rc;
    if (counts_host && (rc = open_counts(m)) != ISR_OK) return rc;
    const Draw draw{x_device, table, nullptr, seed, image_id, one_phase(phase, sample_begin, count)};
    rc = run_slots(m, m->plan[m->use_fused], draw, logits_host, argmax_host, counts_host ? m->dcounts : nullptr, -1);
    if (rc != ISR_OK) return rc;
    if (counts_host) {
        if ((rc = close_counts(m, 1)) != ISR_OK) return rc;
        for (uint32_t i = 0; i < C; ++i) counts_host[i] += m->hcounts[i];
    } else {
        HIP_TRY(hipStreamSynchronize(m->stream));
    }
    return ISR_OK;
}

int isr_debug_tensor(isr_model *m, const uint8_t *x_device, uint32_t sigma, uint64_t seed, uint32_t image_id,
                     uint32_t phase, uint32_t sample, int32_t tensor_id, int8_t *out_host) {
    int rc = check_call(m, x_device, sigma, 0.5, false);
    if (rc != ISR_OK) return rc;
    const ParsedModel &pm = m->pm;
    if (!out_host || phase > 1 || tensor_id < 0 || tensor_id >= (int)pm.tensors.size() || tensor_id == pm.ops.back().out)
        return ISR_ERR_ARG;
    const DeviceNoiseTable *table = nullptr;
    if ((rc = get_table(m, sigma, &table)) != ISR_OK) return rc;
    // tensors that the fused plan never materialises come from the op-by-op plan
    const Plan &pl = (m->use_fused && m->plan[m->use_fused].has[tensor_id]) ? m->plan[m->use_fused] : m->plan[0];
    if ((rc = run_slots(m, pl, Draw{x_device, table, nullptr, seed, image_id, one_phase(phase, sample, 1)}, nullptr, nullptr, nullptr, tensor_id)) != ISR_OK) return rc;
    const TensorDesc &t = pm.tensors[tensor_id];
    const size_t hw = (size_t)t.H * t.W;
    std::vector<int8_t> tmp(hw * t.Cp);
    HIP_TRY(hipMemcpyAsync(tmp.data(), m->ws + pl.toff[tensor_id], tmp.size(), hipMemcpyDeviceToHost, m->stream));
    HIP_TRY(hipStreamSynchronize(m->stream));
    for (int c = 0; c < t.C; ++c)
        for (size_t i = 0; i < hw; ++i) out_host[(size_t)c * hw + i] = tmp[i * t.Cp + c];
    return ISR_OK;
}

int isr_debug_tensor_source(const isr_model *m, int32_t tensor_id, int *from_fused_out) {
    if (!m || !from_fused_out || tensor_id < 0 || tensor_id >= (int)m->pm.tensors.size()) return ISR_ERR_ARG;
    if (m->plan[1].has.empty()) return ISR_ERR_WORKSPACE;   // plans are placed by isr_set_workspace
    *from_fused_out = (m->use_fused && m->plan[m->use_fused].has[tensor_id]) ? 1 : 0;
    return ISR_OK;
}

const char *isr_strerror(int status) {
    switch (status) {
    case ISR_OK: return "ok";
    case ISR_ERR_ARG: return "invalid argument";
    case ISR_ERR_FORMAT: return "malformed model blob";
    case ISR_ERR_UNSUPPORTED: return "model uses a shape or op the kernels do not cover";
    case ISR_ERR_WORKSPACE: return "workspace missing or too small";
    case ISR_ERR_DEVICE: return "HIP call failed";
    default: return "unknown status";
    }
}

int isr_last_device_error(void) { return g_last_hip_error; }

}  // extern "C"
