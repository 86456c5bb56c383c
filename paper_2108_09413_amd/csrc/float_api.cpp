// C ABI of the two floating-point comparison systems of the paper's evaluation (section "Experiments"):
// FloatRS-quant -- continuous Gaussian noise rounded back onto the pixel grid, then the int8 network
// (the integer path's loop with another input stage, api.cpp) -- and FloatRS-fp -- continuous Gaussian
// noise, then the fp32 network derived from the quantized one: every tensor holds the real values
// r = q - z behind the int8 codes and every op is the quantized op without its rounding and without
// the saturation at the ends of the int8 range.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "isr_internal.h"
#include "model.h"

using namespace isr;

#define HIP_TRY(expr)                                     \
    do {                                                  \
        hipError_t e_ = (expr);                           \
        if (e_ != hipSuccess) {                           \
            set_last_device_error((int)e_);               \
            return ISR_ERR_DEVICE;                        \
        }                                                 \
    } while (0)

namespace isr {

struct FloatOp {
    OpType type;
    int a = -1, b = -1, out = -1;
    FConvParams conv{};            // CONV and FC (an FC layer is a convolution over the whole input)
    int res = -1;                  // tensor read by the residual add folded into the convolution, or -1
    int pair = -1;                 // the op before, whose result is that tensor, runs in this op's kernel: its input tensor
    int paired = 0;                // this op runs in the next one's kernel (alone only where its own result is asked for)
    int next = 0;                  // the next op, which reads this one's result, can run in this op's kernel
    float ma = 0.f, mb = 0.f;      // ADD
    int relu = 0;
    FPoolParams pool{};
    float gap_scale = 0.f;
    double flops = 0.0, bytes = 0.0;   // per copy: 2 per multiply-accumulate on real channels; fp32 bytes in + out
};

// Ops that run in the kernel of the op before: none, poolings (of first layers), readers of sums as well.
enum FloatJoin { JOIN_NONE, JOIN_POOLS, JOIN_ALL };

struct FloatNet {
    std::vector<FloatOp> ops;
    // tensor placement: the ops' tensor ids with the int8 planner, whose bytes for B copies hold B / 4 fp32 copies; `merged` with the
    // results of ops that can run in one kernel placed together, which can take more: of as many kinds of them as the workspace has room for
    Plan plan, merged;
    FloatJoin joins = JOIN_NONE;   // of `merged`
    uint32_t planned_chunk = 0;
    size_t planned_bytes = 0;      // of the workspace that `merged` is for
    uint8_t *dconst = nullptr;
    int status = ISR_OK;           // ISR_ERR_UNSUPPORTED when an op has no float kernel
};

void free_float_net(FloatNet *net) {
    if (!net) return;
    if (net->dconst) (void)hipFree(net->dconst);
    delete net;
}

}  // namespace isr

namespace {

// MFMA 32x32 accumulator: register i of lane half h is row 8 (i / 4) + 4 h + i % 4; the weights of
// channel 16 h + i go to that row so that a lane ends up with 16 consecutive channels.
int mfma_row_of_channel(int c) {
    const int h = c >> 4, a = (c & 15) >> 2, b = c & 3;
    return 8 * a + 4 * h + b;
}

// the upper half of the fp32 number: exact for whole numbers of at most 8 bits
uint16_t bf16_of_int(int v) {
    const float f = (float)v;
    uint32_t bits;
    std::memcpy(&bits, &f, 4);
    return (uint16_t)(bits >> 16);
}

size_t put(std::vector<uint8_t> &arena, const void *src, size_t bytes) {
    const size_t off = (arena.size() + 255) & ~(size_t)255;
    arena.resize(off + bytes);
    std::memcpy(arena.data() + off, src, bytes);
    return off;
}

// Weights, per-channel constants and the K table of one convolution (k x k taps over a [H][W][Cin_p] input).  Every other
// channel is computed with its sign reversed (weights, bias and scale negated: the same numbers), beginning with channel
// `first_negated`: the matrix unit's sums are a little too low on average (float_path.hip).
int build_conv(const ParsedModel &pm, const HostOp &o, int k, int stride, int pad, bool fc, int first_negated,
               std::vector<uint8_t> &arena, FloatOp &f) {
    const TensorDesc &ti = pm.tensors[o.a], &to = pm.tensors[o.out];
    if (k > 127) return ISR_ERR_UNSUPPORTED;
    FConvParams &c = f.conv;
    c.H = ti.H; c.W = ti.W; c.Cin_p = ti.Cp; c.Ho = to.H; c.Wo = to.W; c.Cout_p = to.Cp;
    const int bm = fconv_tile_m(c.Cout_p);
    c.Cout_pp = (c.Cout_p + bm - 1) / bm * bm;
    c.k = k; c.stride = stride; c.pad = pad;
    // quads of K of a kernel row; the 7x7 layers on images leave the last of eight empty (fstem_pool_kernel reads pairs of pixels)
    const int row_quads = k * ti.Cp / 4 + (k == 7 && ti.Cp == 4 ? 1 : 0), kq_real = k * row_quads;
    c.Kq = (kq_real + 7) & ~7;
    c.relu = fc ? 0 : o.relu;
    std::vector<uint16_t> w((size_t)c.Kq * c.Cout_pp * 4, 0);
    std::vector<float> bias(c.Cout_pp, 0.f), scale(c.Cout_pp, 0.f);
    std::vector<int32_t> ktab(c.Kq, -1);
    for (int kq = 0; kq < kq_real; ++kq) {
        const int kx = kq % row_quads * 4 / ti.Cp, coff = kq % row_quads * 4 % ti.Cp;
        if (kx < k) ktab[kq] = ((kq / row_quads) << 24) | (kx << 16) | coff;
    }
    std::vector<uint32_t> first_k(k * k);   // place in K of a tap's first channel
    for (int t = 0; t < k * k; ++t) first_k[t] = (uint32_t)(t / k * row_quads * 4 + t % k * ti.Cp);
    for (int oc = 0; oc < to.C; ++oc) {
        const int row = (oc / 32) * 32 + mfma_row_of_channel(oc % 32);
        const int sign = (oc ^ first_negated) & 1 ? 1 : -1;
        for (int ic = 0; ic < ti.C; ++ic)
            for (int t = 0; t < k * k; ++t) {
                const uint32_t kidx = first_k[t] + (uint32_t)ic;
                w[((size_t)(kidx / 32) * c.Cout_pp + row) * 32 + kidx % 32] = bf16_of_int(sign * o.w[((size_t)oc * ti.C + ic) * k * k + t]);
            }
        bias[oc] = (float)sign * (float)o.bias[oc];
        scale[oc] = (float)sign * (fc ? 1.f : (float)std::ldexp((double)o.M0[oc], -(31 + o.shift[oc])));
    }
    // offsets now, pointers after the upload
    c.w = (const uint16_t *)put(arena, w.data(), w.size() * 2);
    c.bias = (const float *)put(arena, bias.data(), bias.size() * 4);
    c.scale = (const float *)put(arena, scale.data(), scale.size() * 4);
    c.ktab = (const int32_t *)put(arena, ktab.data(), ktab.size() * 4);
    f.flops = 2.0 * to.C * to.H * to.W * ti.C * k * k;
    f.bytes = 4.0 * ((double)ti.C * ti.H * ti.W + (double)to.C * to.H * to.W);
    return ISR_OK;
}

int build_float_net(isr_model *m) {
    if (m->fnet) return m->fnet->status;
    FloatNet *net = new FloatNet();
    m->fnet = net;
    const ParsedModel &pm = m->pm;
    std::vector<int> uses(pm.tensors.size(), 0);
    for (const HostOp &o : pm.ops) {
        if (o.a >= 0) uses[o.a]++;
        if (o.b >= 0) uses[o.b]++;
    }
    std::vector<uint8_t> arena(256, 0);
    int adds = 0;   // the channels with reversed sign change from one residual block to the next
    for (const HostOp &o : pm.ops) {
        FloatOp f;
        f.type = o.type; f.a = o.a; f.b = o.b; f.out = o.out;
        const TensorDesc &ti = pm.tensors[o.a], &to = pm.tensors[o.out];
        switch (o.type) {
        case OP_CONV:
            if ((net->status = build_conv(pm, o, o.k, o.stride, o.pad, false, adds & 1, arena, f)) != ISR_OK) return net->status;
            break;
        case OP_FC:
            if (ti.H != ti.W) return net->status = ISR_ERR_UNSUPPORTED;
            if ((net->status = build_conv(pm, o, ti.H, 1, 0, true, adds & 1, arena, f)) != ISR_OK) return net->status;
            break;
        case OP_ADD: {
            ++adds;
            f.ma = (float)std::ldexp((double)o.Ma, -o.sh);
            f.mb = (float)std::ldexp((double)o.Mb, -o.sh);
            f.relu = o.relu;
            f.bytes = 12.0 * to.C * to.H * to.W;
            // the convolution issued right before, read by this add alone: the add moves into its epilogue
            FloatOp *prev = net->ops.empty() ? nullptr : &net->ops.back();
            if (prev && prev->type == OP_CONV && prev->res < 0 && o.a != o.b && (prev->out == o.a || prev->out == o.b) &&
                uses[prev->out] == 1) {
                const bool conv_is_a = prev->out == o.a;
                prev->res = conv_is_a ? o.b : o.a;
                prev->conv.ma = conv_is_a ? f.ma : f.mb;
                prev->conv.mb = conv_is_a ? f.mb : f.ma;
                prev->conv.add_relu = o.relu;
                prev->out = o.out;
                prev->bytes += 4.0 * to.C * to.H * to.W;
                continue;
            }
            break; }
        case OP_MAXPOOL:
            f.pool.H = ti.H; f.pool.W = ti.W; f.pool.Cp = ti.Cp; f.pool.Ho = to.H; f.pool.Wo = to.W;
            f.pool.k = o.k; f.pool.stride = o.stride; f.pool.pad = o.pad;
            f.bytes = 4.0 * ((double)ti.C * ti.H * ti.W + (double)to.C * to.H * to.W);
            break;
        case OP_GAP:
            f.gap_scale = (float)std::ldexp((double)o.Ma, -(31 + o.sh));
            f.bytes = 4.0 * ((double)ti.C * ti.H * ti.W + to.C);
            break;
        }
        net->ops.push_back(f);
    }
    hipError_t e = hipMalloc((void **)&net->dconst, arena.size());
    if (e == hipSuccess) e = hipMemcpy(net->dconst, arena.data(), arena.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) { set_last_device_error((int)e); return net->status = ISR_ERR_DEVICE; }
    for (FloatOp &f : net->ops)
        if (f.type == OP_CONV || f.type == OP_FC) {
            FConvParams &c = f.conv;
            c.w = (const uint16_t *)(net->dconst + (size_t)c.w);
            c.zeros = (const float *)net->dconst;   // the arena starts with 256 zero bytes
            c.bias = (const float *)(net->dconst + (size_t)c.bias);
            c.scale = (const float *)(net->dconst + (size_t)c.scale);
            c.ktab = (const int32_t *)(net->dconst + (size_t)c.ktab);
        }
    // the residual of a folded add that the convolution before computes for it alone: both in one kernel
    for (size_t i = 1; i < net->ops.size(); ++i) {
        FloatOp &f = net->ops[i], &q = net->ops[i - 1];
        if (f.type != OP_CONV || q.type != OP_CONV || f.res < 0 || f.res != q.out || q.res >= 0 || uses[q.out] != 1 || f.a == q.out ||
            !fconv_pair_supported(f.conv, q.conv))
            continue;
        f.pair = q.a;
        q.paired = 1;
        f.flops += q.flops;
        f.bytes += q.bytes - 8.0 * f.conv.Ho * f.conv.Wo * pm.tensors[f.out].C;   // the residual is neither written nor read
        FConvParams &c = f.conv;
        c.w2 = q.conv.w; c.bias2 = q.conv.bias; c.scale2 = q.conv.scale;
        c.H2 = q.conv.H; c.W2 = q.conv.W; c.Cin2_p = q.conv.Cin_p; c.stride2 = q.conv.stride; c.relu2 = q.conv.relu;
    }
    // a closing convolution with its add and the convolution issued next, which reads the sum: one kernel writes both results
    for (size_t i = 0; i + 1 < net->ops.size(); ++i) {
        FloatOp &f = net->ops[i], &g = net->ops[i + 1];
        if (f.type == OP_CONV && g.type == OP_MAXPOOL) {   // a first layer and its pooling, which alone reads it: its result is not stored
            f.next = f.res < 0 && g.a == f.out && uses[f.out] == 1 && fstem_pool_supported(f.conv, g.pool);
            continue;
        }
        f.next = f.type == OP_CONV && g.type == OP_CONV && f.res >= 0 && !f.paired && g.a == f.out && g.res < 0 && g.pair < 0 && !g.paired &&
                 fexpand_supported(f.conv, g.conv);
    }
    return net->status = ISR_OK;
}

// Whether op i + 1 of the net is one of those.
bool float_joined(const FloatNet &net, size_t i, FloatJoin joins) {
    return net.ops[i].next && joins >= (net.ops[i + 1].type == OP_MAXPOOL ? JOIN_POOLS : JOIN_ALL);
}

// Places the float network's tensors for chunks of so many int8-sized copies (a quarter as many fp32 copies), the results of joined ops together.
void place_float_net(const isr_model *m, uint32_t chunk_samples, FloatJoin joins, Plan &pl) {
    const FloatNet &net = *m->fnet;
    pl.ops.clear();
    for (size_t i = 0; i < net.ops.size(); ++i) {   // what the planner looks at: op type and tensor ids
        const FloatOp &f = net.ops[i];
        if (f.paired) continue;
        if (i && float_joined(net, i - 1, joins)) {
            DevOp &both = pl.ops.back();
            (f.type == OP_MAXPOOL ? both.out : both.out2) = f.out;
            continue;
        }
        DevOp d{};
        d.type = f.type; d.a = f.a; d.b = f.pair >= 0 ? f.pair : f.res >= 0 ? f.res : f.b; d.out = f.out;
        pl.ops.push_back(d);
    }
    plan_workspace(m->pm, chunk_samples, pl);
    // a result that is stored only where it is asked for lies where the op that else computes it will put its own
    for (const FloatOp &f : net.ops)
        if (f.pair >= 0) { pl.toff[f.res] = pl.toff[f.out]; pl.has[f.res] = 1; }
}

// Both placements for a workspace of `bytes`, which hold the one op by op.  A first layer with its pooling adds its products in another
// order than the two apart, so isr_float_workspace_bytes asks for the room that they take; what reads a sum is joined where there
// is more, with the same bits.
void plan_float_net(isr_model *m, uint32_t chunk_samples, size_t bytes) {
    FloatNet &net = *m->fnet;
    if (net.planned_chunk == chunk_samples && net.planned_bytes == bytes) return;
    place_float_net(m, chunk_samples, JOIN_NONE, net.plan);
    for (FloatJoin joins : {JOIN_ALL, JOIN_POOLS, JOIN_NONE}) {
        net.joins = joins;
        place_float_net(m, chunk_samples, joins, net.merged);
        if (net.merged.bytes <= bytes) break;
    }
    net.planned_chunk = chunk_samples;
    net.planned_bytes = bytes;
}

// The placement for forwards that end at `stop_tensor` (-1: at the votes): `merged` unless it has no place for that tensor.
const Plan &float_plan(const isr_model *m, int stop_tensor) {
    const FloatNet &net = *m->fnet;
    return stop_tensor < 0 || net.merged.has[stop_tensor] ? net.merged : net.plan;
}

// Copies per chunk of the fp32 network: tensors sit at the offsets of the op-by-op int8 plan, four
// bytes per element, so a quarter of the int8 chunk fits (less when the padded logits need more).
uint32_t float_chunk(const isr_model *m) {
    const TensorDesc &tl = m->pm.tensors[m->pm.ops.back().out];
    const uint64_t by_logits = (uint64_t)m->chunk * m->pm.classes / (uint64_t)tl.Cp;
    return (uint32_t)std::min<uint64_t>(m->chunk / 4, by_logits);
}

// The Monte-Carlo loop of FloatRS-fp over sample indices [begin, begin + count) of one phase.
// raw_noise: stop after the noise stage and leave x + sigma z itself (not recentred) in tensor 0;
// stop_tensor >= 0 ends each forward right after the op that writes that tensor (0: after the noise stage).
int run_fp_range(isr_model *m, const uint8_t *x, float sigma, uint64_t seed, uint32_t image, uint32_t phase, uint32_t begin,
                 uint64_t count, float *logits_host, int32_t *argmax_host, uint32_t *dcounts, bool raw_noise, int stop_tensor = -1) {
    const ParsedModel &pm = m->pm;
    const FloatNet &net = *m->fnet;
    const Plan &pl = float_plan(m, stop_tensor);
    const bool merged = &pl == &net.merged;
    const uint32_t chunk = float_chunk(m);
    if (chunk == 0) return ISR_ERR_WORKSPACE;
    auto tptr = [&](int t) { return (float *)(m->ws + pl.toff[t]); };
    const TensorDesc &tl = pm.tensors[pm.ops.back().out];
    float *dlogits = (float *)(m->ws + pl.logits_off);
    int32_t *dargmax = (int32_t *)(m->ws + pl.argmax_off);
    std::vector<float> stage;
    for (uint64_t done = 0; done < count;) {
        const uint32_t bn = (uint32_t)std::min<uint64_t>(chunk, count - done);
        const bool timed = m->profile_every && (m->chunk_counter++ % m->profile_every) == 0;
        size_t ev = 0;
        struct Work { const char *kernel; int conv; double ops, bytes; };
        std::vector<Work> work;
        auto mark = [&]() -> int {
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
        int rc;
        if ((rc = mark()) != ISR_OK) return rc;
        FloatNoiseParams np{};
        np.x = x; np.out = tptr(0); np.C = pm.C; np.H = pm.H; np.W = pm.W;
        np.key0 = (uint32_t)seed; np.key1 = (uint32_t)(seed >> 32); np.image = image; np.phase = phase;
        np.sample_begin = begin + (uint32_t)done; np.count = bn; np.sigma = sigma;
        np.center = raw_noise ? 0.f : 128.f + (float)pm.tensors[0].zp;
        np.quant = 0;
        HIP_TRY(launch_float_noise(np, m->stream));
        work.push_back({last_kernel_name(), 0, 0.0, (double)bn * pm.H * pm.W * 16});
        // what runs in one kernel, for this number of pixels: op i with the one after it, and with the one before it
        auto expand_runs = [&](size_t i) {
            FConvParams c = net.ops[i].conv;
            c.npix = (int32_t)(bn * c.Ho * c.Wo);
            return merged && float_joined(net, i, net.joins) && net.ops[i].out != stop_tensor && fexpand_wanted(c, net.ops[i + 1].conv);
        };
        auto pair_runs = [&](size_t i) {
            FConvParams c = net.ops[i].conv;
            c.npix = (int32_t)(bn * c.Ho * c.Wo);
            return fconv_pair_wanted(c) || expand_runs(i);
        };
        bool whole = !raw_noise && stop_tensor != 0;
        if (whole) {
            for (size_t i = 0; i < net.ops.size(); ++i) {
                const FloatOp &f = net.ops[i];
                if (f.paired && f.out != stop_tensor && pair_runs(i + 1)) continue;
                if ((rc = mark()) != ISR_OK) return rc;
                const TensorDesc &ti = pm.tensors[f.a], &to = pm.tensors[f.out];
                const FloatOp *last = &f;   // of this launch
                switch (f.type) {
                case OP_CONV:
                case OP_FC: {
                    FConvParams c = f.conv;
                    c.in = tptr(f.a);
                    c.out = f.type == OP_FC ? dlogits : tptr(f.out);
                    if (f.pair >= 0 && pair_runs(i)) c.in2 = tptr(f.pair);
                    else c.res = f.res >= 0 ? tptr(f.res) : nullptr;
                    c.npix = (int32_t)(bn * c.Ho * c.Wo);
                    if (merged && float_joined(net, i, net.joins) && net.ops[i + 1].type == OP_MAXPOOL) {
                        const FloatOp &g = net.ops[++i];
                        FPoolParams q = g.pool;
                        q.out = tptr(g.out); q.B = (int32_t)bn;
                        HIP_TRY(launch_fstem_pool(c, q, m->stream));
                        last = &g;
                        break;
                    }
                    if (expand_runs(i)) {
                        const FloatOp &g = net.ops[++i];
                        FConvParams r = g.conv;
                        r.out = tptr(g.out);
                        HIP_TRY(launch_fexpand(c, r, m->stream));
                        last = &g;
                        break;
                    }
                    HIP_TRY(launch_fconv(c, m->stream));
                    break; }
                case OP_ADD: {
                    FAddParams a{tptr(f.a), tptr(f.b), tptr(f.out), f.ma, f.mb, f.relu, (int64_t)bn * to.H * to.W * to.Cp / 4};
                    HIP_TRY(launch_fadd(a, m->stream));
                    break; }
                case OP_MAXPOOL: {
                    FPoolParams q = f.pool;
                    q.in = tptr(f.a); q.out = tptr(f.out); q.B = (int32_t)bn;
                    HIP_TRY(launch_fmaxpool(q, m->stream));
                    break; }
                case OP_GAP: {
                    FGapParams g{tptr(f.a), tptr(f.out), ti.H * ti.W, ti.Cp, (int32_t)bn, f.gap_scale};
                    HIP_TRY(launch_fgap(g, m->stream));
                    break; }
                }
                work.push_back({last_kernel_name(), f.type == OP_CONV || f.type == OP_FC, f.flops * bn, f.bytes * bn});
                if (f.pair >= 0 && !pair_runs(i)) {   // the op's own part of the pair, which reads the residual
                    work.back().ops -= net.ops[i - 1].flops * bn;
                    work.back().bytes -= (net.ops[i - 1].bytes - 8.0 * to.C * to.H * to.W) * bn;
                }
                if (last != &f) {   // what lies between the two is not read back, and stored only if it is a sum
                    const double between = 4.0 * to.C * to.H * to.W;
                    work.back().ops += last->flops * bn;
                    work.back().bytes += (last->bytes - (last->type == OP_MAXPOOL ? 2.0 : 1.0) * between) * bn;
                }
                if (last->out == stop_tensor) { whole = false; break; }
            }
        }
        if (whole) {
            if ((rc = mark()) != ISR_OK) return rc;
            FVoteParams v{dlogits, pm.classes, tl.Cp, (int32_t)bn, dargmax, dcounts};
            HIP_TRY(launch_fvote(v, m->stream));
            work.push_back({last_kernel_name(), 0, 0.0, (double)bn * pm.classes * 4});
        }
        if (timed) {
            if ((rc = mark()) != ISR_OK) return rc;
            HIP_TRY(hipStreamSynchronize(m->stream));
            for (size_t i = 0; i + 1 < ev && i < work.size(); ++i) {
                float ms = 0.f;
                HIP_TRY(hipEventElapsedTime(&ms, m->events[i], m->events[i + 1]));
                isr_kernel_stat &st = m->stats[work[i].kernel];
                if (st.launches == 0) {
                    std::strncpy(st.name, work[i].kernel, sizeof(st.name) - 1);
                    st.is_conv = work[i].conv;
                }
                st.launches += 1;
                st.total_ms += ms;
                st.alg_ops += work[i].ops;
                st.alg_bytes += work[i].bytes;
            }
        }
        if (logits_host) {   // device rows are padded to the stored channel count
            stage.resize((size_t)bn * tl.Cp);
            HIP_TRY(hipMemcpyAsync(stage.data(), dlogits, stage.size() * 4, hipMemcpyDeviceToHost, m->stream));
            HIP_TRY(hipStreamSynchronize(m->stream));
            for (uint32_t s = 0; s < bn; ++s)
                std::memcpy(logits_host + (done + s) * pm.classes, stage.data() + (size_t)s * tl.Cp, (size_t)pm.classes * 4);
        }
        if (argmax_host) {
            HIP_TRY(hipMemcpyAsync(argmax_host + done, dargmax, (size_t)bn * 4, hipMemcpyDeviceToHost, m->stream));
            HIP_TRY(hipStreamSynchronize(m->stream));
        }
        done += bn;
    }
    return ISR_OK;
}

int check_float_call(isr_model *m, const void *x, float sigma, int system) {
    if (!m || !x) return ISR_ERR_ARG;
    if (system != ISR_FLOATRS_QUANT && system != ISR_FLOATRS_FP) return ISR_ERR_ARG;
    if (!(sigma >= 0.f) || !(sigma <= 4096.f)) return ISR_ERR_ARG;
    if (!m->ws || m->chunk == 0) return ISR_ERR_WORKSPACE;
    if (system == ISR_FLOATRS_FP) {
        const int rc = build_float_net(m);
        if (rc != ISR_OK) return rc;
        plan_float_net(m, m->chunk, m->ws_bytes);
        if (float_chunk(m) == 0 || m->fnet->plan.bytes > m->ws_bytes) return ISR_ERR_WORKSPACE;
    }
    return ISR_OK;
}

int run_system(isr_model *m, const uint8_t *x, float sigma, uint64_t seed, uint32_t image, uint32_t phase, uint32_t begin,
               uint64_t count, int system, void *logits_host, int32_t *argmax_host, uint32_t *dcounts) {
    if (system == ISR_FLOATRS_QUANT)
        return run_quant(m, x, sigma, seed, image, one_phase(phase, begin, (uint32_t)count), (int32_t *)logits_host, argmax_host, dcounts, -1);
    return run_fp_range(m, x, sigma, seed, image, phase, begin, count, (float *)logits_host, argmax_host, dcounts, false);
}

}  // namespace

extern "C" {

size_t isr_float_workspace_bytes(isr_model *m, uint32_t chunk_samples, int system) {
    if (!m || chunk_samples == 0) return 0;
    if (system == ISR_FLOATRS_QUANT) return isr_workspace_bytes(m, chunk_samples);
    if (system != ISR_FLOATRS_FP || build_float_net(m) != ISR_OK) return 0;
    size_t need = isr_workspace_bytes(m, chunk_samples);
    Plan pl;
    for (FloatJoin joins : {JOIN_NONE, JOIN_POOLS}) {
        place_float_net(m, chunk_samples, joins, pl);
        need = std::max(need, pl.bytes);
    }
    return need;
}

uint32_t isr_float_chunk(const isr_model *m, int system) {
    if (!m || !m->ws || m->chunk == 0) return 0;
    if (system == ISR_FLOATRS_QUANT) return m->chunk;
    return system == ISR_FLOATRS_FP ? float_chunk(m) : 0;
}

int isr_float_certify(isr_model *m, const uint8_t *x_device, float sigma, uint32_t n0, uint32_t n, double alpha,
                      uint64_t seed, uint32_t image_id, int system, isr_result *out, uint32_t *counts0_host,
                      uint32_t *counts1_host) {
    int rc = check_float_call(m, x_device, sigma, system);
    if (rc != ISR_OK) return rc;
    if (!out || n0 == 0 || n == 0 || !(alpha > 0.0 && alpha < 1.0)) return ISR_ERR_ARG;
    const uint32_t C = (uint32_t)m->pm.classes;
    if ((rc = open_counts(m)) != ISR_OK) return rc;
    if (system == ISR_FLOATRS_QUANT) {
        if ((rc = run_quant(m, x_device, sigma, seed, image_id, Slots{0, n0, {n0, n}, 1, 0, 0}, nullptr, nullptr, m->dcounts, -1)) != ISR_OK) return rc;
    } else {
        if ((rc = run_system(m, x_device, sigma, seed, image_id, 0, 0, n0, system, nullptr, nullptr, m->dcounts)) != ISR_OK) return rc;
        if ((rc = run_system(m, x_device, sigma, seed, image_id, 1, 0, n, system, nullptr, nullptr, m->dcounts + C)) != ISR_OK) return rc;
    }
    if ((rc = close_counts(m, 2)) != ISR_OK) return rc;
    if (counts0_host) std::memcpy(counts0_host, m->hcounts, sizeof(uint32_t) * C);
    if (counts1_host) std::memcpy(counts1_host, m->hcounts + C, sizeof(uint32_t) * C);
    rc = isr_decide_certify(m->hcounts, m->hcounts + C, C, (double)sigma, n, alpha, out);
    out->radius_int = 0;          // the lattice quantile belongs to the discrete law of the integer path
    out->radius_sq_int = 0;
    return rc;
}

int isr_float_debug_noisy(isr_model *m, const uint8_t *x_device, float sigma, uint64_t seed, uint32_t image_id,
                          uint32_t phase, uint32_t sample_begin, uint32_t count, int system, void *out_host) {
    int rc = check_float_call(m, x_device, sigma, system);
    if (rc != ISR_OK) return rc;
    if (!out_host || count == 0 || phase > 1 || count > isr_float_chunk(m, system)) return ISR_ERR_ARG;
    const ParsedModel &pm = m->pm;
    const size_t hw = (size_t)pm.H * pm.W;
    if (system == ISR_FLOATRS_QUANT) {
        if ((rc = run_quant(m, x_device, sigma, seed, image_id, one_phase(phase, sample_begin, count), nullptr, nullptr, nullptr, 0)) != ISR_OK) return rc;
        std::vector<int8_t> tmp(count * hw * 4);
        HIP_TRY(hipMemcpyAsync(tmp.data(), m->ws + m->plan[m->use_fused].toff[0], tmp.size(), hipMemcpyDeviceToHost, m->stream));
        HIP_TRY(hipStreamSynchronize(m->stream));
        int8_t *o = (int8_t *)out_host;
        for (uint32_t s = 0; s < count; ++s)
            for (int c = 0; c < pm.C; ++c)
                for (size_t i = 0; i < hw; ++i) o[((size_t)s * pm.C + c) * hw + i] = tmp[((size_t)s * hw + i) * 4 + c];
        return ISR_OK;
    }
    if ((rc = run_fp_range(m, x_device, sigma, seed, image_id, phase, sample_begin, count, nullptr, nullptr, nullptr, true)) != ISR_OK) return rc;
    std::vector<float> tmp(count * hw * 4);
    HIP_TRY(hipMemcpyAsync(tmp.data(), m->ws + float_plan(m, -1).toff[0], tmp.size() * 4, hipMemcpyDeviceToHost, m->stream));
    HIP_TRY(hipStreamSynchronize(m->stream));
    float *o = (float *)out_host;
    for (uint32_t s = 0; s < count; ++s)
        for (int c = 0; c < pm.C; ++c)
            for (size_t i = 0; i < hw; ++i) o[((size_t)s * pm.C + c) * hw + i] = tmp[((size_t)s * hw + i) * 4 + c];
    return ISR_OK;
}

int isr_float_debug_forward(isr_model *m, const uint8_t *x_device, float sigma, uint64_t seed, uint32_t image_id,
                            uint32_t phase, uint32_t sample_begin, uint32_t count, int system, void *logits_host,
                            int32_t *argmax_host, uint32_t *counts_host) {
    int rc = check_float_call(m, x_device, sigma, system);
    if (rc != ISR_OK) return rc;
    if (count == 0 || phase > 1) return ISR_ERR_ARG;
    const uint32_t C = (uint32_t)m->pm.classes;
    if (counts_host && (rc = open_counts(m)) != ISR_OK) return rc;
    rc = run_system(m, x_device, sigma, seed, image_id, phase, sample_begin, count, system, logits_host, argmax_host,
                    counts_host ? m->dcounts : nullptr);
    if (rc != ISR_OK) return rc;
    if (counts_host) {
        if ((rc = close_counts(m, 1)) != ISR_OK) return rc;
        for (uint32_t i = 0; i < C; ++i) counts_host[i] += m->hcounts[i];
    } else {
        HIP_TRY(hipStreamSynchronize(m->stream));
    }
    return ISR_OK;
}

int isr_float_debug_tensor(isr_model *m, const uint8_t *x_device, float sigma, uint64_t seed, uint32_t image_id,
                           uint32_t phase, uint32_t sample, int32_t tensor_id, float *out_host) {
    int rc = check_float_call(m, x_device, sigma, ISR_FLOATRS_FP);
    if (rc != ISR_OK) return rc;
    const ParsedModel &pm = m->pm;
    if (!out_host || phase > 1 || tensor_id < 0 || tensor_id >= (int)pm.tensors.size() || tensor_id == pm.ops.back().out)
        return ISR_ERR_ARG;
    bool stored = tensor_id == 0;   // an add folded into a convolution leaves that convolution's own output unstored
    for (const FloatOp &f : m->fnet->ops) stored = stored || f.out == tensor_id;
    if (!stored) return ISR_ERR_UNSUPPORTED;
    if ((rc = run_fp_range(m, x_device, sigma, seed, image_id, phase, sample, 1, nullptr, nullptr, nullptr, false, tensor_id)) != ISR_OK) return rc;
    const TensorDesc &t = pm.tensors[tensor_id];
    const size_t hw = (size_t)t.H * t.W;
    std::vector<float> tmp(hw * t.Cp);
    HIP_TRY(hipMemcpyAsync(tmp.data(), m->ws + float_plan(m, tensor_id).toff[tensor_id], tmp.size() * 4, hipMemcpyDeviceToHost, m->stream));
    HIP_TRY(hipStreamSynchronize(m->stream));
    for (int c = 0; c < t.C; ++c)
        for (size_t i = 0; i < hw; ++i) out_host[(size_t)c * hw + i] = tmp[i * t.Cp + c];
    return ISR_OK;
}

}  // extern "C"
