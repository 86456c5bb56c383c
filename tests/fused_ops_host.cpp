// Reads a model blob and prints the ops of its fused plans: which kernel takes them, and the classes of their requantisations together.
// Built and run by tests/test_fused_ops_host.py.
#include <cstdio>
#include <string>
#include <vector>

#include "isr_internal.h"
#include "plan.h"

using namespace isr;

int main(int argc, char **argv) {
    if (argc != 2) return 1;
    std::FILE *f = std::fopen(argv[1], "rb");
    if (!f) return 1;
    std::vector<uint8_t> blob;
    for (int c; (c = std::fgetc(f)) != EOF;) blob.push_back((uint8_t)c);
    std::fclose(f);
    ParsedModel pm;
    std::string why;
    std::vector<DevOp> ops;
    ConstArena arena;
    arena.put(nullptr, 256);
    if (parse_model(blob.data(), blob.size(), pm, why) != ISR_OK || build_device_ops(pm, ops, arena) != ISR_OK) return 1;
    rebase_device_ops(ops, arena.host.data());
    std::vector<DevOp> fused;
    build_fused_plan(pm, ops, fused, false);
    for (const DevOp &d : fused) {
        const ConvParams &c = d.conv;
        int rq = c.rq & (c.fuse_add == 2 ? c.rq2 : ~0);
        if (d.bneck) rq &= d.conv2.rq & (d.bneck >= 2 ? d.conv3.rq : ~0) & (d.bneck == 4 ? d.conv3.rq2 : ~0);
        if (d.reduce) rq &= d.conv4.rq;
        if (d.xr) rq &= d.conv2.rq;
        std::printf("type %d stem %d bneck %d reduce %d xr %d k %d stride %d cin %d cout %d next %d form %d tie_free %d add_tie_free %d\n", (int)d.type, d.stem_pool, d.bneck, d.reduce, d.xr, c.k, c.stride,
                    c.Cin_p, c.Cout_p, d.xr ? d.conv2.Cout_p : 0, d.type == OP_CONV ? rq_form(rq) : -1, c.tie_free, c.fuse_add ? c.add_tie_free : -1);
    }
    return 0;
}
