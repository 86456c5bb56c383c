// Reads a model blob, places its fused plan for chunks of some copies, and prints for every three consecutive ops that each read the
// one before what images_apart says, and whether the bytes that an image's ops write and another image's ops still read are
// disjoint, image by image.  Built and run by tests/test_plan_host.py.
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
    for (uint32_t copies : {1u, 2u, 5u, 64u}) {
        Plan pl;
        build_fused_plan(pm, ops, pl.ops, false);
        plan_segments(pm, copies, pl);
        plan_workspace(pm, copies, pl);
        for (size_t i = 0; i + 2 < pl.ops.size(); ++i) {
            const DevOp *d = &pl.ops[i];
            if (d[1].a != d[0].out || d[2].a != d[1].out) continue;
            struct Range { size_t from, to; };
            auto image = [&](int t, uint32_t j) {
                const TensorDesc &x = pm.tensors[t];
                const size_t n = (size_t)x.H * x.W * x.Cp, at = pl.toff[t] + j * n;
                return Range{at, at + n};
            };
            bool apart = true;
            for (uint32_t j = 0; j < copies; ++j)
                for (uint32_t k = 0; k < copies; ++k)
                    for (int w = 0; w < 3; ++w)
                        for (int r = 0; r < 3; ++r) {
                            if (j == k || d[w].head || d[w].type == OP_FC) continue;
                            const Range out = image(d[w].out, j), in = image(d[r].a, k);
                            if (out.from < in.to && in.from < out.to) apart = false;
                        }
            std::printf("copies %u narrow %d %d %d head %d apart %d by_bytes %d\n", copies, d[0].narrow, d[1].narrow, d[2].narrow, d[2].head, (int)images_apart(pm, pl, i), (int)apart);
        }
    }
    return 0;
}
