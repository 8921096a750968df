// Host-only check of the workspace layout (bns_workspace.hpp), built with g++ and run on a machine without a GPU.
//
// The slots of the single-launch kernels must hold nothing but their own stamped words, whatever calls use the memory
// one after the other: the slots lie at one place for every shape of both layouts, and no region of partial sums of any
// shape begins below their end.  Prints "shapes <n>".
#include <stdio.h>
#include <stdlib.h>

#include <random>

#include "../../paper_1810_10962_amd/csrc/bns_validate.hpp"
#include "../../paper_1810_10962_amd/csrc/bns_workspace.hpp"

using namespace bns;

namespace {
int g_bad = 0;
void expect(bool ok, const char* what, const Dims& d, size_t sum_bytes) {
    if (ok) return;
    fprintf(stderr, "%s: layout %d, %d channels, sums of %zu bytes\n", what, d.layout, d.C, sum_bytes);
    ++g_bad;
}
}  // namespace

int main() {
    std::mt19937_64 rng(20181026);
    const size_t pair = 2 * sizeof(unsigned long long);
    const int count = 200000;
    for (int i = 0; i < count; ++i) {
        Dims d = {};
        d.N = d.H = d.W = d.HW = 1;
        d.C = int32_t(1u << (rng() % 25));
        d.C = int32_t(rng() % uint64_t(d.C)) + 1;
        if (i < 5000) d.C = i + 1;
        d.layout = (rng() & 1) ? BNS_NHWC : BNS_NCHW;
        // pairs of floats per channel: N x C x H x W up to 64, N x H x W x C 1 to 2048
        const size_t splits = d.layout == BNS_NCHW ? size_t(most_splits(d.C)) : 1 + rng() % 2048;
        expect(splits >= 1 && (d.layout == BNS_NHWC || splits <= 64), "partial sums per channel", d, splits);
        const size_t sum_bytes = (size_t(d.C) * splits * 8 + 255) & ~size_t(255);
        const WorkspaceLayout w = workspace_layout(sum_bytes);
        expect(w.slots == kHeaderBytes, "the slots begin behind the header", d, sum_bytes);
        expect(w.sums >= w.slots + w.slot_bytes, "partial sums inside the slots", d, sum_bytes);
        expect(w.total >= w.sums + 2 * sum_bytes, "two regions of sums", d, sum_bytes);
        expect(w.slots % 256 == 0 && w.sums % 256 == 0 && w.total % 256 == 0, "alignment", d, sum_bytes);
        // what the kernels of this layout write there: 8192 blocks, four sets; 256 blocks of 128 channels, two sets
        const size_t own = d.layout == BNS_NCHW ? size_t(8192) * pair * 4 : size_t(256) * 128 * pair * 2;
        expect(w.slot_bytes >= own, "slots of the layout's own kernels", d, sum_bytes);
        // ... and no other shape's sums lie in them, either layout's
        expect(w.slot_bytes == kSlotBytes, "one size of slots", d, sum_bytes);
        expect(w.sums >= kHeaderBytes + kSlotBytes, "partial sums in another shape's slots", d, sum_bytes);
        if (d.layout == BNS_NCHW)
            expect((w.total <= kBuiltinNchwBytes) == (d.C <= 3840), "what the built-in scratch holds", d, sum_bytes);
    }
    if (g_bad) return 3;
    printf("shapes %d\n", count);
    return 0;
}
