// Host-only check of the rows that the single-launch N x H x W x C kernels hold (bns_nhwc_rows.hpp), built with g++ and run on a machine
// without a GPU.
//
//   rules_harness rows   "<V> <backward> <mixed> <rounds> <regs> <park>" for every number of rows per thread
#include <stdio.h>
#include <string.h>

#include <initializer_list>

#include "../../paper_1810_10962_amd/csrc/bns_nhwc_rows.hpp"

using namespace bns;

namespace {
int rows() {
    for (int V : {1, 4, 8})
        for (int backward = 0; backward < 2; ++backward)
            for (int mixed = 0; mixed < 2; ++mixed)
                for (int n = 1; n <= 130; ++n) {
                    const RowsHeld h = rows_held(V, backward != 0, mixed != 0, row_variant(n, V, backward != 0, mixed != 0));
                    printf("%d %d %d %d %d %d\n", V, backward, mixed, n, h.regs, h.park);
                }
    return 0;
}
}  // namespace

int main(int argc, char** argv) {
    if (argc != 2) return 2;
    return !strcmp(argv[1], "rows") ? rows() : 2;
}
