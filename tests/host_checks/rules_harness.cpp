// Host-only check of the rule of the kernels of one block per compute unit (bns_resident_plan.hpp) and of the rows that the single-launch
// N x H x W x C kernels hold (bns_nhwc_rows.hpp), built with g++ and run on a machine without a GPU.
//
//   rules_harness rule   reads "N C H W dtype mode n_s patch_h patch_w n_v per_channel backward" lines and prints "<kernel> <T> <rounds>":
//                           0 other kernels, 1 all registers for one tensor, 2 x beside dy
//   rules_harness sweep  random layers: what a taken plan must hold to, whatever the rule
//   rules_harness tiles  "<groups> <channels> <most> <members>" and, for every number of members and of threads, how they add the sums up:
//                           "<members> <threads> <threads at work> <polled at a time>"
//   rules_harness rows   "<V> <backward> <mixed> <rounds> <regs> <park>" for every number of rows per thread
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <initializer_list>
#include <random>

#include "../../paper_1810_10962_amd/csrc/bns_nhwc_rows.hpp"
#include "../../paper_1810_10962_amd/csrc/bns_resident_plan.hpp"

using namespace bns;

namespace {
constexpr int kUnits = 256;

struct Layer {
    bns_shape shape;
    bns_spec spec;
    int32_t n_v, backward;
};

bool choose(const Layer& l, int opt, Dims* d, ResidentChoice* c) {
    if (check_shape(&l.shape, d) != BNS_OK) return false;
    bns_shape real = l.shape;
    real.N -= l.n_v;
    if (check_spec(&real, &l.spec) != BNS_OK) return false;
    const IndexParams ip = l.n_v ? make_index_params_mixed(l.shape, l.spec, 7, l.n_v) : make_index_params(l.shape, l.spec, 7);
    *c = resident_choice(*d, ip, l.backward != 0, l.n_v > 0, opt, kUnits);
    return true;
}

int rule() {
    Layer l = {};
    while (scanf("%d %d %d %d %d %d %d %d %d %d %d %d", &l.shape.N, &l.shape.C, &l.shape.H, &l.shape.W, &l.shape.dtype, (int*)&l.spec.mode,
                 &l.spec.n_s, &l.spec.patch_h, &l.spec.patch_w, &l.n_v, &l.spec.fs_per_channel, &l.backward) == 12) {
        Dims d;
        ResidentChoice c;
        if (!choose(l, 0, &d, &c)) return 2;
        printf("%d %d %d\n", !c.take ? 0 : c.keep_x ? 2 : 1, int(c.plan.T), int(c.plan.rounds));
    }
    return 0;
}

int sweep() {
    std::mt19937_64 rng(20181026);
    auto any = [&](int lo, int hi) { return lo + int(rng() % uint64_t(hi - lo + 1)); };
    int taken = 0, bad = 0;
    for (int i = 0; i < 400000; ++i) {
        Layer l = {};
        const int top = any(1, 8);
        l.shape.N = any(2, top < 3 ? 400 : 130);
        l.shape.C = any(1, 1 << any(0, 10));
        l.shape.H = any(1, 16 * top);
        l.shape.W = any(1, 16 * top);
        l.shape.dtype = any(0, 1);
        l.spec.mode = any(0, 4);
        l.n_v = l.spec.mode != BNS_VDN && any(0, 3) == 0 ? any(1, l.shape.N - 1) : 0;
        l.spec.n_s = any(1, l.shape.N - l.n_v);
        l.spec.patch_h = any(1, l.shape.H);
        l.spec.patch_w = any(1, l.shape.W);
        l.spec.fs_per_channel = any(0, 1);
        l.backward = any(0, 1);
        Dims d;
        ResidentChoice c;
        const int opt = any(0, 4);
        if (!choose(l, opt, &d, &c) || !c.take) continue;
        ++taken;
        const ResidentPlan& p = c.plan;
        const int64_t vectors = int64_t(d.N) * c.plane_vectors;
        const bool ok = opt != 2 && p.T >= 1 && p.teams >= 1 && p.T * p.teams <= kUnits && p.T <= kResMaxTeam &&         // all blocks at once
                        p.T * kResThreads * int64_t(c.held) >= vectors && p.teams * p.rounds >= d.C && p.teams <= d.C &&  // every vector, every channel
                        int64_t(c.plane_vectors) * c.vector >= d.HW && (int64_t(c.plane_vectors) - 1) * c.vector < d.HW &&
                        d.HW >= c.vector && c.odd == (d.HW % c.vector != 0) && !(c.odd && c.patch && !c.general) &&
                        c.held == resident_vectors(l.shape.dtype == BNS_F32, c.odd, c.general, l.backward != 0, c.keep_x) &&
                        !(c.keep_x && !l.backward) && !(l.n_v && (!l.backward || !c.keep_x));
        if (!ok && ++bad < 5) fprintf(stderr, "%dx%dx%dx%d dtype %d opt %d\n", d.N, d.C, d.H, d.W, d.dtype, opt);
    }
    if (bad) return 3;
    printf("taken %d\n", taken);
    return 0;
}

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

int tiles() {
    for (int channels : {4, 8, 32, 52, 64, 128})
        for (int most : {0, 1, 7, 64, 256})
            for (int groups = 1; groups <= 1100; groups += groups < 600 ? 1 : 37) printf("m %d %d %d %d\n", groups, channels, most, tile_members(groups, channels, most));
    for (int threads = 4; threads <= 512; ++threads)
        for (int T = 1; T <= 256; ++T) {
            const TileExchange x = tile_exchange(T, threads);
            printf("x %d %d %d %d\n", T, threads, x.groups, x.polled);
        }
    return 0;
}
}  // namespace

int main(int argc, char** argv) {
    if (argc != 2) return 2;
    if (!strcmp(argv[1], "rule")) return rule();
    if (!strcmp(argv[1], "sweep")) return sweep();
    if (!strcmp(argv[1], "tiles")) return tiles();
    return !strcmp(argv[1], "rows") ? rows() : 2;
}
