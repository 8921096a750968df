// Which calls take the kernels of one block per compute unit (bns_resident.hip) and how: plain C++ without HIP headers, so that a host
// compiler can check it alone.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <numeric>

#include "bns_index.hpp"
#include "bns_validate.hpp"

namespace bns {

constexpr int kResThreads = 512;
constexpr int kResMaxTeam = 256;

// Vectors per thread: what the registers hold of one tensor, or of x and of dy.  In bf16 the place of each element, forward where S cuts rows
// that are no whole number of vectors, and the elements that two vectors of an odd plane share, backward, need registers, too.
constexpr int resident_vectors(bool f32, bool odd, bool general, bool backward, bool keep_x) {
    return keep_x ? 25 : f32 ? 49 : backward ? (odd ? 48 : 49) : (general ? 46 : 49);
}

// Teams for a kernel of K vectors per thread: the fewest rounds that blocks of K vectors allow; in a single round, as many
// blocks as there are compute units, or as leave each thread something to do.
struct ResidentPlan {
    int64_t T = 0, teams = 0, rounds = 0;
    double used = 0.0;      // share of a block's registers in use
    double fill = 0.0;      // the same over the device and all rounds
};
inline ResidentPlan resident_plan(int64_t chunks, int64_t C, int K, int cus) {
    ResidentPlan p;
    const int64_t least = (chunks + K - 1) / K, most = std::min<int64_t>(cus, kResMaxTeam);
    if (least > most) return p;
    p.T = cus / least >= C ? std::max(least, std::min<int64_t>({cus / C, (chunks + 3) / 4, most})) : least;
    p.teams = std::min<int64_t>(cus / p.T, C);
    p.rounds = (C + p.teams - 1) / p.teams;
    p.used = double(chunks) / double(p.T * K);
    p.fill = double(chunks) * double(C) / (double(cus) * K * double(p.rounds));
    return p;
}

struct ResidentChoice {
    bool take = false, keep_x = false;
    bool odd = false;           // planes that are no whole number of vectors
    bool patch = false;         // S cuts planes ...
    bool general = false;       // ... whose rows are no whole number of vectors
    int vector = 0, held = 0;   // elements per vector, vectors per thread
    uint32_t plane_vectors = 0;
    ResidentPlan plan;
};

// What the rule asks of a layer.
struct ResidentLayer {
    bool f32, odd, patch, general, everything;
    int64_t plane, stride;      // vectors of a plane, bytes from a sample to the next
    double samples, rows, columns;      // shares of the samples, and of the rows and columns of a plane, whose vectors touch S
};

// A thread's vectors lie T * 512 vectors apart.  Places of the plane that they take in turn: where a plane is 512 vectors
// (64x64 bf16, T = 1) each thread stays at one, and the threads at a patch have it in every sample -- more than the on-chip
// store holds -- while the others have nothing to do.
inline int64_t resident_places(const ResidentPlan& p, const ResidentLayer& l) {
    const int64_t step = p.T * kResThreads % l.plane;
    return step == 0 ? 1 : l.plane / std::gcd(step, l.plane);
}
// The largest share of a thread's vectors that touch S.
inline double resident_dense(const ResidentPlan& p, const ResidentLayer& l) {
    if (!l.patch) return l.samples;
    const int64_t places = resident_places(p, l);
    return l.samples * (places < 8 ? std::ceil(double(places) * l.rows) / double(places) : l.rows * l.columns);
}
// ... and with samples a multiple of 1 MiB apart as well, what the device reads at one time lies in few memory channels, unless all channels
// of the layer are read at once (us, other kernels / these): 94x128x64x64 bf16, everything, 63.4 / 113.6, 97x128x64x64 f32 112.7 / 154.9,
// 128x256x32x32 bf16 39.6 / 49.1; but 98x112x64x64 bf16 62.5 / 49.6, and in one round 93x128x64x64 bf16 62.1 / 49.3.
inline bool resident_aliased(const ResidentPlan& p, const ResidentLayer& l) {
    return p.rounds > 1 && l.stride % (1 << 20) == 0 && resident_places(p, l) == 1;
}

// Where these kernels are the faster ones: where the registers are well used, which is what fewer rounds, hence fewer pauses for an
// exchange, come from.  The lines were drawn by 3000 drawn layers, 8 to 300 MB, each timed with the other single-launch and streaming
// kernels and with both of these (times in us, theirs / these).  Backward, of about 600 layers taken 5 are more than 3 % slower (worst
// 33x140x62x62 f32 40.0 / 44.1) and 550 more than 3 % faster, 1.17 times the speed in the geometric mean; with lines at 0.5 to 0.6 it was 71 of 813.
//   forward: 64x256x56x56 bf16, one round, Batch Sampling 36.7 / 34.5, a patch 39.7 / 37.0, everything 38.9 / 36.4; 45x48x105x105 f32 (0.91
//     of the registers) 42.9 / 40.9, but 42x64x90x90 (0.85) 35.9 / 37.7.  Two rounds only where the other kernels read all of x twice, too:
//     everything 64x64x112x112 f32 82.4 / 77.7, 51x256x60x60 f32 84.1 / 75.0, 15x512x112x112 bf16 76.2 / 72.6, 52x512x60x60 bf16 88.1 /
//     87.7; Batch Sampling 64x256x56x56 f32 71.9 / 75.6.  Part of odd planes, which streaming takes well: 33x256x55x55 f32 40.3 / 43.1,
//     113x256x42x42 bf16 42.6 / 44.7 (everything 32x256x55x55 f32 46.5 / 42.9).  A patch whose rows are no whole number of vectors:
//     64x256x55x55 bf16 47.3 / 51.2.
inline bool resident_forward_pays(const ResidentPlan& p, const ResidentLayer& l) {
    return p.T > 0 && p.fill >= 0.9 && !l.general && (l.everything || (p.rounds == 1 && !l.odd)) && p.rounds <= 2;
}
//   backward, dy alone (S small): 64x256x56x56, Batch Sampling, bf16 (one round) 64.9 / 49.4, f32 (two) 114.1 / 106.1; one round
//     21x250x64x64 f32 (0.84 of the device) 50.2 / 41.4; two 26x384x60x60 f32 (0.70) 94.6 / 81.3, 19x193x96x96 (0.66) 84.7 / 72.7, but 64x160x56x56
//     (0.62) 69.8 / 75.1, 30x320x80x80 bf16 (0.60) 74.0 / 77.2; three rounds 28x671x46x46 f32 109.5 / 114.4.  Patches that threads meet at few places:
//     48x172x64x64 bf16 (one) 49.1 / 60.0, two rounds 64x48x96x96 f32 (three) 66.4 / 79.2, but one round 21x192x64x64 f32 (two) 40.7 / 36.2.  Patches whose rows are no whole number of
//     vectors: f32 two rounds 128x128x43x45 (0.62) 81.4 / 96.1, 34x127x93x93 (0.73) 100.3 / 108.0, one 106x240x27x27 (0.73) 51.2 / 52.6, 33x192x55x55 (0.75)
//     55.1 / 43.2, 48x96x60x61 (0.66) 46.4 / 44.1; bf16 96x48x100x100 (0.90) 65.0 / 69.4.  Where more of a thread's
//     vectors touch S than LDS holds (a third of 49) the rest is read again: 64x256x56x56 f32, Batch Sampling of 26, 32, 38 and 48 of the 64 samples,
//     113.9 / 107.7, 114.7 / 113.5, 114.2 / 117.0, 114.5 / 123.2, a patch of half and of nine tenths of the points 118.3 / 121.9, 118.8 / 137.5;
//     21x250x64x64 f32, two places, a patch of 28 rows 53.7 / 45.0, of 35 rows 53.5 / 55.0; bf16 64x256x56x56, 38 and 48 samples, 66.3 /
//     59.8, 66.6 / 63.7 (x beside dy 54.1 and 53.7: the better from 32 samples on).  bf16 planes that
//     are no whole number of vectors need too much arithmetic per vector: 59x80x71x71 41.3 / 53.5.
inline bool resident_big_pays(const ResidentPlan& p, const ResidentLayer& l) {
    if (p.T == 0 || (l.odd && !l.f32) || resident_aliased(p, l) || resident_dense(p, l) > (l.f32 ? 0.5 : 0.6)) return false;
    if (l.patch && resident_places(p, l) < (p.rounds == 1 ? 2 : 4)) return false;
    if (l.general && (!l.f32 || p.fill < (p.rounds > 1 ? 0.8 : l.odd ? 0.75 : 0.6))) return false;
    if (p.rounds == 1) return p.used >= (l.f32 ? 0.65 : 0.75) && p.fill >= 0.5;
    return p.rounds == 2 && p.fill >= 0.66;
}
//   backward, x beside dy: one round 25x128x64x64 f32 37.2 / 26.7, 59x80x71x71 bf16 41.3 / 34.8, but 60x128x27x27 f32 (0.44 of a block's
//     registers) 15.5 / 17.4, 34x160x35x35 f32 (0.53 of the device) 16.7 / 17.3, bf16 odd planes 54x96x55x55 (0.60) 27.0 / 31.4; two 64x256x56x56 bf16,
//     everything, 66.9 / 53.9, but 79x512x28x28 bf16 (0.64) 42.8 / 43.9, bf16 odd planes 48x128x83x83 (0.81) 67.7 / 72.3, 18x133x56x54 f32 (0.28)
//     26.3 / 29.8; three, teams of 8 and 16: f32 32x96x112x112 100.2 / 91.2, 96x96x64x64 89.3 / 83.1, 48x84x96x96 85.1 / 85.5, 64x48x112x112 103.1 /
//     92.2, bf16 128x48x112x112 143.5 / 92.8; four, teams of 16: f32 64x64x112x112 124.6 / 119.5, 128x64x80x80 131.8 / 123.0, bf16 128x64x112x112 196.8 /
//     115.2; teams of 8: bf16 128x128x80x80 147.3 / 114.7, but f32 64x128x80x80 121.9 / 123.9, 128x128x54x54 122.5 / 124.4; teams of 4 64x256x56x56
//     f32 115.5 / 119.6 (the pipelined kernel needs teams of several dozen blocks for the large channels).
inline bool resident_pair_pays(const ResidentPlan& p, const ResidentLayer& l) {
    if (p.T == 0 || resident_aliased(p, l)) return false;
    if (l.patch && !l.f32 && resident_places(p, l) < 4) return false;
    if (p.rounds == 1) return p.used >= (l.general ? 0.9 : 0.8) && p.fill >= (!l.f32 && (l.odd || l.general) ? 0.75 : 0.66);
    if (l.general && !l.f32) return false;
    if (p.rounds == 2) return p.fill >= (l.odd && !l.f32 ? 0.85 : 0.66);
    return p.rounds <= 4 && p.fill >= 0.94 && p.T >= (p.rounds == 4 && l.f32 ? 16 : 8);
}

// opt: the "resident" option.
inline ResidentChoice resident_choice(const Dims& d, const IndexParams& ip, bool backward, bool mixed, int opt, int cus) {
    ResidentChoice c;
    const bool f32 = d.dtype == BNS_F32;
    c.vector = f32 ? 4 : 8;
    if (opt == 2 || d.HW < c.vector || cus <= 0 || (mixed && !backward)) return c;
    const bns_box& b = ip.shared;
    c.odd = d.HW % c.vector != 0;
    c.patch = b.h_cnt * b.w_cnt != d.HW;
    c.general = c.patch && d.W % c.vector != 0;
    c.plane_vectors = uint32_t((d.HW + c.vector - 1) / c.vector);
    const int64_t chunks = (int64_t(d.N) * c.plane_vectors + kResThreads - 1) / kResThreads;
    if (opt == 0 && chunks * d.C < int64_t(cus) * 8) return c;              // (nothing below comes near)
    ResidentLayer l;
    l.f32 = f32;
    l.odd = c.odd;
    l.patch = c.patch;
    l.general = c.general;
    l.everything = !ip.per_channel && b.n_cnt == d.N && b.h_cnt == d.H && b.w_cnt == d.W;
    l.plane = c.plane_vectors;
    l.stride = int64_t(d.C) * d.HW * (f32 ? 4 : 2);
    l.samples = double(b.n_cnt) / double(d.N);
    l.rows = double(b.h_cnt) / double(d.H);
    l.columns = c.general ? 1.0 : std::min(1.0, double(b.w_cnt + c.vector - 1) / double(d.W));
    const ResidentPlan big = resident_plan(chunks, d.C, resident_vectors(f32, c.odd, c.general, backward, false), cus);
    const ResidentPlan pair = resident_plan(chunks, d.C, resident_vectors(f32, c.odd, c.general, backward, true), cus);
    if (opt != 0) {
        c.take = true;
        c.keep_x = backward && (mixed || opt == 4 || (opt == 1 && l.everything));
    } else if (!backward) {
        c.take = resident_forward_pays(big, l);
    } else {
        const bool pair_ok = resident_pair_pays(pair, l), big_ok = !l.everything && !mixed && resident_big_pays(big, l);
        c.take = pair_ok || big_ok;
        c.keep_x = pair_ok && !(big_ok && big.rounds < pair.rounds && resident_dense(big, l) <= (f32 ? 0.5 : 0.45));
    }
    c.plan = c.keep_x ? pair : big;
    c.held = resident_vectors(f32, c.odd, c.general, backward, c.keep_x);
    if (c.plan.T == 0) c.take = false;
    return c;
}

}  // namespace bns
