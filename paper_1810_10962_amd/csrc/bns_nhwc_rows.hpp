// Rows per thread that the single-launch N x H x W x C kernels hold (bns_nhwc_fused.hip): plain C++ without HIP headers, so that a host
// compiler can check it alone.
#pragma once

namespace bns {

// Rows in registers and, behind them, in LDS.
struct RowsHeld {
    int regs, park;
};

constexpr int kRowKeepX = 16;       // rows up to which a thread's loads all come first; backward holds x beside dy
constexpr int kRowPark = 14;        // 112 of the 160 KiB of LDS
// What the registers hold beside the sums, without scratch memory (Eq. 4 forward walks the rows twice, with more in flight where there are
// rows in LDS, too).
constexpr int rows_in_registers(int V, bool backward, bool mixed, bool parks) {
    return backward ? (V == 8 ? 35 : 40) : mixed ? (V == 8 && parks ? 16 : 20) : (V == 8 ? 36 : 40);
}
constexpr int rows_most(int V, bool backward, bool mixed) { return rows_in_registers(V, backward, mixed, true) + kRowPark; }

// Variants: steps of four rows beyond 16, the last of up to eight.  Rows that a variant holds and a thread has not are loaded (the last row again and again)
// and dropped all the same, which costs nearly what a row costs: with 24 and 49 (54) rows only, bf16 x 512 backward with 26
// rows per thread ran at 0.83, f32 x 256 at 0.81 of the speed of a kernel with a condition around every load, now at 1.07
// and 1.00; forward 0.93 and 0.92, now 1.09 and 1.07.
constexpr int kRowVariants = 9;
constexpr RowsHeld rows_held(int V, bool backward, bool mixed, int variant) {
    const int steps[] = {4, 8, 16, 20, 24, 28, 32};
    const bool parks = variant == kRowVariants - 1;
    const int all = rows_in_registers(V, backward, mixed, parks);
    if (V > 1 || variant < 3) {
        if (variant < 7) return RowsHeld{steps[variant] < all ? steps[variant] : all, 0};
    }
    return RowsHeld{all, parks ? kRowPark : 0};             // (fewer of them for single elements)
}
// The smallest variant that holds them.
constexpr int row_variant(int rounds, int V, bool backward, bool mixed) {
    int v = 0;
    while (v + 1 < kRowVariants && rows_held(V, backward, mixed, v).regs + rows_held(V, backward, mixed, v).park < rounds) ++v;
    return v;
}

// Forward: whether all loads of a thread come before its first sum beyond 16 rows, too, each under a condition.  Where rows begin on
// no 64 bytes, the blocks of neighbouring tiles read the same lines, and they meet in the L2 when both request everything at once, not
// when each goes at the pace of its sums (us, paced against this: f32 16x150x1xW, 24 rows per thread, 34.4 / 32.1, 44 rows 61.0 / 55.8; 79
// channels, 24 rows, 39.0 / 35.9; bf16 x 431, 28 rows, 43.3 / 41.5).  Rows beyond the registers are then read twice; LDS holds them
// better in bf16 (431 channels, 44 rows, 1.18 of the speed of the paced kernel without it against 1.14, 50 rows 1.25 against 1.16).  Where
// rows are aligned the pace is worth 7 % and more.
constexpr bool rows_first(int rounds, int V, bool backward, bool mixed, long pitch) {
    return !backward && !mixed && V > 1 && rounds > kRowKeepX && pitch % 64 != 0 && (V == 4 || rounds <= rows_in_registers(V, false, false, false));
}

// Blocks that share the rows of a column tile: two rows per thread and no fewer (against four, over 22 drawn layers of up to 4 MB, 1.04 of the speed
// forward and 1.09 backward, three 1.02 and 1.04; one 1.03 and 1.09, but 0.89 / 0.92 at 54x144x10x13 bf16); four where more members would make a
// block read more than 4096 pairs of sums (16x48x55x55 bf16, a patch, 256 members 13.7 / 13.7 us, 143 11.6 / 11.9).  groups: rows of the
// tile over the rows that a block takes at a time; channels of the tile; most: what the device holds.
constexpr int tile_members(int groups, int channels, int most) {
    const int two = (groups + 1) / 2, four = (groups + 3) / 4, pairs = 4096 / channels;
    const int few = two < pairs ? two : pairs, want = four > few ? four : few;
    return most < 1 ? 1 : want < most ? want : most;
}

// How the threads that share a channel (at most `threads` of them) add up the sums of T members: as many as leave each of them the same
// number, which it polls in as few turns of up to kRowPoll as that takes.
constexpr int kRowPoll = 8;
struct TileExchange {
    int groups, polled;     // threads, members that a thread polls at a time
};
constexpr TileExchange tile_exchange(int T, int threads) {
    const int each = (T + threads - 1) / threads, turns = (each + kRowPoll - 1) / kRowPoll;
    return TileExchange{(T + each - 1) / each, (each + turns - 1) / turns};
}

// Whether stores leave the non-temporal hint out: lines that two tiles share are then put together in the L2.  With the hint against without,
// forward, 90 drawn layers of several tiles whose rows begin on no 64 bytes, f32 / bf16: 1.05 / 1.02 from 2 to 8 MB, 1.10 / 1.09 to 30 MB, 1.37 / 1.53
// beyond, one layer below 0.97 (us: 23x150x104x104 bf16 68.8 / 37.9, 6x252x109x106 f32 49.8 / 33.5, 50x150x19x19 f32 11.5 / 10.5, whose written
// bytes by counters went from 1.28 times the least to 1.03, backward from 1.33).  One tile
// that holds whole rows 0.88 (43x16x103x102 bf16) to 0.97, rows on 64 bytes 0.90 (8 to 30 MB).  Backward 1.03 to 1.06 up to 30 MB where vectors,
// too, begin anywhere (39 layers, none below 0.98; 50x150x19x19 f32 13.7 / 12.6, 26x293x32x30 f32 25.9 / 22.4), 0.98 where they begin on 16
// bytes; beyond 30 MB either way (71x162x45x45 bf16 52.7 / 41.9, 20x478x52x52 f32, a patch, 84 / 94).  Forward, what is written then lies in the
// memory-side cache in the place of what was read: backward on its own is as fast as before (600 layers, 1.00 beyond 30 MB), right after
// forward on the same tensors it finds less of x there (f32 of 70 MB and more: the two together 1.00, at worst 0.94, 3x1023x90x90 152 / 162).  Tiles are
// 128 to 256 bytes wide, most of their lines are shared, and a hint for the others would change little.
// Not for Eq. 4, whose kernels have no such flavour: 250 layers, forward 1.05 (none below 0.97), backward 1.00 (22 below), which another
// 36 kernels (1.4 MB) were not spent on.
constexpr bool shares_lines(int tiles, long pitch, long bytes, bool backward) {
    return tiles > 1 && (backward ? pitch % 16 != 0 && bytes < 30000000 : pitch % 64 != 0);
}

}  // namespace bns
