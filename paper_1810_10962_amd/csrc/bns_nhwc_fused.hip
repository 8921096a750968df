// Single-launch kernels for the N x H x W x C layout: the statistics (or the sums of Eq. 5) and the element-wise pass of
// one direction in one kernel, with as much of the tensor as fits kept in registers in between.
//
// The tensor is a matrix of M = N*H*W rows by C columns.  A block of 512 threads owns a tile of CT <= 128 columns
// and one of T shares of the rows: thread (ty, tx) holds V channels of the rows (k * T + j) * TY + ty, so
// that the device as a whole walks the tensor front to back.  The first K of a thread's rows stay in registers, the next L in LDS;
// what does not fit is read again in the second phase, from the memory-side cache if it fits there.  The T blocks of a tile exchange
// their column sums once, through the stamped slots of the other single-launch kernels (bns_fused_device.hpp); with T = 1 nothing
// crosses blocks.
//
// Bound by memory, by the exchange and, in small tensors, by a chain of latencies and of instructions (one instruction of every wave
// costs a block of 512 threads 3.4 ns: two waves per SIMD, four cycles each).  By stamps on the device, 50x150x19x19 f32 forward, us:
// 1.2 until a block has requested its rows, 1.5 until the first of them are there, 0.8 for a thread's sums, 0.8 for the block's, 1.7 for
// the words of 84 team-mates, 0.9 to add them up and for the constants, 0.9 for its stores and 1.5 until they are done.  Measured against the streaming
// kernels (three launches per direction), us forward / backward, Batch Sampling: 64x256x40x40 f32 43.9 / 70.1 against 39.1 / 55.4;
// 64x256x56x56 bf16 47.6 / 71.2 against 42.5 / 57.4 (45.5 / 65.7 when loads had conditions around them and rows beyond the registers were
// read twice), full BN 58.5 / 85.8 against 44.7 / 65.9 (backward 70.4 while it spilled registers); 67x512x11x11 f32 16.2 / 21.0 against
// 11.5 / 13.7.
//
// Columns that are no whole number of vectors: the last vector of a row is moved back so that it ends with the row.  The
// channels it shares with the vector before it are computed twice, with the same bits.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "bns_device.hpp"
#include "bns_fused_device.hpp"
#include "bns_internal.hpp"
#include "bns_nhwc_device.hpp"
#include "bns_nhwc_rows.hpp"

namespace bns {

namespace {

constexpr int kRowThreads = 512;
constexpr int kRowMaxTile = 128;        // channels of a column tile
constexpr int kRowBatch = 8;            // rows that are not kept: read again this many at a time

struct RowArgs {
    FusedArgs f;            // tensors, vectors, exchange; f.T members per tile, f.num_teams tiles
    RowSet S;
    RowBox B;
    FastDiv tx_div, ct_div; // column lanes and channels of a tile
    uint32_t M;             // rows
    uint32_t s_lo;          // first row of S, if S is one run of rows
    uint32_t virtual_rows;  // Eq. 4: rows of the virtual set
    int32_t CV;             // column vectors of a row
    int32_t TY;             // row lanes
    int32_t rounds;         // rows per thread
    uint32_t pitch;         // bytes of a row
    int32_t keep_x;         // backward: x is read again where it lies in S, leave it in the memory-side cache
    FastDiv tiles_div;      // column tiles
    int32_t eights;         // blocks that are dealt out in eights (see row_lane)
    int32_t sum_groups;     // threads that share a channel in tile_sums, and in tile_collect
    int32_t member_groups;
    int32_t polled;         // members that a thread polls at a time
    uint32_t pivot_off[kPivotRows];     // byte offsets of the rows that the pivots are taken from
    int32_t mute_channel;   // 1 + a channel that no member publishes (host-forced give-up, for tests of that path); 0: none
};

struct RowLane {
    int tile, j;            // column tile, share of the rows
    int tx, ty;
    int col, local;         // first channel of the thread's vector, in the row and in the tile
    int width;              // channels of this tile
    bool live;
};

template <int V>
__device__ __forceinline__ RowLane row_lane(const RowArgs& A) {
    RowLane l;
    const int TX = int(A.tx_div.d), CT = TX * V;
    // Consecutive blocks go to consecutive XCDs: the tiles of one share of the rows go to one of them (shares in eights).
    const uint32_t b = blockIdx.x;
    if (int(b) >= A.eights) {
        l.j = int(fdiv(b, A.tiles_div));
        l.tile = int(b) - l.j * A.f.num_teams;
    } else {
        const uint32_t e = fdiv(b / 8u, A.tiles_div);
        l.tile = int(b / 8u) - int(e) * A.f.num_teams;
        l.j = int(e * 8u + b % 8u);
    }
    l.ty = int(fdiv(threadIdx.x, A.tx_div));
    l.tx = int(threadIdx.x) - l.ty * TX;
    const int cv = l.tile * TX + l.tx;
    l.live = l.ty < A.TY && cv < A.CV;
    l.col = min((l.live ? cv : l.tile * TX) * V, A.f.C - V);
    l.local = l.col - l.tile * CT;
    l.width = min(CT, A.f.C - l.tile * CT);
    return l;
}

// Rows of S (or, SET = 1, of the virtual set of Eq. 4).
__device__ __forceinline__ bool in_set(const RowArgs& A, int set, uint32_t row) {
    if (set == 1) return row < A.virtual_rows;
    return A.S.contiguous ? row - A.s_lo < A.S.rows : row_in(A.B, row);
}

// Pairs of sums in LDS, first and second side by side.
typedef double pair_t __attribute__((ext_vector_type(2)));

// Sums over i < n of p[i * CT], eight loads in flight, in a fixed order.  (A loop, and the whole batches without conditions: an
// instruction costs a block of 512 threads 3.4 ns, and everybody waits for these.)
__device__ __forceinline__ void add_strided(const pair_t* p, int CT, int n, double& s1, double& s2) {
    s1 = s2 = 0.0;
    int i = 0;
#pragma unroll 1
    for (; i + 8 <= n; i += 8) {
        pair_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = p[(i + u) * CT];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            s1 += v[u].x;
            s2 += v[u].y;
        }
    }
#pragma unroll 1
    for (; i < n; i += 4) {
        pair_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = p[min(i + u, n - 1) * CT];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            s1 += i + u < n ? v[u].x : 0.0;
            s2 += i + u < n ? v[u].y : 0.0;
        }
    }
}

// Column sums of the block, by thread t < CT for channel t of the tile: per-thread sums through LDS, added in fp64 in a
// fixed order (first over the row lanes g, g + Q, ..., then over g).  What it costs is a chain of LDS round trips and the instructions
// between them, so the two sums of a channel lie side by side, eight row lanes are requested at a time, and no more than
// kSumGroups threads share a channel, whose sums one thread then adds (2x512x14x14 f32, 16 channels, 128 row lanes: 1.5 us with
// 32 groups added one after the other, 1.4 us with four requests of single sums at a time and offsets by multiplication).
constexpr int kSumGroups = 8;
template <int V>
__device__ __forceinline__ void tile_sums(const RowArgs& A, const RowLane& l, const double (&a)[V], const double (&q)[V], float* lds,
                                          pair_t* part, double& s1, double& s2) {
    typedef float vec_t __attribute__((ext_vector_type(V < 2 ? 2 : 4)));
    typedef float both_t __attribute__((ext_vector_type(2)));
    constexpr int kPairs = V < 2 ? 1 : 2;                   // channels of a 128-bit write
    const uint32_t CT = A.ct_div.d;
    __syncthreads();                                        // lds and part may still be read from the previous use
    if (l.live) {
        vec_t* to = reinterpret_cast<vec_t*>(lds + 2u * (__umul24(uint32_t(l.ty), CT) + uint32_t(l.tx * V)));
#pragma unroll
        for (int e = 0; e < V; e += kPairs) {
            vec_t w;
#pragma unroll
            for (int i = 0; i < kPairs; ++i) {
                w[2 * i] = float(a[e + i]);
                w[2 * i + 1] = float(q[e + i]);
            }
            to[e / kPairs] = w;
        }
    }
    __syncthreads();
    const uint32_t g = fdiv(threadIdx.x, A.ct_div), ch = threadIdx.x - __umul24(g, CT);
    const int Q = A.sum_groups;
    s1 = s2 = 0.0;
    if (int(g) < Q && int(ch) < l.width) {
        // where channel ch lies in a row lane's sums: the last vector of a row may have been moved back
        const int vec = min(int(ch) / V, (l.width - 1) / V), first = min(vec * V, A.f.C - V - l.tile * int(CT));
        const both_t* at = reinterpret_cast<const both_t*>(lds) + (vec * V + (int(ch) - first));
        const uint32_t hop = uint32_t(Q) * CT, last = uint32_t(A.TY - 1) * CT;
        uint32_t off = __umul24(g, CT);
        int r = 0;                                          // row lanes before the batch's first, the same for the whole block
#pragma unroll 1
        for (; r + 8 * Q <= A.TY; r += 8 * Q, off += 8u * hop) {
            both_t u[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) u[i] = at[off + uint32_t(i) * hop];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                s1 += double(u[i].x);
                s2 += double(u[i].y);
            }
        }
#pragma unroll 1
        for (; r < A.TY; r += 4 * Q, off += 4u * hop) {
            both_t u[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) u[i] = at[min(off + uint32_t(i) * hop, last)];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool there = off + uint32_t(i) * hop <= last;
                s1 += double(there ? u[i].x : 0.f);
                s2 += double(there ? u[i].y : 0.f);
            }
        }
        part[threadIdx.x] = pair_t{s1, s2};
    }
    __syncthreads();
    if (int(threadIdx.x) < l.width) add_strided(part + threadIdx.x, int(CT), Q, s1, s2);
}

// Exchange of the column sums between the T members of a tile: every member reads all T pairs of every channel.  Words are
// stamped as in the other single-launch kernels.  Slots: [set][tile][member][first or second sum][channel]: the lanes of a wave that
// reads a member's sums, one channel each, take whole cache lines.  (Every such read goes past the L2, and T members read T * CT pairs:
// with the two words of a pair side by side each line was fetched twice, 36 MB in the exchange of 50x150x19x19 f32.)
// (32-bit offsets: beside a full register file, sixteen 64-bit addresses went through scratch memory)
__device__ __forceinline__ uint32_t sum_slot(const RowArgs& A, const RowLane& l, int set, int member, int ch) {
    const uint32_t tile = uint32_t(set * A.f.num_teams + l.tile), T = uint32_t(A.f.T), CT = A.ct_div.d;
    return ((tile * T + uint32_t(member)) * 2u * CT + uint32_t(ch)) * 8u;        // of the first sum; the second lies CT words further
}
__device__ __forceinline__ void put_word(unsigned long long* p, uint32_t stamp, uint32_t payload) {
    __hip_atomic_store(p, (static_cast<unsigned long long>(stamp) << 32) | payload, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// This member's pair of channel t: published by thread t.
__device__ __forceinline__ void tile_publish(const RowArgs& A, const RowLane& l, uint32_t stamp, int set, double s1, double s2) {
    if (A.f.T == 1 || int(threadIdx.x) >= l.width || A.f.mute) return;
    if (A.mute_channel == l.tile * int(A.ct_div.d) + int(threadIdx.x) + 1) return;
    const uint32_t mine = sum_slot(A, l, set, l.j, int(threadIdx.x));
    put_word(at_byte(A.f.slots, mine), stamp, __float_as_uint(float(s1)));
    put_word(at_byte(A.f.slots, mine + A.ct_div.d * 8u), stamp, __float_as_uint(float(s2)));
}

// Adds the pairs of members first, first + step, ... of channel ch, A.polled of them polled at a time until all carry the stamp; bounded
// like poll_pair.  If a wait ran out: NaN, and lost[ch] is set (lost = null: the caller does not ask).
__device__ __forceinline__ void add_members(const RowArgs& A, const RowLane& l, uint32_t stamp, int set, uint32_t ch, uint32_t first,
                                            uint32_t step, uint32_t* lost, double& s1, double& s2) {
    const FusedArgs& F = A.f;
    const uint32_t CT = A.ct_div.d, pair = CT * 16u, hop = step * pair, row = uint32_t(A.polled) * hop;
    const uint32_t base = sum_slot(A, l, set, 0, int(ch)), last = base + uint32_t(F.T - 1) * pair;
    uint32_t limit = F.spin_limit;
    s1 = s2 = 0.0;
    for (uint32_t off = base + __umul24(first, pair); off <= last; off += row) {
        unsigned long long w1[kRowPoll], w2[kRowPoll];
        for (uint32_t spin = 0;; ++spin) {
            if (spin >= limit) {
                __hip_atomic_fetch_add(&F.hdr->expired, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                s1 = s2 = __builtin_nan("");
                if (lost) lost[ch] = 1u;
                return;
            }
#pragma unroll
            for (int u = 0; u < kRowPoll; ++u)
                if (u < A.polled) {
                    const uint32_t at = min(off + uint32_t(u) * hop, last);
                    w1[u] = __hip_atomic_load(at_byte(F.slots, at), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    w2[u] = __hip_atomic_load(at_byte(F.slots, at + CT * 8u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            bool all = true;
#pragma unroll
            for (int u = 0; u < kRowPoll; ++u)
                if (u < A.polled) all = all && uint32_t(w1[u] >> 32) == stamp && uint32_t(w2[u] >> 32) == stamp;
            if (all) break;
            if ((spin & 1023u) == 1023u && __hip_atomic_load(&F.hdr->expired, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u)
                limit = F.spin_limit / 64u + 1u;
            __builtin_amdgcn_s_sleep(2);
        }
#pragma unroll
        for (int u = 0; u < kRowPoll; ++u)
            if (u < A.polled) {
                const bool there = off + uint32_t(u) * hop <= last;
                s1 += double(there ? __uint_as_float(uint32_t(w1[u])) : 0.f);
                s2 += double(there ? __uint_as_float(uint32_t(w2[u])) : 0.f);
            }
    }
}

// Totals over the members, by thread t < CT.  Every sum is taken in a fixed order, so all members get the same bits.
// A wait that runs out leaves NaN in that channel and sets its word of lost.
__device__ __forceinline__ void tile_collect(const RowArgs& A, const RowLane& l, uint32_t stamp, int set, pair_t* part, uint32_t* lost,
                                             double& s1, double& s2) {
    if (A.f.T == 1) return;
    const uint32_t CT = A.ct_div.d, g = fdiv(threadIdx.x, A.ct_div), ch = threadIdx.x - __umul24(g, CT);
    const int Q = A.member_groups;
    __syncthreads();                                        // part may still be read
    if (int(g) < Q && int(ch) < l.width) {
        // (words are requested for every member at once, and none twice: the polls of all blocks share one path)
        add_members(A, l, stamp, set, ch, g, uint32_t(Q), lost, s1, s2);
        part[threadIdx.x] = pair_t{s1, s2};
    }
    __syncthreads();
    if (int(threadIdx.x) < l.width) add_strided(part + threadIdx.x, int(CT), Q, s1, s2);
}

// A thread's way down the rows: the next row, and its byte offset from the tensor's first element, column included.
// (ANEW: each phase walks anew instead of keeping one offset per row alive, where there are many)
template <bool ANEW>
struct RowWalk {
    uint32_t row, off;
    __device__ __forceinline__ void next(uint32_t step, uint32_t hop) {
        if (ANEW) asm volatile("" : "+v"(row), "+v"(off));
        row += step;
        off += hop;
    }
};

template <typename T, int V, bool NT>
__device__ __forceinline__ typename RawVec<T, V>::raw_t row_load(const T* p) {
    typedef typename RawVec<T, V>::raw_t raw_t;
    typedef raw_t elem_t __attribute__((aligned(sizeof(T))));
    if (NT) return __builtin_nontemporal_load(reinterpret_cast<const elem_t*>(p));
    return *reinterpret_cast<const elem_t*>(p);
}
// SHARED: part of the lines is written by two blocks.  Stores with the non-temporal hint send their part of a line on to the memory; plain ones
// wait for the other part in the L2 (see shares_lines).
template <typename T, int V, bool SHARED>
__device__ __forceinline__ void row_store(T* p, typename RawVec<T, V>::raw_t r) {
    typedef typename RawVec<T, V>::raw_t raw_t;
    typedef raw_t elem_t __attribute__((aligned(sizeof(T))));
    if (SHARED) *reinterpret_cast<elem_t*>(p) = r;
    else __builtin_nontemporal_store(r, reinterpret_cast<elem_t*>(p));
}

// Forward: Eq. 3 (Eq. 4 if MIXED), Eq. 8, Eq. 1.  A thread keeps K rows in registers and L in LDS; rows beyond are read again.
// Beyond 16 rows loads are unconditional (past the end the last row is read) and run kAhead rows ahead of the sums: a condition around a load
// makes every later wait one for all loads, and a thread that issues all of them first finds most of its rows there before it
// adds the first one up.  FIRST: all loads come first all the same (see rows_first).
template <typename T, int V, int K, int L, bool MIXED, bool FIRST, bool SHARED>
__global__ __launch_bounds__(kRowThreads, 2) void nhwc_fused_forward_kernel(RowArgs A) {
    typedef RawVec<T, V> RV;
    typedef typename RV::raw_t raw_t;
    __shared__ raw_t park[L > 0 ? L * kRowThreads : 1];
    __shared__ float __attribute__((aligned(16))) lds[2 * kRowThreads * V];
    __shared__ pair_t part[kRowThreads];
    __shared__ float piv[(MIXED ? 2 : 1) * kRowMaxTile];
    __shared__ float4 consts[kRowMaxTile];
    __shared__ uint32_t words[3], lost[kRowMaxTile];
    touch_arguments<RowArgs>();
    const FusedArgs& F = A.f;
    const RowLane l = row_lane<V>(A);
    const T* x = static_cast<const T*>(F.x);
    T* y = static_cast<T*>(F.out);
    const unsigned long long state = stamp_request(F);
    const uint32_t step = uint32_t(F.T) * uint32_t(A.TY), hop = step * A.pitch;
    const uint32_t column = uint32_t(l.col) * uint32_t(sizeof(T)), last = (A.M - 1u) * A.pitch + column;
    typedef RowWalk<(K > 16)> Walk;
    auto walk_from = [&](int k) {
        const uint32_t row = opaque(uint32_t(l.j) * uint32_t(A.TY) + uint32_t(l.ty)) + uint32_t(k) * step;
        return Walk{row, row * A.pitch + column};
    };

    // The pivot of a channel is the mean of its first few sampled rows (see coarse), read by the first row lane.
    raw_t pv[kPivotRows], pw[MIXED ? kPivotRows : 1];
    if (l.ty == 0) {
#pragma unroll
        for (int i = 0; i < kPivotRows; ++i) {
            pv[i] = row_load<T, V, false>(at_byte(x, A.pivot_off[i] + column));
            if constexpr (MIXED) pw[i] = row_load<T, V, false>(at_byte(x, min(uint32_t(i), A.virtual_rows - 1u) * A.pitch + column));
        }
    }
    constexpr int kAhead = FIRST || K < kRowKeepX ? K : kRowKeepX;
    constexpr bool kAgain = L > 0 || (FIRST && K > kRowKeepX);         // takes more rows than it holds, too
    // The registers are full: what a channel needs waits in LDS for its sums.  (Half as many polls at a time instead: 64x256x40x40 f32 40.3
    // against 39.1 us, 56x56 full BN 81.6 against 80.2.)
    constexpr bool kStow = K + L > 52;
    constexpr bool kTight = K <= kAhead;                    // all loads come before the first sum: only those that are needed
    raw_t v[K], u[L > 0 ? L : 1];
    Walk wl = walk_from(K);                              // of the loads
    if constexpr (L > 0) {
#pragma unroll
        for (int k = 0; k < L; ++k) {
            u[k] = row_load<T, V, true>(at_byte(x, min(wl.off, last)));
            wl.next(step, hop);
        }
    }
    wl = walk_from(0);
    auto load = [&](int k) {
        v[k] = row_load<T, V, true>(at_byte(x, min(wl.off, last)));
        wl.next(step, hop);
    };
    if constexpr (!kAgain) {
#pragma unroll
        for (int k = 0; k < kAhead; ++k)
            if (!kTight || k < A.rounds) load(k);
    }
    if (l.ty == 0 && l.live) {
        float p[V], f[V];
#pragma unroll
        for (int e = 0; e < V; ++e) p[e] = 0.f;
        if (A.S.pivot_rows == uint32_t(kPivotRows)) {
#pragma unroll
            for (int i = 0; i < kPivotRows; ++i) {
                RV::unpack(pv[i], f);
#pragma unroll
                for (int e = 0; e < V; ++e) p[e] += f[e];
            }
        } else {
#pragma unroll
            for (int i = 0; i < kPivotRows; ++i) {
                RV::unpack(pv[i], f);
#pragma unroll
                for (int e = 0; e < V; ++e) p[e] += uint32_t(i) < A.S.pivot_rows ? f[e] : 0.f;
            }
        }
#pragma unroll
        for (int e = 0; e < V; ++e) piv[l.local + e] = coarse(p[e] * A.S.inv_pivot_rows);
        if constexpr (MIXED) {
            const uint32_t rows = min(uint32_t(kPivotRows), A.virtual_rows);
#pragma unroll
            for (int e = 0; e < V; ++e) p[e] = 0.f;
#pragma unroll
            for (int i = 0; i < kPivotRows; ++i) {
                RV::unpack(pw[i], f);
#pragma unroll
                for (int e = 0; e < V; ++e) p[e] += uint32_t(i) < rows ? f[e] : 0.f;
            }
#pragma unroll
            for (int e = 0; e < V; ++e) piv[kRowMaxTile + l.local + e] = coarse(p[e] / float(rows));
        }
    }
    if (threadIdx.x < uint32_t(kRowMaxTile)) lost[threadIdx.x] = 0u;
    stamp_accept(F, state, words);
    __syncthreads();
    const uint32_t stamp = read_stamp(F, words);

    double s1 = 0.0, s2 = 0.0, u1 = 0.0, u2 = 0.0;          // thread t < CT: the sums of channel t
    float ga = 0.f, be = 0.f, rm = 0.f, rv = 0.f;
    const int c = l.tile * int(A.ct_div.d) + int(threadIdx.x);
    const bool leads = int(threadIdx.x) < l.width;
    auto channel = [&]() {
        ga = F.gamma[c];
        be = F.beta[c];
        if (l.j == 0 && F.running_mean) rm = F.running_mean[c];
        if (l.j == 0 && F.running_var) rv = F.running_var[c];
    };
#pragma unroll
    for (int set = 0; set < (MIXED ? 2 : 1); ++set) {
        double a[V], q[V];
        float p[V];
#pragma unroll
        for (int e = 0; e < V; ++e) {
            a[e] = q[e] = 0.0;
            p[e] = piv[set * kRowMaxTile + l.local + e];
        }
        // Up to four rows of the walk are added in fp32, their sum goes into the fp64 accumulator.
        auto add = [&](auto rows, Walk& w, auto&& row_of) {
            constexpr int R = decltype(rows)::value;
            bool in[R], any = false;
#pragma unroll
            for (int i = 0; i < R; ++i) {
                in[i] = w.row < A.M && in_set(A, set, w.row);
                any |= in[i];
                w.next(step, hop);
            }
            if (any) {
                float fa[V], fq[V];
#pragma unroll
                for (int e = 0; e < V; ++e) fa[e] = fq[e] = 0.f;
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    float f[V];
                    RV::unpack(row_of(i), f);
#pragma unroll
                    for (int e = 0; e < V; ++e) {
                        const float d = in[i] ? f[e] - p[e] : 0.f;
                        fa[e] += d;
                        fq[e] = fmaf(d, d, fq[e]);
                    }
                }
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    a[e] += double(fa[e]);
                    q[e] += double(fq[e]);
                }
            }
            if constexpr (!kTight) {                        // (the sums keep pace with the loads, or the registers run out)
#pragma unroll
                for (int e = 0; e < V; ++e) asm volatile("" : "+v"(a[e]), "+v"(q[e]));
            }
        };
        typedef std::integral_constant<int, 4> four;
        // Rows that are not kept are read for the statistics if they are in S: two batches of eight in flight.
        auto passing = [&]() {
            const uint32_t rb = walk_from(0).row;
            auto batch = [&](raw_t(&w)[8], int k) {
                bool any = false;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const uint32_t row = rb + uint32_t(k + i) * step;
                    any |= row < A.M && in_set(A, set, row);
                }
                if (any) {
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        w[i] = row_load<T, V, false>(at_byte(x, min((rb + uint32_t(k + i) * step) * A.pitch + column, last)));
                }
                return any;
            };
            auto add8 = [&](const raw_t(&w)[8], int k) {
                Walk at = walk_from(k);
                add(four(), at, [&](int i) { return w[i]; });
                add(four(), at, [&](int i) { return w[4 + i]; });
            };
            raw_t w0[8], w1[8];
            bool any0 = batch(w0, K + L), any1 = false;
            for (int k = K + L; k < A.rounds; k += 16) {
                if (k + 8 < A.rounds) any1 = batch(w1, k + 8);
                if (any0) add8(w0, k);
                if (k + 8 >= A.rounds) break;
                if (k + 16 < A.rounds) any0 = batch(w0, k + 16);
                if (any1) add8(w1, k + 8);
            }
        };
        if (kAgain && A.rounds > K + L) passing();
        if constexpr (kAgain && L == 0) {
            if (set == 0) {
#pragma unroll
                for (int k = 0; k < K; ++k)
                    if (k < A.rounds) load(k);
            }
        }
        if constexpr (L > 0) {
            if (set == 0) {
#pragma unroll
                for (int k = 0; k < kAhead; ++k) load(k);
            }
            static_assert(L % 2 == 0, "pairs of rows");
            Walk w = walk_from(K);
#pragma unroll
            for (int k = 0; k < L; k += 2) {
                if (set == 0) {
                    park[k * kRowThreads + threadIdx.x] = u[k];
                    park[(k + 1) * kRowThreads + threadIdx.x] = u[k + 1];
                }
                add(std::integral_constant<int, 2>(), w, [&](int i) { return set == 0 ? u[k + i] : park[(k + i) * kRowThreads + threadIdx.x]; });
            }
        }
        Walk w = walk_from(0);
#pragma unroll
        for (int k = 0; k < K; k += 4) {
            if (set == 0) {
#pragma unroll
                for (int i = k + kAhead; i < k + kAhead + 4 && i < K; ++i) load(i);
            }
            if (!kTight || k < A.rounds) {
                static_assert(K % 4 == 0, "four rows at a time");
                if constexpr (!kTight) {
#pragma unroll
                    for (int i = k; i < k + 4; ++i) opaque_raw(v[i]);
                }
                add(four(), w, [&](int i) { return v[k + i]; });
            }
        }
        double t1, t2;
        if (kStow && set == 0 && leads) channel();
        tile_sums<V>(A, l, a, q, lds, part, t1, t2);
        tile_publish(A, l, stamp, set, t1, t2);
        if (set == 0) {
            s1 = t1;
            s2 = t2;
        } else {
            u1 = t1;
            u2 = t2;
        }
    }
    if (leads) {
        if (kStow) consts[threadIdx.x] = float4{ga, be, rm, rv};
        else channel();
    }
    tile_collect(A, l, stamp, 0, part, lost, s1, s2);
    if (MIXED) tile_collect(A, l, stamp, 1, part, lost, u1, u2);
    if (leads) {
        if (kStow) {
            const float4 w = consts[threadIdx.x];
            ga = w.x;
            be = w.y;
            rm = w.z;
            rv = w.w;
        }
        const double m1 = s1 * F.inv_s64;
        double mean = double(piv[threadIdx.x]) + m1;
        double var = s2 * F.inv_s64 - m1 * m1;
        if (!(var >= 0.0)) var = (var != var) ? var : 0.0;  // clamp rounding; keep NaN visible
        if constexpr (MIXED) {
            const double mv = u1 * F.inv_s_v;
            const double e_v = double(piv[kRowMaxTile + threadIdx.x]) + mv;
            double var_v = u2 * F.inv_s_v - mv * mv;
            if (!(var_v >= 0.0)) var_v = (var_v != var_v) ? var_v : 0.0;
            if (l.j == 0) {
                F.mean_parts[c] = float(e_v);
                F.mean_parts[F.C + c] = float(mean);
            }
            const double bm = double(F.mix_beta);
            mean = bm * e_v + (1.0 - bm) * mean;
            var = bm * var_v + (1.0 - bm) * var;
        }
        const float mu = float(mean);
        const float r = float(inv_sqrt(var + double(F.eps)));
        if (l.j == 0) {
            F.save_mean[c] = mu;
            F.save_invstd[c] = r;
            const double al = double(F.momentum);
            // (a wait for a team-mate that ran out leaves NaN statistics in its channel, whose moving averages then stay as they are)
            const bool arrived = F.T == 1 || lost[threadIdx.x] == 0u;
            if (F.running_mean && arrived) F.running_mean[c] = float((1.0 - al) * double(rm) + al * mean);
            if (F.running_var && arrived) F.running_var[c] = float((1.0 - al) * double(rv) + al * var);
        }
        consts[threadIdx.x] = float4{mu, ga * r, be, 0.f};
    }
    __syncthreads();
    if (l.live) {
        float mu[V], sc[V], sh[V];
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const float4 k4 = consts[l.local + e];
            mu[e] = k4.x;
            sc[e] = k4.y;
            sh[e] = k4.z;
        }
        auto finish = [&](const raw_t& w, const Walk& at) {
            float f[V];
            RV::unpack(w, f);
#pragma unroll
            for (int e = 0; e < V; ++e) f[e] = fmaf(f[e] - mu[e], sc[e], sh[e]);
            if (at.row < A.M) row_store<T, V, SHARED>(at_byte(y, at.off), RV::pack(f));
        };
        Walk w = walk_from(0);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (!kTight || k < A.rounds) {
                opaque_raw(v[k]);
                finish(v[k], w);
                w.next(step, hop);
            }
        }
        if constexpr (kAgain) {
#pragma unroll
            for (int k = 0; k < L; ++k) {
                finish(park[k * kRowThreads + threadIdx.x], w);
                w.next(step, hop);
            }
            for (int k = K + L; k < A.rounds; k += kRowBatch) {
                raw_t r[kRowBatch];
                Walk wr = w;
#pragma unroll
                for (int i = 0; i < kRowBatch; ++i) {
                    r[i] = row_load<T, V, true>(at_byte(x, min(wr.off, last)));
                    wr.next(step, hop);
                }
#pragma unroll
                for (int i = 0; i < kRowBatch; ++i) {
                    finish(r[i], w);
                    w.next(step, hop);
                }
            }
        }
    }
    team_done(F, l.j, stamp);
}

// Backward: the sums of Eq. 5, Eq. 6.  dy stays in registers (K rows) and LDS (L rows); x of the rows of S is read again (KEEPX:
// stays, too).  Loads as in the forward kernel.
template <typename T, int V, int K, int L, bool KEEPX, bool MIXED, bool SHARED>
__global__ __launch_bounds__(kRowThreads, 2) void nhwc_fused_backward_kernel(RowArgs A) {
    typedef RawVec<T, V> RV;
    typedef typename RV::raw_t raw_t;
    __shared__ raw_t park[L > 0 ? L * kRowThreads : 1];
    __shared__ float __attribute__((aligned(16))) lds[2 * kRowThreads * V];
    __shared__ pair_t part[kRowThreads];
    __shared__ float4 consts[(MIXED ? 2 : 1) * kRowMaxTile];
    __shared__ uint32_t words[3];
    touch_arguments<RowArgs>();
    const FusedArgs& F = A.f;
    const RowLane l = row_lane<V>(A);
    const T* x = static_cast<const T*>(F.x);
    const T* dy = static_cast<const T*>(F.dy);
    T* dx = static_cast<T*>(F.out);
    const unsigned long long state = stamp_request(F);
    const uint32_t step = uint32_t(F.T) * uint32_t(A.TY), hop = step * A.pitch;
    const uint32_t column = uint32_t(l.col) * uint32_t(sizeof(T)), last = (A.M - 1u) * A.pitch + column;
    typedef RowWalk<(K > 16)> Walk;
    auto walk_from = [&](int k) {
        const uint32_t row = uint32_t(l.j) * uint32_t(A.TY) + uint32_t(l.ty) + uint32_t(k) * step;
        return Walk{row, row * A.pitch + column};
    };
    float mu[V];
#pragma unroll
    for (int e = 0; e < V; ++e) mu[e] = F.save_mean[l.col + e];

    double a[V], q[V];
    float fa[V], fq[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
        a[e] = q[e] = 0.0;
        fa[e] = fq[e] = 0.f;
    }
    // Up to four rows are added in fp32 (add), their sum goes into the fp64 accumulator (flush).  Rows past the end, copies of
    // the last one, are dropped.
    const uint32_t block0 = uint32_t(l.j) * uint32_t(A.TY);
    auto add = [&](const raw_t& wg, const raw_t& wx, uint32_t row, int k) {
        const bool whole = block0 + uint32_t(k) * step + uint32_t(A.TY) <= A.M;            // (the same for the whole block)
        float g[V], t[V];
        RV::unpack(wg, g);
        RV::unpack(wx, t);
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const float h = whole || row < A.M ? g[e] : 0.f, d = whole || row < A.M ? t[e] - mu[e] : 0.f;
            fa[e] += h;
            fq[e] = fmaf(h, d, fq[e]);
            // (two channels at a time: with all eight of a bf16 vector unpacked at once 35 + 14 rows went through 48 bytes of scratch
            // memory; 16x512x1xW, 49 rows per thread, 1.00 -> 1.05 of the speed of 28 rows and no LDS)
            if (V == 8 && e % 2 == 1) asm volatile("" : "+v"(fa[e - e % 2]), "+v"(fq[e - e % 2]), "+v"(fa[e]), "+v"(fq[e]));
        }
    };
    auto flush = [&]() {
#pragma unroll
        for (int e = 0; e < V; ++e) {
            a[e] += double(fa[e]);
            q[e] += double(fq[e]);
            fa[e] = fq[e] = 0.f;
            asm volatile("" : "+v"(a[e]), "+v"(q[e]));
        }
    };
    raw_t g[K], xk[KEEPX ? K : 1];
    if constexpr (KEEPX) {
        static_assert(K <= 16, "all loads come before the first sum: only those that are needed");
        Walk wl = walk_from(0), w = wl;
        auto load = [&](int k) {
            const uint32_t off = min(wl.off, last);
            g[k] = row_load<T, V, true>(at_byte(dy, off));
            xk[k] = row_load<T, V, true>(at_byte(x, off));
            wl.next(step, hop);
        };
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (k < A.rounds) load(k);
#pragma unroll
        for (int k = 0; k < K; k += 4) {
            if (k < A.rounds) {
#pragma unroll
                for (int i = k; i < k + 4; ++i) {
                    opaque_raw(xk[i]);
                    add(g[i], xk[i], w.row, i);
                    w.next(step, hop);
                }
                flush();
            }
        }
    } else {
        auto first_pass = [&](auto plain) {
            constexpr bool kNt = !decltype(plain)::value;
            // Rows that are not kept come first, while the registers are free: dy is left in the memory-side cache.
            auto batch = [&](raw_t(&wg)[4], raw_t(&wx)[4], int k) {
                Walk w = walk_from(k);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t off = min(w.off, last);
                    wg[i] = row_load<T, V, false>(at_byte(dy, off));
                    wx[i] = row_load<T, V, kNt>(at_byte(x, off));
                    w.next(step, hop);
                }
            };
            auto add4 = [&](const raw_t(&wg)[4], const raw_t(&wx)[4], int k) {
                Walk w = walk_from(k);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    add(wg[i], wx[i], w.row, k + i);
                    w.next(step, hop);
                }
                flush();
            };
            if (K + L < A.rounds) {
                raw_t g0[4], x0[4], g1[4], x1[4], g2[4], x2[4];     // three batches in flight
                batch(g0, x0, K + L);
                if (K + L + 4 < A.rounds) batch(g1, x1, K + L + 4);
                for (int k = K + L;; k += 12) {
                    if (k + 8 < A.rounds) batch(g2, x2, k + 8);
                    add4(g0, x0, k);
                    if (k + 4 >= A.rounds) break;
                    if (k + 12 < A.rounds) batch(g0, x0, k + 12);
                    add4(g1, x1, k + 4);
                    if (k + 8 >= A.rounds) break;
                    if (k + 16 < A.rounds) batch(g1, x1, k + 16);
                    add4(g2, x2, k + 8);
                    if (k + 12 >= A.rounds) break;
                }
            }
            // The rows of LDS, then those of the registers: two rows of both tensors at a time, two such pairs in flight.
            static_assert(L % 2 == 0, "pairs of rows");
            Walk wl = walk_from(K), w = wl;
            raw_t d0[2], d1[2], x0[2], x1[2];
            auto request = [&](int k, raw_t(&d)[2], raw_t(&xb)[2]) {        // k: rows of LDS first, L of them
                if (k == L) wl = walk_from(0);
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    if (k + i < L + K) {
                        const uint32_t off = min(wl.off, last);
                        if (k < L) d[i] = row_load<T, V, true>(at_byte(dy, off));
                        else g[k + i - L] = row_load<T, V, true>(at_byte(dy, off));
                        xb[i] = row_load<T, V, kNt>(at_byte(x, off));
                        wl.next(step, hop);
                    }
            };
            auto take = [&](int k, raw_t(&d)[2], raw_t(&xb)[2]) {
                if (k == L) w = walk_from(0);
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    if (k + i < L + K) {
                        opaque_raw(xb[i]);
                        if (k < L) {
                            park[(k + i) * kRowThreads + threadIdx.x] = d[i];
                            add(d[i], xb[i], w.row, K + k + i);
                        } else {
                            add(g[k + i - L], xb[i], w.row, k + i - L);
                        }
                        w.next(step, hop);
                    }
                if (k % 4 == 2 || k + 2 >= L + K) flush();
            };
            request(0, d0, x0);
#pragma unroll
            for (int k = 0; k < L + K; k += 4) {
                if (k + 2 < L + K) request(k + 2, d1, x1);
                take(k, d0, x0);
                if (k + 4 < L + K) request(k + 4, d0, x0);
                if (k + 2 < L + K) take(k + 2, d1, x1);
            }
        };
        if (A.keep_x) first_pass(std::true_type());
        else first_pass(std::false_type());
    }
    stamp_accept(F, state, words);
    double s1, s2;
    tile_sums<V>(A, l, a, q, lds, part, s1, s2);            // (its barriers lie between the stamp's write and its first read)
    const uint32_t stamp = read_stamp(F, words);
    tile_publish(A, l, stamp, 0, s1, s2);
    const int c = l.tile * int(A.ct_div.d) + int(threadIdx.x);
    const bool leads = int(threadIdx.x) < l.width;
    float r = 0.f, ga = 0.f, centre = 0.f, e_v = 0.f;
    if (leads) {
        r = F.save_invstd[c];
        ga = F.gamma[c];
        centre = MIXED ? F.mean_parts[F.C + c] : F.save_mean[c];
        if (MIXED) e_v = F.mean_parts[c];
    }
    tile_collect(A, l, stamp, 0, part, nullptr, s1, s2);
    if (leads) {
        const float dbeta = float(s1);
        const float dgamma = float(s2 * double(r));
        if (l.j == 0) {
            F.dbeta[c] = dbeta;
            F.dgamma[c] = dgamma;
        }
        const float ar = ga * r, w = MIXED ? F.w_s : F.inv_s;
        consts[threadIdx.x] = float4{ar, ar * w * dbeta, ar * w * dgamma * r, centre};
        if (MIXED) consts[kRowMaxTile + threadIdx.x] = float4{0.f, ar * F.w_v * dbeta, ar * F.w_v * dgamma * r, e_v};
    }
    __syncthreads();
    if (l.live) {
        float ar[V], k1[V], k2[V], ce[V];
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const float4 kc = consts[l.local + e];
            ar[e] = kc.x;
            k1[e] = kc.y;
            k2[e] = kc.z;
            ce[e] = kc.w;
        }
        auto finish = [&](const raw_t& gr, const raw_t& xr, bool sampled, const Walk& at) {
            float f[V];
            RV::unpack(gr, f);
            if (MIXED && at.row < A.virtual_rows) {
                float fx[V];
                RV::unpack(xr, fx);
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const float4 kc = consts[kRowMaxTile + l.local + e];
                    f[e] = fmaf(ar[e], f[e], -fmaf(kc.z, fx[e] - kc.w, kc.y));
                }
            } else if (sampled) {
                float fx[V];
                RV::unpack(xr, fx);
#pragma unroll
                for (int e = 0; e < V; ++e) f[e] = fmaf(ar[e], f[e], -fmaf(k2[e], fx[e] - ce[e], k1[e]));
            } else {
#pragma unroll
                for (int e = 0; e < V; ++e) f[e] *= ar[e];
            }
            if (at.row < A.M) row_store<T, V, SHARED>(at_byte(dx, at.off), RV::pack(f));
        };
        auto sampled_here = [&](uint32_t row) { return row < A.M && ((MIXED && row < A.virtual_rows) || in_set(A, 0, row)); };
        Walk w = walk_from(0);
        // x of the rows of S is requested four rows at a time
#pragma unroll
        for (int k0 = 0; k0 < K + L; k0 += 4) {
            if (K <= 16 && k0 >= A.rounds) break;
            bool sampled[4];
            raw_t xr[4];
            Walk wx = w;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (k0 + i < K + L) {
                    sampled[i] = sampled_here(wx.row);
                    if constexpr (KEEPX) {
                        opaque_raw(xk[k0 + i]);
                        xr[i] = xk[k0 + i];
                    } else if (sampled[i]) {
                        xr[i] = row_load<T, V, true>(at_byte(x, wx.off));
                    }
                    wx.next(step, hop);
                }
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (k0 + i < K + L) {
                    if (k0 + i < K) {
                        opaque_raw(g[k0 + i < K ? k0 + i : 0]);
                        finish(g[k0 + i < K ? k0 + i : 0], xr[i], sampled[i], w);
                    } else {
                        finish(park[(k0 + i - K) * kRowThreads + threadIdx.x], xr[i], sampled[i], w);
                    }
                    w.next(step, hop);
                }
        }
        if constexpr (!KEEPX) {
            for (int k = K + L; k < A.rounds; k += kRowBatch) {
                raw_t r[kRowBatch], xr[kRowBatch];
                bool sampled[kRowBatch];
                Walk wr = w;
#pragma unroll
                for (int i = 0; i < kRowBatch; ++i) {
                    r[i] = row_load<T, V, true>(at_byte(dy, min(wr.off, last)));
                    sampled[i] = sampled_here(wr.row);
                    if (sampled[i]) xr[i] = row_load<T, V, true>(at_byte(x, wr.off));
                    wr.next(step, hop);
                }
#pragma unroll
                for (int i = 0; i < kRowBatch; ++i) {
                    finish(r[i], xr[i], sampled[i], w);
                    w.next(step, hop);
                }
            }
        }
    }
    team_done(F, l.j, stamp);
}

// Rows per thread up to which a block takes every row of its columns (13x29x7x10 bf16, 8 rows: 10.7 / 12.7 us against 10.0 /
// 8.7 streaming; 28x64x6x6 f32, 8 rows: forward 8.1 against 11.9; backward 52x349x4x4 f32, 7 rows, 12.7 against 10.5).
constexpr int row_solo(int V, bool backward) { return V == 8 ? (backward ? 4 : 5) : (backward ? 4 : 8); }

template <typename T, int V, int I, bool MIXED, bool FIRST, bool SHARED>
const void* row_forward() {
    constexpr RowsHeld h = rows_held(V, false, MIXED, I);
    return reinterpret_cast<const void*>(
        &nhwc_fused_forward_kernel<T, V, h.regs, FIRST ? 0 : h.park, MIXED, FIRST && (h.regs > kRowKeepX), SHARED>);
}
template <typename T, int V, int I, bool MIXED, bool SHARED>
const void* row_backward() {
    constexpr RowsHeld h = rows_held(V, true, MIXED, I);
    return reinterpret_cast<const void*>(&nhwc_fused_backward_kernel<T, V, h.regs, h.park, (h.regs <= kRowKeepX), MIXED, SHARED>);
}

template <typename T, int V>
const void* row_kernel(int variant, bool backward, bool mixed, bool first, bool shared) {
    constexpr bool kTiles = V > 1;                          // (fewer channels than a vector are one tile)
#define BNS_ROW_CASE(I)                                                                             \
    case I:                                                                                         \
        return backward ? (mixed    ? row_backward<T, V, I, true, false>()                           \
                           : shared ? row_backward<T, V, I, false, kTiles>()                         \
                                    : row_backward<T, V, I, false, false>())                         \
               : mixed  ? row_forward<T, V, I, true, false, false>()                                 \
               : shared ? (first ? row_forward<T, V, I, false, kTiles, kTiles>()                     \
                                 : row_forward<T, V, I, false, false, kTiles>())                     \
               : first  ? row_forward<T, V, I, false, kTiles, false>()                               \
                        : row_forward<T, V, I, false, false, false>();
    switch (variant) {
        BNS_ROW_CASE(0)
        BNS_ROW_CASE(1)
        BNS_ROW_CASE(2)
        BNS_ROW_CASE(3)
        BNS_ROW_CASE(4)
        BNS_ROW_CASE(5)
        BNS_ROW_CASE(6)
        BNS_ROW_CASE(7)
        BNS_ROW_CASE(8)
    }
#undef BNS_ROW_CASE
    static_assert(kRowVariants == 9, "one case each");
    return nullptr;
}

}  // namespace

hipError_t launch_nhwc_fused(const Dims& d, const IndexParams& ip, bool backward, const FusedIo& io, float eps, float momentum,
                             void* header, void* slots, size_t slot_bytes, hipStream_t st, const FusedMix* mix,
                             bool may_create_event, bool may_wait, bool* solo) {
    const bns_box& b = ip.shared;
    const int full = d.dtype == BNS_F32 ? 4 : 8, V = d.C < full ? 1 : full, opt = g_tuning.nhwc_fused;
    if (opt == 2 || g_tuning.nhwc_small == 2) return hipErrorNotSupported;
    const uint32_t M = uint32_t(d.N) * uint32_t(d.HW);
    int cus = 0;
    hipError_t e = device_units(&cus);
    if (e != hipSuccess) return e;
    // Column tiles of up to 128 channels, and never a last tile narrower than a vector.
    const int CV = (d.C + V - 1) / V;
    const size_t bytes = size_t(M) * size_t(d.C) * (d.dtype == BNS_F32 ? 4 : 2);
    auto lanes_for = [&](int lanes) {
        int t = std::min({CV, lanes, kRowMaxTile / V});
        while (d.C % V != 0 && t < CV && (CV - 1) % t == 0) ++t;
        return t;
    };
    auto groups_for = [&](int lanes) { return int((int64_t(M) + kRowThreads / lanes - 1) / (kRowThreads / lanes)); };
    const int want = g_tuning.nhwc_fused_lanes;
    int TX = lanes_for(want > 0 ? want : 4), T = 1, groups = groups_for(TX);   // rows TY at a time
    // Few rows: every block takes all rows of a narrow tile, and nothing crosses blocks.
    if (groups > row_solo(V, backward) || (opt == 1 && may_wait && M > 64u)) {
        if (opt != 1 && bytes <= kNhwcFusedBytes && M > kNhwcFewRows) return hipErrorNotSupported;
        // Width of a tile: 128 or 256 bytes where rows begin at multiples of 64 (a tile that shares its cache lines with the
        // next one costs a third: 63x160x44x44 f32 backward, us: 8 lanes 44, 9 lanes 82, 16 lanes 48), else 8 to 16 lanes; and what
        // leaves few lanes, threads and compute units without work, with a price on the T * CT pairs of sums that every member
        // reads (128x64x32x32 f32 forward: 128 members x 32 channels 17.6, 256 x 64 20.8; 50x150x19x19 f32: 85 x 52 13.5 / 14.9, 51 x
        // 32 12.5 / 13.9).  The times below are estimates, us, of what depends on the width.  Rows that begin on no 64 bytes: fitted to
        // 1800 passes over tensors of 0.2 to 130 MB, each timed with two to five widths; over 4100 further ones, with all of them, the tile it picks takes
        // 1.02 of the time of the best, 117 times more than 1.1, at most 1.42 (prices as for aligned rows, over the 1800: 1.03, 1.5).  That was with the non-temporal hint on all stores; without it on
        // shared lines (shares_lines), 98 layers with nine widths each: 1.01 of the best in both directions, none more than 1.08.  A line shared between tiles costs as much as 115 bytes of one's own (13x293x67x67 f32
        // forward, 8 lanes 61.9, 16 lanes 48.0); idle compute units cost less than their share, since small tensors do not fill
        // the memory's queues; 1024 pairs are polled in one go (25x382x8x8 bf16 forward, 8 members x 72 channels 9.2, 13 x 128 10.6).
        const bool aligned = size_t(d.C) * (d.dtype == BNS_F32 ? 4 : 2) % 64 == 0;
        double best = 0.0;
        for (int lanes = want > 0 ? want : 8; lanes <= (want > 0 ? want : 16); lanes += aligned ? 8 : 1) {
            const int tx = lanes_for(lanes), g = groups_for(tx), count = (CV + tx - 1) / tx;
            const int t = tile_members(g, tx * V, cus / count);
            // what a narrower tile, idle lanes, threads or compute units cost is a share of the time at the memory
            const double use = double(CV) / double(count * tx) * double(kRowThreads / tx * tx) / kRowThreads * std::min(1.0, double(count * t) / cus);
            const double moved = double(bytes) * (backward ? 3 : 2), pairs = double(t) * tx * V / 4096.0;
            const double time = aligned ? moved / 6.2e6 / use / ((tx > 8) == (V == 4) ? 1.0 : 0.97) + 1.1 * pairs
                                        : moved / 6.9e6 / std::sqrt(use * std::sqrt(use)) * (count > 1 ? 1.0 + 7.2 / tx : 1.0) *
                                                  (tx % 8 == 0 ? 1.0 : 1.07) + 2.1 * pairs + (pairs > 0.25 ? 0.7 : 0.0);
            if (tx * V <= kRowMaxTile && (best == 0.0 || time < best)) {
                best = time;
                TX = tx;
                groups = g;
                T = t;
            }
        }
        if (T == 1 && opt != 1) return hipErrorNotSupported;
    }
    if (TX * V > kRowMaxTile) return hipErrorNotSupported;
    const int tiles = (CV + TX - 1) / TX, TY = kRowThreads / TX, sets = mix && !backward ? 2 : 1;
    if (T > 1) {
        // Kernels whose blocks wait for each other stay out of HIP graphs in this layout: a replay beside other calls
        // could keep a block's team-mates off the device, and the streaming kernels have no such limit.
        if (!may_wait) return hipErrorNotSupported;
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        const bool known = hipStreamIsCapturing(st, &cap) == hipSuccess;
        (void)hipGetLastError();
        if (!known || cap != hipStreamCaptureStatusNone) return hipErrorNotSupported;
    }
    if (T > 1 && size_t(sets) * tiles * size_t(TX * V) * size_t(T) * 16 > slot_bytes) return hipErrorNotSupported;
    const int rounds = (groups + T - 1) / T;
    // Beyond what a block holds, rows are read twice, and the streaming kernels' short blocks do that faster; where the line
    // lies (us, streaming against this, forward / backward, 64x256xHxH): f32 44x44 (61 rows per thread), Batch Sampling 54.6 / 82.7 against
    // 50.3 / 66.9, a patch 54.9 / 82.2 against 51.7 / 67.9; 48x48 (72) 59.3 / 96.5 against 60.6 / 83.9, 58.3 / 96.0 against 62.8 / 83.0; 56x56 (98)
    // 76.6 / 127.7 against 83.4 / 119.1; 128 samples of it (196) 145 / 256 against 165 / 250; bf16 64x64 (64) 57.4 / 89.3 against 54.2 / 83.2, a
    // patch 57.9 / 90.2 against 62.2 / 94.5, 60x60 (57) 56.3 / 81.2 against 50.6 / 71.4; 72x72 (81) 69.9 / 109.9 against 68.0 / 109.1; 80x80 (100) 82.8 /
    // 132.2 against 84.3 / 138.2.
    // Full BN forward reads everything twice there, up to where little of it is left in the memory-side cache: f32 128 samples (196
    // rows) 201 against 179, 160 (245) 245 against 240, 192 (294) 295 against 296, 256 (392) 391 against 411; bf16 the same
    // rows, 320 samples 251 against 245, 512 398 against 410.
    // A last tile with idle lanes costs their share of the bandwidth: 41x80x80x80 f32 (20 of 24 lanes, 49 rows) forward 41.6
    // against 45.1, 26x80x100x101 (48) backward 69.9 against 74.4, 100x96x60x60 bf16 (12 of 16, 44 rows) backward 60.5 against 77.0, full BN
    // forward 45.8 against 40.4 with 46 rows, 78x80x70x70 64.9 against 69.8 with 72.
    const bool everything = b.n_cnt == d.N && b.h_cnt == d.H && b.w_cnt == d.W, idle = CV * 10 < tiles * TX * 9;
    const int most = rows_most(V, backward, mix != nullptr), regs = rows_in_registers(V, backward, mix != nullptr, false);
    // Rows that begin on no 64 bytes are slower the second time, too: 91x92x56x56 f32, a patch, 53 rows, backward 76.5 against 100.6
    // full BN forward, 56 rows, 57.8 against 73.9 (where streaming has to take narrower accesses for want of whole vectors, this is
    // still the faster).
    // (Since those are stored without the hint: 850 layers of 4 to 190 MB, streaming over this kernel, forward / backward.  Whole vectors, part of the rows, f32
    // 1.22 / 1.11 at 21 to 36 rows, 1.05 / 0.97 at 41 to 50, 0.89 / 0.91 at 51 to 64, 0.79 / 0.88 to 82: the line holds; bf16 1.14 / 1.06 at 21 to 36, but 1.36 / 1.08
    // at 41 to 50, six layers, which stay with streaming.)
    const bool split_lines = size_t(d.C) * (d.dtype == BNS_F32 ? 4 : 2) % 64 != 0 && d.C % V == 0;
    // Where streaming takes single elements the line lies further out: Eq. 4 backward 112x407x25x25 f32, 58 rows, 177.2 against 115.1, 19x659x53x53 bf16, 70 rows,
    // 157.5 against 82.3; backward with idle lanes 32x393x40x40 f32 116.2 against 76.8, 16x431x1xW bf16, 66 to 81 rows, twice the time; bf16 rows of
    // whole vectors 1.02 (66 rows) to 1.05 (81) the other way, 132 and 660 channels (64-bit accesses) forward, a patch, 44 to 60 rows, 1.1.  (Without the hint this kernel is ahead in f32 up to the last rows timed: streaming over
    // it 1.6 at 50 to 64 rows, 1.46 to 82, 1.34 to 130 forward, 1.5 to 1.6 backward, Eq. 4 forward 1.3 to 1.65 at 36 to 82; the lines below, drawn with it, still give
    // such layers to streaming forward: 33x209x67x67 f32 109.5 against 74.4 us.)
    const bool single = d.C % 4 != 0;
    const int limit = !backward && everything && !mix                         ? (idle && !single ? regs + regs * 2 / 5 : split_lines ? regs : 256)
                      : (idle && !single) || split_lines                      ? regs
                      : mix && (!backward || !single)                         ? (backward ? 64 : 34)
                      : backward                                              ? (V != 8 ? 128 : d.C % V == 0 ? 64 : 81)
                      : make_rowset(d, b).contiguous                          ? (V != 8 ? 66 : d.C % 8 == 4 ? 50 : 81)
                                                                              : (V != 8 ? 62 : d.C % 8 == 4 ? regs : 58);
    if (opt != 1 && T > 1 && rounds > limit) return hipErrorNotSupported;
    // Ragged bf16 rows of small tensors: streaming takes single elements, and that is enough (3x107x18x18, 208 KB, backward 8.0 against 14.2
    // us, 5x230x11x11, 278 KB, 9.1 / 8.2 against 9.5 / 9.3, 4x190x16x16, 389 KB, 8.8 / 8.0 against 9.6 / 9.6; 18x122x10x10, 439 KB, 10.8 / 9.9
    // against 9.6 / 9.1).  Of 200 drawn layers of 180 to 400 KB this launch took 1.04 of streaming's time forward and 1.11 backward; but 0.94
    // in full BN forward, 0.97 in Eq. 4 forward, and 0.87 (60 layers) where streaming has 64-bit accesses, which save it little: 8x28x23x23 (237 KB) 11.0
    // / 10.5 against 8.3 / 8.3.  (Below: 13x137x7x7, 175 KB, backward 9.4 against 10.3, 37x143x5x5, 265 KB, 11.6 / 11.2 against 9.4 / 9.8.)
    const bool elements = single && (backward || (!everything && !mix));
    if (opt != 1 && T > 1 && V == 8 && d.C % V != 0 && bytes < (elements ? 400000u : 180000u)) return hipErrorNotSupported;
    // bf16 rows that do not begin on cache lines: tiles of one and the same line are read by different blocks (us, streaming against this:
    // 12x432x73x70, 52 rows per thread, 34.7 / 45.7 against 37.8 / 50.9; 60x336x38x38, 28 rows, 38.4 / 53.7 against 41.0 / 54.1; 75x1296x15x16, 25 rows,
    // 34.1 / 44.6 against 34.2 / 39.5; 27x272x37x40, 12 rows, 23.7 / 31.5 against 22.7 / 22.9).
    // Full BN forward, which streaming reads twice as well, until it reads rows again itself (4x1736x84x84 70.7 against 65.5).
    const size_t pitch = size_t(d.C) * 2;
    // Backward, S part of the rows, the line also lies where streaming's column lanes are nearly all at work and rows are short (17 to 26 rows per
    // thread, 16x120x1xW (15 of 16 lanes) 32.9 / 34.2 to 42.5 / 43.5, 248 (31 of 32) 35.4 / 35.2 to 44.6 / 46.9; 336 (42 of 64) 41.7 / 33.6, 600
    // (75 of 128) 53.2 / 41.1, 72 (9 of 16) 49.4 / 35.7).
    const bool whole_lanes = CV <= 32 && CV % 16 != 0 && 10 * CV >= 9 * ((CV + 15) / 16 * 16);
    const int lines = !backward || (whole_lanes && !everything) ? 16 : 26;
    if (opt != 1 && T > 1 && rounds > lines && V == 8 && d.C % V == 0 && !(everything && !backward && rounds <= most) &&
        pitch % (backward ? 64 : 128) != 0)
        return hipErrorNotSupported;
    // Byte offsets are 32-bit.  Those of rows past the end may wrap: loads are clamped to the last row, so what is read lies in the
    // tensor, and sums and stores go by the row's number.
    if (bytes >= (size_t(1) << 32)) return hipErrorNotSupported;

    RowArgs A;
    FusedArgs& F = A.f;
    F = FusedArgs();
    F.x = io.x;
    F.dy = io.dy;
    F.out = io.out;
    F.gamma = io.gamma;
    F.beta = io.beta;
    F.save_mean = io.save_mean;
    F.save_invstd = io.save_invstd;
    F.running_mean = io.running_mean;
    F.running_var = io.running_var;
    F.dgamma = io.dgamma;
    F.dbeta = io.dbeta;
    F.hdr = static_cast<TeamHeader*>(header);
    F.slots = static_cast<unsigned long long*>(slots);
    F.C = d.C;
    F.T = T;
    F.num_teams = tiles;
    F.stamp_advance = 2u;
    F.stamp_seed = next_stamp_seed();
    const int spin = g_tuning.test_spin_limit;
    F.spin_limit = spin > 0 ? uint32_t(spin) : kSpinLimit;
    F.mute = g_tuning.test_mute_exchange;
    A.mute_channel = g_tuning.test_mute_channel;
    F.eps = eps;
    F.momentum = momentum;
    const double points = double(b.n_cnt) * double(b.h_cnt) * double(b.w_cnt);
    F.inv_s64 = 1.0 / points;
    F.inv_s = float(F.inv_s64);
    F.inv_s_v = 1.0;
    A.virtual_rows = 0;
    if (mix) {
        A.virtual_rows = uint32_t(mix->n_v) * uint32_t(d.HW);
        F.n_v = mix->n_v;
        F.mix_beta = mix->mix_beta;
        const double virtual_points = double(mix->n_v) * double(d.HW);
        F.inv_s_v = 1.0 / virtual_points;
        F.w_v = float(double(mix->mix_beta) / virtual_points);
        F.w_s = float((1.0 - double(mix->mix_beta)) / points);
        F.mean_parts = mix->mean_parts;
    }
    A.S = make_rowset(d, b);
    A.B = make_rowbox(d, b);
    A.s_lo = (uint32_t(b.n0) * uint32_t(d.H) + uint32_t(b.h0)) * uint32_t(d.W) + uint32_t(b.w0);
    A.tx_div = make_fastdiv(uint32_t(TX));
    A.ct_div = make_fastdiv(uint32_t(TX * V));
    A.tiles_div = make_fastdiv(uint32_t(tiles));
    A.eights = T / 8 * 8 * tiles;
    const int threads = kRowThreads / (TX * V);             // that share a channel
    const TileExchange exchange = tile_exchange(T, threads);
    A.sum_groups = std::min(threads, kSumGroups);
    A.member_groups = exchange.groups;
    A.polled = exchange.polled;
    for (int i = 0; i < kPivotRows; ++i)
        A.pivot_off[i] = sampled_row(A.S, std::min(uint32_t(i), A.S.pivot_rows - 1u)) * uint32_t(bytes / M);
    A.M = M;
    A.CV = CV;
    A.TY = TY;
    A.rounds = rounds;
    A.pitch = uint32_t(d.C) * (d.dtype == BNS_F32 ? 4u : 2u);
    A.keep_x = bytes <= kKeepBytes;
    const bool mixed = mix != nullptr, first = rows_first(rounds, V, backward, mixed, long(A.pitch));
    const bool shared = shares_lines(tiles, long(A.pitch), long(bytes), backward);
    const int variant = row_variant(rounds, V, backward, mixed);
    const void* kernel = V == 8               ? row_kernel<bf16_t, 8>(variant, backward, mixed, first, shared)
                         : V == 4             ? row_kernel<float, 4>(variant, backward, mixed, first, shared)
                         : d.dtype == BNS_F32 ? row_kernel<float, 1>(variant, backward, mixed, first, shared)
                                              : row_kernel<bf16_t, 1>(variant, backward, mixed, first, shared);
    *solo = T == 1;
    t_last_team[backward] = T;
    t_last_variant[backward] = 0;
    void* params[] = {&A};
    return launch_waiting(kernel, dim3(uint32_t(tiles) * uint32_t(T)), dim3(kRowThreads), params, T > 1, may_create_event, st);
}

}  // namespace bns
