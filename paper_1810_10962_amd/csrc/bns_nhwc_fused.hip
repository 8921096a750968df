// Single-launch kernels for the N x H x W x C layout: the statistics (or the sums of Eq. 5) and the element-wise pass of
// one direction in one kernel, with as much of the tensor as fits kept in registers in between.
//
// The tensor is a matrix of M = N*H*W rows by C columns.  A block of 512 threads owns a tile of CT <= 128 columns
// and one of T shares of the rows: thread (ty, tx) holds V channels of the rows (k * T + j) * TY + ty, so
// that the device as a whole walks the tensor front to back.  The first K of a thread's rows stay in registers; what does not
// fit is read again in the second phase, from the memory-side cache if it fits there (64x256x56x56 bf16 through the L2s, by
// counters: backward 370 MB, 308 are the least; forward 210, 206).  The T blocks of a tile exchange their column sums once,
// through the stamped slots of the other single-launch kernels (bns_fused_device.hpp); with T = 1 nothing crosses blocks.
//
// Bound by memory, by the exchange (about 3 us between the last load and the first store) and, where rows are read twice, by
// a persistent grid's shallower queue of loads.  Measured against the streaming kernels (three launches per direction), us
// forward / backward, Batch Sampling: 50x150x19x19 f32 13.8 / 15.5 against 17.7 / 25.4 (one element per access there);
// 64x512x14x14 bf16 14.7 / 15.9 against 19.1 / 25.6; 64x256x28x28 f32 24.1 / 32.5 against 31.8 / 40.8; 64x256x56x56 bf16
// 45.9 / 65.7 against 48.4 / 72.2 (the step of the benchmark 115 against 118; in its loops of one direction the forward gains nothing,
// 50.8 against 50.7), full BN 48.1 / 78.3 against 59.5 / 88.0.
//
// Columns that are no whole number of vectors: the last vector of a row is moved back so that it ends with the row.  The
// channels it shares with the vector before it are computed twice, with the same bits.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "bns_device.hpp"
#include "bns_fused_device.hpp"
#include "bns_internal.hpp"
#include "bns_nhwc_device.hpp"

namespace bns {

namespace {

constexpr int kRowThreads = 512;
constexpr int kRowMaxTile = 128;        // channels of a column tile
constexpr int kRowPoll = 8;             // team-mates polled at a time
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
    int32_t keep_x;         // backward: x is read again where it lies in S, leave it in the memory-side cache
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
    const int eights = A.f.T / 8 * 8 * A.f.num_teams, b = int(blockIdx.x);
    if (b >= eights) {
        l.j = b / A.f.num_teams;
        l.tile = b - l.j * A.f.num_teams;
    } else {
        const int e = b / (8 * A.f.num_teams), r = b - e * 8 * A.f.num_teams;
        l.tile = r / 8;
        l.j = e * 8 + r % 8;
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

// Column sums of the block, by thread t < CT for channel t of the tile: per-thread sums through LDS, added in fp64 in a
// fixed order (first over the row lanes q, q + Q, ..., then over q).
template <int V>
__device__ __forceinline__ void tile_sums(const RowArgs& A, const RowLane& l, const double (&a)[V], const double (&q)[V], float* lds,
                                          double* part, double& s1, double& s2) {
    const int CT = int(A.ct_div.d);
    __syncthreads();                                        // lds and part may still be read from the previous use
    if (l.live) {
#pragma unroll
        for (int e = 0; e < V; ++e) {
            lds[l.ty * CT + l.local + e] = float(a[e]);
            lds[(A.TY + l.ty) * CT + l.local + e] = float(q[e]);
        }
    }
    __syncthreads();
    const int g = int(fdiv(threadIdx.x, A.ct_div)), ch = int(threadIdx.x) - g * CT, Q = kRowThreads / CT;
    s1 = s2 = 0.0;
    if (g < Q && ch < l.width) {
        for (int r = g; r < A.TY; r += Q) {
            s1 += double(lds[r * CT + ch]);
            s2 += double(lds[(A.TY + r) * CT + ch]);
        }
        part[g * CT + ch] = s1;
        part[kRowThreads + g * CT + ch] = s2;
    }
    __syncthreads();
    if (int(threadIdx.x) < l.width) {
        for (int i = 1; i < Q; ++i) {
            s1 += part[i * CT + ch];
            s2 += part[kRowThreads + i * CT + ch];
        }
    }
}

// Exchange of the column sums between the T members of a tile: every member reads all T pairs of every channel.  Words are
// stamped as in the other single-launch kernels.  Slots: [set][tile][member][channel], so a member's pairs are written side by side.
__device__ __forceinline__ unsigned long long* pair_slot(const RowArgs& A, const RowLane& l, int set, int member, int ch) {
    const size_t tile = size_t(set * A.f.num_teams + l.tile), T = size_t(A.f.T), CT = A.ct_div.d;
    return A.f.slots + 2 * ((tile * T + size_t(member)) * CT + size_t(ch));
}
__device__ __forceinline__ void put_word(unsigned long long* p, uint32_t stamp, uint32_t payload) {
    __hip_atomic_store(p, (static_cast<unsigned long long>(stamp) << 32) | payload, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Waits until the N words that `at(i)` names carry the stamp; bounded like poll_pair.  False if the wait ran out.
template <int N, typename At>
__device__ __forceinline__ bool poll_words(const FusedArgs& F, uint32_t stamp, At&& at, uint32_t (&payload)[N]) {
    uint32_t limit = F.spin_limit;
    for (uint32_t spin = 0; spin < limit; ++spin) {
        unsigned long long w[N];
#pragma unroll
        for (int i = 0; i < N; ++i) w[i] = __hip_atomic_load(at(i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        bool all = true;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            all &= uint32_t(w[i] >> 32) == stamp;
            payload[i] = uint32_t(w[i]);
        }
        if (all) return true;
        if ((spin & 1023u) == 1023u && __hip_atomic_load(&F.hdr->expired, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u)
            limit = F.spin_limit / 64u + 1u;
        __builtin_amdgcn_s_sleep(2);
    }
    __hip_atomic_fetch_add(&F.hdr->expired, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return false;
}

// This member's pair of channel t: published by thread t.
__device__ __forceinline__ void tile_publish(const RowArgs& A, const RowLane& l, uint32_t stamp, int set, double s1, double s2) {
    if (A.f.T == 1 || int(threadIdx.x) >= l.width || A.f.mute) return;
    if (A.mute_channel == l.tile * int(A.ct_div.d) + int(threadIdx.x) + 1) return;
    unsigned long long* mine = pair_slot(A, l, set, l.j, int(threadIdx.x));
    put_word(mine, stamp, __float_as_uint(float(s1)));
    put_word(mine + 1, stamp, __float_as_uint(float(s2)));
}

// Adds the pairs of members first, first + step, ... of channel ch, B of them polled at a time.  If a wait ran out: NaN, and
// lost[ch] is set (lost = null: the caller does not ask).
template <int B>
__device__ __forceinline__ void add_members(const RowArgs& A, const RowLane& l, uint32_t stamp, int set, int ch, int first, int step,
                                            uint32_t* lost, double& s1, double& s2) {
    s1 = s2 = 0.0;
    for (int m0 = first; m0 < A.f.T; m0 += B * step) {
        uint32_t w[2 * B];
        const bool ok = poll_words<2 * B>(A.f, stamp, [&](int i) {
            return pair_slot(A, l, set, min(m0 + (i / 2) * step, A.f.T - 1), ch) + (i & 1);
        }, w);
        if (!ok) {
            s1 = s2 = __builtin_nan("");
            if (lost) lost[ch] = 1u;
            return;
        }
#pragma unroll
        for (int u = 0; u < B; ++u)
            if (m0 + u * step < A.f.T) {
                s1 += double(__uint_as_float(w[2 * u]));
                s2 += double(__uint_as_float(w[2 * u + 1]));
            }
    }
}

// Totals over the members, by thread t < CT.  Every sum is taken in a fixed order, so all members get the same bits.
// A wait that runs out leaves NaN in that channel and sets its word of lost.
__device__ __forceinline__ void tile_collect(const RowArgs& A, const RowLane& l, uint32_t stamp, int set, double* part, uint32_t* lost,
                                             double& s1, double& s2) {
    if (A.f.T == 1) return;
    const int CT = int(A.ct_div.d), T = A.f.T;
    const int g = int(fdiv(threadIdx.x, A.ct_div)), ch = int(threadIdx.x) - g * CT, Q = kRowThreads / CT;
    __syncthreads();                                        // part may still be read
    if (g < Q && ch < l.width) {
        add_members<kRowPoll>(A, l, stamp, set, ch, g, Q, lost, s1, s2);
        part[g * CT + ch] = s1;
        part[kRowThreads + g * CT + ch] = s2;
    }
    __syncthreads();
    if (int(threadIdx.x) < l.width) {
        for (int i = 1; i < Q && i < T; ++i) {
            s1 += part[i * CT + ch];
            s2 += part[kRowThreads + i * CT + ch];
        }
    }
}

template <typename T, int V, bool NT>
__device__ __forceinline__ typename RawVec<T, V>::raw_t row_load(const T* p) {
    typedef typename RawVec<T, V>::raw_t raw_t;
    typedef raw_t elem_t __attribute__((aligned(sizeof(T))));
    if (NT) return __builtin_nontemporal_load(reinterpret_cast<const elem_t*>(p));
    return *reinterpret_cast<const elem_t*>(p);
}
template <typename T, int V>
__device__ __forceinline__ void row_store(T* p, typename RawVec<T, V>::raw_t r) {
    typedef typename RawVec<T, V>::raw_t raw_t;
    typedef raw_t elem_t __attribute__((aligned(sizeof(T))));
    __builtin_nontemporal_store(r, reinterpret_cast<elem_t*>(p));
}

// Forward: Eq. 3 (Eq. 4 if MIXED), Eq. 8, Eq. 1.
template <typename T, int V, int K, bool MIXED>
__global__ __launch_bounds__(kRowThreads, 2) void nhwc_fused_forward_kernel(RowArgs A) {
    typedef RawVec<T, V> RV;
    __shared__ float lds[2 * kRowThreads * V];
    __shared__ double part[2 * kRowThreads];
    __shared__ float piv[(MIXED ? 2 : 1) * kRowMaxTile];
    __shared__ float4 consts[kRowMaxTile];
    __shared__ uint32_t words[3], lost[kRowMaxTile];
    const FusedArgs& F = A.f;
    const RowLane l = row_lane<V>(A);
    const size_t C = size_t(F.C);
    const T* x = static_cast<const T*>(F.x) + l.col;
    T* y = static_cast<T*>(F.out) + l.col;
    const unsigned long long state = stamp_request(F);
    const uint32_t step = uint32_t(F.T) * uint32_t(A.TY), last = A.M - 1u;

    // The pivot of a channel is the mean of its first few sampled rows (see coarse), read by the first row lane.
    typename RV::raw_t pv[kPivotRows], pw[MIXED ? kPivotRows : 1];
    if (l.ty == 0) {
#pragma unroll
        for (int i = 0; i < kPivotRows; ++i) {
            const uint32_t row = sampled_row(A.S, min(uint32_t(i), A.S.pivot_rows - 1u));
            pv[i] = row_load<T, V, false>(x + size_t(row) * C);
            if constexpr (MIXED) pw[i] = row_load<T, V, false>(x + size_t(min(uint32_t(i), A.virtual_rows - 1u)) * C);
        }
    }
    typename RV::raw_t v[K];
    auto keep_rows = [&]() {
        const uint32_t ra = opaque(uint32_t(l.j) * uint32_t(A.TY) + uint32_t(l.ty));
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (k < A.rounds) v[k] = row_load<T, V, true>(x + size_t(min(ra + uint32_t(k) * step, last)) * C);
    };
    if (K <= 16) keep_rows();
    if (l.ty == 0 && l.live) {
        float p[V], f[V];
#pragma unroll
        for (int e = 0; e < V; ++e) p[e] = 0.f;
#pragma unroll
        for (int i = 0; i < kPivotRows; ++i) {
            RV::unpack(pv[i], f);
#pragma unroll
            for (int e = 0; e < V; ++e) p[e] += uint32_t(i) < A.S.pivot_rows ? f[e] : 0.f;
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
#pragma unroll
    for (int set = 0; set < (MIXED ? 2 : 1); ++set) {
        double a[V], q[V];
        float p[V];
#pragma unroll
        for (int e = 0; e < V; ++e) {
            a[e] = q[e] = 0.0;
            p[e] = piv[set * kRowMaxTile + l.local + e];
        }
        // four rows at a time: their differences are added in fp32, the sum goes into the fp64 accumulator
        auto add4 = [&](const typename RV::raw_t (&w)[4], uint32_t row) {
            bool m[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t ru = row + uint32_t(u) * step;
                m[u] = ru < A.M && in_set(A, set, ru);
            }
            if (m[0] | m[1] | m[2] | m[3]) {
                float d[4][V];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    RV::unpack(w[u], d[u]);
#pragma unroll
                    for (int e = 0; e < V; ++e) d[u][e] = m[u] ? d[u][e] - p[e] : 0.f;
                }
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    a[e] += double((d[0][e] + d[1][e]) + (d[2][e] + d[3][e]));
                    q[e] += double(fmaf(d[3][e], d[3][e], fmaf(d[2][e], d[2][e], fmaf(d[1][e], d[1][e], d[0][e] * d[0][e]))));
                }
            }
        };
        const uint32_t rb = opaque(uint32_t(l.j) * uint32_t(A.TY) + uint32_t(l.ty));
        // Rows that are not kept are read for the statistics if they are in S: two batches of eight in flight.  Those of the
        // first set come before the rows that are kept, while the registers are free.
        auto passing = [&]() {
            auto batch = [&](typename RV::raw_t(&w)[8], int k) {
                bool any = false;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const uint32_t row = rb + uint32_t(k + u) * step;
                    any |= row < A.M && in_set(A, set, row);
                }
                if (any) {
#pragma unroll
                    for (int u = 0; u < 8; ++u) w[u] = row_load<T, V, false>(x + size_t(min(rb + uint32_t(k + u) * step, last)) * C);
                }
                return any;
            };
            auto add8 = [&](const typename RV::raw_t(&w)[8], int k) {
                const typename RV::raw_t lo[4] = {w[0], w[1], w[2], w[3]}, hi[4] = {w[4], w[5], w[6], w[7]};
                add4(lo, rb + uint32_t(k) * step);
                add4(hi, rb + uint32_t(k + 4) * step);
            };
            typename RV::raw_t w0[8], w1[8];
            bool any0 = batch(w0, K), any1 = false;
            for (int k = K; k < A.rounds; k += 16) {
                if (k + 8 < A.rounds) any1 = batch(w1, k + 8);
                if (any0) add8(w0, k);
                if (k + 8 >= A.rounds) break;
                if (k + 16 < A.rounds) any0 = batch(w0, k + 16);
                if (any1) add8(w1, k + 8);
            }
        };
        if (K > 16 && A.rounds > K) passing();
        if (K > 16 && set == 0) keep_rows();
#pragma unroll
        for (int k = 0; k < K; k += 4) {
            if (k < A.rounds) {
                const typename RV::raw_t w[4] = {v[k], v[k + 1], v[k + 2], v[k + 3]};
                add4(w, rb + uint32_t(k) * step);
            }
        }
        double t1, t2;
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
    float ga = 0.f, be = 0.f, rm = 0.f, rv = 0.f;
    const int c = l.tile * int(A.ct_div.d) + int(threadIdx.x);
    const bool leads = int(threadIdx.x) < l.width;
    if (leads) {
        ga = F.gamma[c];
        be = F.beta[c];
        if (l.j == 0 && F.running_mean) rm = F.running_mean[c];
        if (l.j == 0 && F.running_var) rv = F.running_var[c];
    }
    tile_collect(A, l, stamp, 0, part, lost, s1, s2);
    if (MIXED) tile_collect(A, l, stamp, 1, part, lost, u1, u2);
    if (leads) {
        const double m1 = s1 / F.s;
        double mean = double(piv[threadIdx.x]) + m1;
        double var = s2 / F.s - m1 * m1;
        if (!(var >= 0.0)) var = (var != var) ? var : 0.0;  // clamp rounding; keep NaN visible
        if constexpr (MIXED) {
            const double mv = u1 / F.s_v;
            const double e_v = double(piv[kRowMaxTile + threadIdx.x]) + mv;
            double var_v = u2 / F.s_v - mv * mv;
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
        const float r = float(1.0 / sqrt(var + double(F.eps)));
        if (l.j == 0) {
            F.save_mean[c] = mu;
            F.save_invstd[c] = r;
            const double al = double(F.momentum);
            // (a wait for a team-mate that ran out leaves NaN statistics in its channel, whose moving averages then stay as they are)
            const bool arrived = F.T == 1 || static_cast<volatile uint32_t*>(lost)[threadIdx.x] == 0u;
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
        const uint32_t rc = opaque(uint32_t(l.j) * uint32_t(A.TY) + uint32_t(l.ty));
        auto finish = [&](const typename RV::raw_t& w, uint32_t row) {
            float f[V];
            RV::unpack(w, f);
#pragma unroll
            for (int e = 0; e < V; ++e) f[e] = fmaf(f[e] - mu[e], sc[e], sh[e]);
            if (row < A.M) row_store<T, V>(y + size_t(row) * C, RV::pack(f));
        };
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (k < A.rounds) {
                opaque_raw(v[k]);
                finish(v[k], rc + uint32_t(k) * step);
            }
        }
        if (K > 16) {
            for (int k = K; k < A.rounds; k += kRowBatch) {
                typename RV::raw_t w[kRowBatch];
                const uint32_t row = rc + uint32_t(k) * step;
#pragma unroll
                for (int u = 0; u < kRowBatch; ++u) w[u] = row_load<T, V, true>(x + size_t(min(row + uint32_t(u) * step, last)) * C);
#pragma unroll
                for (int u = 0; u < kRowBatch; ++u) finish(w[u], row + uint32_t(u) * step);
            }
        }
    }
    team_done(F, l.j, stamp);
}

// Backward: the sums of Eq. 5, Eq. 6.  dy stays in registers; x of the rows of S is read again (KEEPX: stays, too).
template <typename T, int V, int K, bool KEEPX, bool MIXED>
__global__ __launch_bounds__(kRowThreads, 2) void nhwc_fused_backward_kernel(RowArgs A) {
    typedef RawVec<T, V> RV;
    typedef typename RV::raw_t raw_t;
    __shared__ float lds[2 * kRowThreads * V];
    __shared__ double part[2 * kRowThreads];
    __shared__ float4 consts[(MIXED ? 2 : 1) * kRowMaxTile];
    __shared__ uint32_t words[3];
    const FusedArgs& F = A.f;
    const RowLane l = row_lane<V>(A);
    const size_t C = size_t(F.C);
    const T* x = static_cast<const T*>(F.x) + l.col;
    const T* dy = static_cast<const T*>(F.dy) + l.col;
    T* dx = static_cast<T*>(F.out) + l.col;
    const unsigned long long state = stamp_request(F);
    const uint32_t step = uint32_t(F.T) * uint32_t(A.TY), last = A.M - 1u;
    float mu[V];
#pragma unroll
    for (int e = 0; e < V; ++e) mu[e] = F.save_mean[l.col + e];

    double a[V], q[V];
#pragma unroll
    for (int e = 0; e < V; ++e) a[e] = q[e] = 0.0;
    // four rows at a time, rows k .. k + 3 of the thread: added in fp32, the sum goes into the fp64 accumulator.  Rows past the
    // end (copies of the last one, or never loaded) are dropped.
    const uint32_t block0 = uint32_t(l.j) * uint32_t(A.TY);
    auto add4 = [&](const raw_t(&wg)[4], const raw_t(&wx)[4], int k) {
        float p[4][V], t[4][V];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            float fx[V];
            RV::unpack(wg[u], p[u]);
            RV::unpack(wx[u], fx);
#pragma unroll
            for (int e = 0; e < V; ++e) t[u][e] = fx[e] - mu[e];
        }
        if (block0 + uint32_t(k + 3) * step + uint32_t(A.TY) > A.M) {       // (the same for the whole block)
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (block0 + uint32_t(l.ty) + uint32_t(k + u) * step >= A.M) {
#pragma unroll
                    for (int e = 0; e < V; ++e) p[u][e] = t[u][e] = 0.f;
                }
        }
#pragma unroll
        for (int e = 0; e < V; ++e) {
            a[e] += double((p[0][e] + p[1][e]) + (p[2][e] + p[3][e]));
            q[e] += double(fmaf(p[1][e], t[1][e], p[0][e] * t[0][e]) + fmaf(p[3][e], t[3][e], p[2][e] * t[2][e]));
        }
    };
    raw_t g[K], xk[KEEPX ? K : 1];
    const uint32_t r0 = opaque(uint32_t(l.j) * uint32_t(A.TY) + uint32_t(l.ty));
    constexpr int XB = K < 8 ? K : 8;                       // rows of x in flight beside those of dy
    if constexpr (KEEPX) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (k < A.rounds) {
                const size_t off = size_t(min(r0 + uint32_t(k) * step, last)) * C;
                g[k] = row_load<T, V, true>(dy + off);
                xk[k] = row_load<T, V, true>(x + off);
            }
#pragma unroll
        for (int k = 0; k < K; k += 4)
            if (k < A.rounds) {
                const raw_t wg[4] = {g[k], g[k + 1], g[k + 2], g[k + 3]}, wx[4] = {xk[k], xk[k + 1], xk[k + 2], xk[k + 3]};
                add4(wg, wx, k);
            }
    } else {
        auto first_pass = [&](auto plain) {
            constexpr bool kNt = !decltype(plain)::value;
            // Rows that are not kept come first, while the registers are free: dy is left in the memory-side cache.
            auto batch = [&](raw_t(&wg)[4], raw_t(&wx)[4], int k) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const size_t off = size_t(min(r0 + uint32_t(k + u) * step, last)) * C;
                    wg[u] = row_load<T, V, false>(dy + off);
                    wx[u] = row_load<T, V, kNt>(x + off);
                }
            };
            if (K < A.rounds) {
                raw_t g0[4], x0[4], g1[4], x1[4], g2[4], x2[4];     // three batches in flight
                batch(g0, x0, K);
                if (K + 4 < A.rounds) batch(g1, x1, K + 4);
                for (int k = K;; k += 12) {
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
#pragma unroll
            for (int k0 = 0; k0 < K; k0 += XB) {
                raw_t xv[XB];
                const uint32_t ra = opaque(r0);
#pragma unroll
                for (int u = 0; u < XB; ++u)
                    if (k0 + u < K && k0 + u < A.rounds)
                        g[k0 + u] = row_load<T, V, true>(dy + size_t(min(ra + uint32_t(k0 + u) * step, last)) * C);
#pragma unroll
                for (int u = 0; u < XB; ++u)
                    if (k0 + u < K && k0 + u < A.rounds)
                        xv[u] = row_load<T, V, kNt>(x + size_t(min(ra + uint32_t(k0 + u) * step, last)) * C);
#pragma unroll
                for (int u = 0; u < XB; u += 4)
                    if (k0 + u < K && k0 + u < A.rounds) {
                        const raw_t wg[4] = {g[k0 + u], g[k0 + u + 1], g[k0 + u + 2], g[k0 + u + 3]};
                        const raw_t wx[4] = {xv[u], xv[u + 1], xv[u + 2], xv[u + 3]};
                        add4(wg, wx, k0 + u);
                    }
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
        const uint32_t rc = opaque(uint32_t(l.j) * uint32_t(A.TY) + uint32_t(l.ty));
        auto finish = [&](raw_t gr, raw_t xr, bool sampled, uint32_t row) {
            float f[V];
            RV::unpack(gr, f);
            if (MIXED && row < A.virtual_rows) {
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
            if (row < A.M) row_store<T, V>(dx + size_t(row) * C, RV::pack(f));
        };
        auto sampled_here = [&](uint32_t row) { return row < A.M && ((MIXED && row < A.virtual_rows) || in_set(A, 0, row)); };
        // x of the rows of S is requested four rows at a time
#pragma unroll
        for (int k0 = 0; k0 < K; k0 += 4) {
            if (k0 < A.rounds) {
                bool sampled[4];
                raw_t xr[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint32_t row = rc + uint32_t(k0 + u) * step;
                    sampled[u] = sampled_here(row);
                    if constexpr (KEEPX) {
                        opaque_raw(xk[k0 + u]);
                        xr[u] = xk[k0 + u];
                    } else if (sampled[u]) {
                        xr[u] = row_load<T, V, true>(x + size_t(row) * C);
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    opaque_raw(g[k0 + u]);
                    finish(g[k0 + u], xr[u], sampled[u], rc + uint32_t(k0 + u) * step);
                }
            }
        }
        if constexpr (!KEEPX) {
            for (int k = K; k < A.rounds; k += kRowBatch) {
                raw_t w[kRowBatch], xr[kRowBatch];
                bool sampled[kRowBatch];
                const uint32_t row = rc + uint32_t(k) * step;
#pragma unroll
                for (int u = 0; u < kRowBatch; ++u) {
                    const uint32_t ru = row + uint32_t(u) * step;
                    w[u] = row_load<T, V, true>(dy + size_t(min(ru, last)) * C);
                    sampled[u] = sampled_here(ru);
                    if (sampled[u]) xr[u] = row_load<T, V, true>(x + size_t(ru) * C);
                }
#pragma unroll
                for (int u = 0; u < kRowBatch; ++u) finish(w[u], xr[u], sampled[u], row + uint32_t(u) * step);
            }
        }
    }
    team_done(F, l.j, stamp);
}

// Rows kept in registers per thread.  Backward keeps x beside dy up to 16 rows.
constexpr int kRowKeeps[] = {4, 8, 16, 40};     // (the last: see most_rows)
constexpr int kNumRowKeeps = sizeof(kRowKeeps) / sizeof(kRowKeeps[0]);
// Rows per thread up to which a block takes every row of its columns (13x29x7x10 bf16, 8 rows: 10.7 / 12.7 us against 10.0 /
// 8.7 streaming; 28x64x6x6 f32, 8 rows: forward 8.1 against 11.9; backward 52x349x4x4 f32, 7 rows, 12.7 against 10.5).
constexpr int row_solo(int V, bool backward) { return V == 8 ? (backward ? 4 : 5) : (backward ? 4 : 8); }
// What the registers hold beside the sums (Eq. 4 forward walks the rows twice).
constexpr int most_rows(int V, bool backward, bool mixed) {
    return backward ? (V == 8 ? 28 : 40) : mixed ? 20 : (V == 8 ? 36 : 40);
}

template <typename T, int V>
const void* row_kernel(int variant, bool backward, bool mixed) {
#define BNS_ROW_CASE(I, KF, KM, K, KX)                                                                                         \
    case I:                                                                                                             \
        if (backward)                                                                                                   \
            return mixed ? reinterpret_cast<const void*>(&nhwc_fused_backward_kernel<T, V, K, KX, true>)                \
                         : reinterpret_cast<const void*>(&nhwc_fused_backward_kernel<T, V, K, KX, false>);              \
        return mixed ? reinterpret_cast<const void*>(&nhwc_fused_forward_kernel<T, V, KM, true>)                         \
                     : reinterpret_cast<const void*>(&nhwc_fused_forward_kernel<T, V, KF, false>);
    switch (variant) {
        BNS_ROW_CASE(0, 4, 4, 4, true)
        BNS_ROW_CASE(1, 8, 8, 8, true)
        BNS_ROW_CASE(2, 16, 16, 16, true)
        BNS_ROW_CASE(3, most_rows(V, false, false), most_rows(V, false, true), most_rows(V, true, false), false)
    }
#undef BNS_ROW_CASE
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
        // next one costs a third: 63x160x44x44 f32 backward, us: 8 lanes 44, 9 lanes 82, 16 lanes 48), else 8 to 16 lanes, rather
        // more (12x432x73x70 bf16, 864 bytes per row: 9 lanes 56, 14 lanes 47); and what leaves few lanes, threads and compute
        // units without work, with a price on the T * CT pairs of sums that every member reads (128x64x32x32 f32 forward:
        // 128 members x 32 channels 17.6, 256 x 64 20.8).
        const bool aligned = size_t(d.C) * (d.dtype == BNS_F32 ? 4 : 2) % 64 == 0;
        double best = 0.0;
        for (int lanes = want > 0 ? want : 8; lanes <= (want > 0 ? want : 16); lanes += aligned ? 8 : 1) {
            const int tx = lanes_for(lanes), g = groups_for(tx), count = (CV + tx - 1) / tx;
            const int t = std::min((g + 3) / 4, std::max(1, cus / count));
            const double width = aligned ? ((tx > 8) == (V == 4) ? 1.0 : 0.97) : 1.0 + 0.02 * (tx - 8);
            const double pairs = double(t) * tx * V / 4096.0;
            const double score = double(CV) / double(count * tx) * double(kRowThreads / tx * tx) / kRowThreads *
                                 std::min(1.0, double(count * t) / cus) * width * std::max(0.1, 1.0 - 0.08 * std::max(0.0, pairs - 1.0));
            if (score > best) {
                best = score;
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
    // Beyond what the registers hold, rows are read twice, and the streaming kernels' short blocks do that faster; where the line
    // lies (us, streaming against this, forward / backward, 64x256xHxW): f32 40x40 (50 rows per thread), Batch Sampling
    // 44.0 / 71.2 against 43.8 / 58.5, a patch 47.1 / 71.1 against 47.6 / 58.9; 56x56 (98 rows) 76 / 130 against 83 / 130.
    // Full BN forward reads everything twice there, up to where little of it is left in the memory-side cache: f32 128 samples (196
    // rows) 196 against 187, 160 (245) 245 against 240, 192 (294) 295 against 296, 256 (392) 391 against 411; bf16 the same
    // rows, 320 samples 251 against 245, 512 398 against 410.
    // A last tile with idle lanes costs their share of the bandwidth: 41x80x80x80 f32 (20 of 24 lanes, 49 rows) forward 41.6
    // against 45.1, 100x96x60x60 bf16 (12 of 16, 44 rows) backward 60.5 against 77.0, 60x80x64x64 f32 backward 67.7 against 73.9, full BN
    // forward 45.8 against 40.4 with 46 rows, 78x80x70x70 64.9 against 69.8 with 72.
    const bool everything = b.n_cnt == d.N && b.h_cnt == d.H && b.w_cnt == d.W, idle = CV * 10 < tiles * TX * 9;
    const int most = most_rows(V, backward, mix != nullptr);
    // Rows that begin on no 64 bytes are slower the second time, too: 91x92x56x56 f32, a patch, 53 rows, backward 76.5 against 100.6
    // (where streaming has to take narrower accesses for want of whole vectors, this is still the faster).
    const bool split_lines = size_t(d.C) * (d.dtype == BNS_F32 ? 4 : 2) % 64 != 0 && d.C % V == 0;
    const int limit = !backward && everything && !mix                         ? (idle ? most + most * 2 / 5 : 256)
                      : idle || split_lines                                   ? most
                      : backward                                              ? 64
                      : make_rowset(d, b).contiguous                          ? most + most * 2 / 5
                                                                              : most;
    if (opt != 1 && T > 1 && rounds > limit) return hipErrorNotSupported;
    // Ragged bf16 rows of small tensors: streaming takes single elements, and that is enough (13x137x7x7 backward 9.4 against 11.1 us,
    // 21x58x12x12 forward 9.8 against 11.2; 12x26x25x25, 390 KB, 9.9 / 11.2 against 10.5 / 10.1).
    if (opt != 1 && T > 1 && V == 8 && d.C % V != 0 && bytes < 400000) return hipErrorNotSupported;
    // bf16 rows that do not begin on cache lines: tiles of one and the same line are read by different blocks (12x432x73x70, us:
    // 42 / 52 against 35 / 48 streaming; 60x336x38x38 40 / 52 against 33 / 53; below 16 rows per thread this is the faster, forward
    // with rows that begin on no 64 bytes below 10: 27x272x37x40, 12 rows, 25.0 against 21.7, 10x176x68x68, 8 rows, 20.5 against 22.7).
    // Full BN forward, which streaming reads twice as well, until it reads rows again itself (4x1736x84x84 70.7 against 65.5).
    const size_t pitch = size_t(d.C) * 2;
    const int lines = backward || pitch % 64 == 0 ? 16 : 10;
    if (opt != 1 && T > 1 && rounds > lines && V == 8 && d.C % V == 0 && !(everything && !backward && rounds <= most) &&
        pitch % (backward ? 64 : 128) != 0)
        return hipErrorNotSupported;
    int variant = 0;
    while (variant + 1 < kNumRowKeeps && kRowKeeps[variant] < rounds) ++variant;

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
    F.s = double(b.n_cnt) * double(b.h_cnt) * double(b.w_cnt);
    F.inv_s = float(1.0 / F.s);
    F.s_v = 1.0;
    A.virtual_rows = 0;
    if (mix) {
        A.virtual_rows = uint32_t(mix->n_v) * uint32_t(d.HW);
        F.n_v = mix->n_v;
        F.mix_beta = mix->mix_beta;
        F.s_v = double(mix->n_v) * double(d.HW);
        F.w_v = float(double(mix->mix_beta) / F.s_v);
        F.w_s = float((1.0 - double(mix->mix_beta)) / F.s);
        F.mean_parts = mix->mean_parts;
    }
    A.S = make_rowset(d, b);
    A.B = make_rowbox(d, b);
    A.s_lo = (uint32_t(b.n0) * uint32_t(d.H) + uint32_t(b.h0)) * uint32_t(d.W) + uint32_t(b.w0);
    A.tx_div = make_fastdiv(uint32_t(TX));
    A.ct_div = make_fastdiv(uint32_t(TX * V));
    A.M = M;
    A.CV = CV;
    A.TY = TY;
    A.rounds = rounds;
    A.keep_x = bytes <= kKeepBytes;
    const bool mixed = mix != nullptr;
    const void* kernel = V == 8               ? row_kernel<bf16_t, 8>(variant, backward, mixed)
                         : V == 4             ? row_kernel<float, 4>(variant, backward, mixed)
                         : d.dtype == BNS_F32 ? row_kernel<float, 1>(variant, backward, mixed)
                                              : row_kernel<bf16_t, 1>(variant, backward, mixed);
    *solo = T == 1;
    void* params[] = {&A};
    return launch_waiting(kernel, dim3(uint32_t(tiles) * uint32_t(T)), dim3(kRowThreads), params, T > 1, may_create_event, st);
}

}  // namespace bns
