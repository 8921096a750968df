// Kernels for the N x H x W x C layout (the layout the paper writes its tensors in,
// Appendix A: B_l in R^{N x H x W x C}, statistics over dimensions 0, 1, 2).
//
// The tensor is a matrix of M = N*H*W rows and C columns, channels fastest.  Per-channel
// reductions are column sums; the location set S is a set of ROWS: a contiguous block of rows for
// Batch Sampling / NS / VDN, h_cnt runs of w_cnt consecutive rows per sample for Feature Sampling
// (one patch location per layer, as in Alg. 2).  A 128-bit access holds V consecutive channels of
// one row.
//
// All four streaming kernels share one decomposition.  A block is TX column lanes x TY row lanes
// (TX * TY = 256, TX = up to 64 accesses = one wave per row).  Block (tile, k) owns TX * V channels
// and the k-th share of the rows; a thread keeps the per-channel constants of its V channels in
// registers and walks its rows, so the element-wise passes load no parameter twice and divide
// nothing, and the reductions end with one LDS step over the TY row lanes and one partial per
// channel and block: partial[k][c].  The finalize kernels add the partials of a channel in a fixed
// order in fp64, so results are bit-identical from run to run.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "bns_device.hpp"
#include "bns_fused_device.hpp"
#include "bns_internal.hpp"
#include "bns_nhwc_device.hpp"

namespace bns {

namespace {

struct Tiling {
    int32_t C, CV;              // channels, channel vectors per row
    int32_t log2_tx, splits;    // TX = 1 << log2_tx column lanes; blocks along the rows
    uint32_t rows_per_block;
};

struct Lane {
    int tx, ty, TY, k, cv;
    bool live;
};

__device__ __forceinline__ Lane lane_of(const Tiling& t) {
    Lane l;
    const int TX = 1 << t.log2_tx;
    l.TY = kBlock >> t.log2_tx;
    l.tx = threadIdx.x & (TX - 1);
    l.ty = threadIdx.x >> t.log2_tx;
    const int tile = blockIdx.x / t.splits;
    l.k = blockIdx.x - tile * t.splits;
    l.cv = tile * TX + l.tx;
    l.live = l.cv < t.CV;
    return l;
}

// Adds a[], q[] over the TY row lanes of the block (fixed order) and writes one partial per channel.  lds: [2][TY][stride], 16-byte aligned.
// Every channel of the tile has a thread of its own, and reads of LDS are requested eight at a time.  (With the V channels of a vector
// left to one thread, one read after the other, this took 3 us of a block of 32 bf16 lanes and 7 us with two of them: 111x16x9x9 bf16, a patch of
// 2x2, statistics 8.5 -> 4.5 us, sums of Eq. 5 9.3 -> 4.3; 128x256x56x56 bf16, Batch Sampling, whole call 80.5 / 119.7 -> 77.2 / 117.0.)
template <int V>
__device__ __forceinline__ void write_partials(const float (&a)[V], const float (&q)[V], float* lds, const Tiling& t, const Lane& l,
                                               Partial* __restrict__ partial) {
    constexpr int kLog = V == 8 ? 3 : V == 4 ? 2 : 0, kWidth = V < 4 ? 1 : 4;
    typedef float vec_t __attribute__((ext_vector_type(kWidth)));
    const int log2_stride = t.log2_tx + kLog, stride = 1 << log2_stride;        // floats per row lane
    vec_t* va = reinterpret_cast<vec_t*>(lds + l.ty * stride + l.tx * V);
    vec_t* vq = reinterpret_cast<vec_t*>(lds + (l.TY + l.ty) * stride + l.tx * V);
#pragma unroll
    for (int i = 0; i < V; i += kWidth) {
        vec_t wa, wq;
#pragma unroll
        for (int e = 0; e < kWidth; ++e) {
            wa[e] = a[i + e];
            wq[e] = q[i + e];
        }
        va[i / kWidth] = wa;
        vq[i / kWidth] = wq;
    }
    __syncthreads();
    const int per = kBlock >> log2_stride;              // threads per channel of the tile (TY / V of them)
    int rows = l.TY;
    if (V > 1 && per >= 2) {
        // few channels, many row lanes: every thread adds a share of the row lanes of one channel (16 channels, 64 row lanes:
        // one thread per channel takes 63 dependent steps through LDS), then the shares of a channel are added in order
        const int ch = int(threadIdx.x) & (stride - 1), g = int(threadIdx.x) >> log2_stride;
        float ra[V], rq[V], sa = 0.f, sq = 0.f;
#pragma unroll
        for (int i = 0; i < V; ++i) {
            ra[i] = lds[(g + i * per) * stride + ch];
            rq[i] = lds[(l.TY + g + i * per) * stride + ch];
        }
#pragma unroll
        for (int i = 0; i < V; ++i) {
            sa += ra[i];
            sq += rq[i];
        }
        __syncthreads();
        lds[g * stride + ch] = sa;
        lds[(l.TY + g) * stride + ch] = sq;
        __syncthreads();
        rows = per;
    }
    const int first = (l.cv - l.tx) * V;                // the tile's first channel
    for (int ch = int(threadIdx.x); ch < stride && first + ch < t.C; ch += kBlock) {
        float sa = 0.f, sq = 0.f;
        for (int r = 0; r < rows; r += 8) {
            float ra[8], rq[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int row = min(r + i, rows - 1);
                ra[i] = lds[row * stride + ch];
                rq[i] = lds[(l.TY + row) * stride + ch];
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                sa = r + i == 0 ? ra[i] : r + i < rows ? sa + ra[i] : sa;
                sq = r + i == 0 ? rq[i] : r + i < rows ? sq + rq[i] : sq;
            }
        }
        partial[size_t(l.k) * t.C + size_t(first + ch)] = Partial{sa, sq};
    }
}

// Forward statistics (Eq. 3): partial[k][c] = (sum (x - p_c), sum (x - p_c)^2) over the k-th share of
// S, p_c = mean of x over the first few sampled rows.
//
// A row lane takes its rows kStatRows at a time.  The loads of the next batch are issued before the
// current one is added up, and the pivot rows travel together with the first batch, so a block with few
// rows (a small S spread over the whole device) waits for memory once and a block with many rows keeps
// two batches in flight.  Row indices past the end of the share are clamped to its last row and their
// terms dropped, so every load is unconditional.  CONTIG: the rows of S are one contiguous run (Batch
// Sampling, full BN, NS, the virtual set), so the sampled row needs no division.  KEEP: loads without the
// non-temporal hint, so that the normalization pass finds the rows of S in the memory-side cache.
constexpr int kStatRows = 8;

template <typename T, int V, bool CONTIG, bool KEEP>
__global__ __launch_bounds__(kBlock) void nhwc_stats_partial_kernel(const T* __restrict__ x,
                                                                    Partial* __restrict__ partial, RowSet S, Tiling t) {
    __shared__ __align__(16) float lds[2 * kBlock * V];
    __shared__ float piv[kWave * V];                             // at most 64 column lanes
    const Lane l = lane_of(t);
    const uint32_t i0 = uint32_t(l.k) * t.rows_per_block;
    const uint32_t i1 = min(i0 + t.rows_per_block, S.rows);      // i1 > i0: no block is empty
    const uint32_t TY = uint32_t(l.TY);
    const uint32_t step = uint32_t(kStatRows) * TY;
    const uint32_t batches = (i1 - i0 + step - 1u) / step;      // the same for every thread of the block
    float a[V], q[V], p[V];
    double A[V], Q[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
        a[e] = q[e] = p[e] = 0.f;
        A[e] = Q[e] = 0.0;
    }
    {
        // (lanes past the last channel vector repeat it: they take part in the barrier below and write nothing)
        const T* xc = x + size_t(l.live ? l.cv : t.CV - 1) * V;
        const uint32_t first = sampled_row(S, 0u);
        auto row_of = [&](uint32_t i) { return CONTIG ? first + i : sampled_row(S, i); };
        auto fetch = [&](Vec<T, V>(&v)[kStatRows], uint32_t i) {
#pragma unroll
            for (int u = 0; u < kStatRows; ++u) {
                const T* p = xc + size_t(row_of(min(i + uint32_t(u) * TY, i1 - 1u))) * t.C;
                if (KEEP) v[u].load(p); else v[u].load_nt(p);
            }
        };
        auto add = [&](const Vec<T, V>(&v)[kStatRows], uint32_t i) {
            if (i + uint32_t(kStatRows - 1) * TY < i1) {         // every row of the batch belongs to the share
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    float d[kStatRows];
#pragma unroll
                    for (int u = 0; u < kStatRows; ++u) d[u] = v[u].f[e] - p[e];
                    A[e] += double(((d[0] + d[1]) + (d[2] + d[3])) + ((d[4] + d[5]) + (d[6] + d[7])));
                    float sq = d[0] * d[0];
#pragma unroll
                    for (int u = 1; u < kStatRows; ++u) sq = fmaf(d[u], d[u], sq);
                    Q[e] += double(sq);
                }
            } else {
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    float d[kStatRows];
#pragma unroll
                    for (int u = 0; u < kStatRows; ++u) d[u] = i + uint32_t(u) * TY < i1 ? v[u].f[e] - p[e] : 0.f;
                    A[e] += double(((d[0] + d[1]) + (d[2] + d[3])) + ((d[4] + d[5]) + (d[6] + d[7])));
                    float sq = d[0] * d[0];
#pragma unroll
                    for (int u = 1; u < kStatRows; ++u) sq = fmaf(d[u], d[u], sq);
                    Q[e] += double(sq);
                }
            }
        };
        static_assert(kStatRows == 8, "the sums above are written out for eight rows");
        Vec<T, V> pv[kPivotRows], v0[kStatRows], v1[kStatRows];
        uint32_t i = i0 + uint32_t(l.ty);
        // The pivot rows are the same few rows for every block of the launch: only the first row lane of a block
        // reads them and hands the pivots to the others through LDS (every thread of every block reading them put
        // thousands of requests on the few L2 channels that hold those rows).
        if (l.ty == 0) {
#pragma unroll
            for (int j = 0; j < kPivotRows; ++j)     // no branches: all loads in flight together
                pv[j].load(xc + size_t(row_of(min(uint32_t(j), S.pivot_rows - 1u))) * t.C);
        }
        fetch(v0, i);
        if (l.ty == 0) {
#pragma unroll
            for (int j = 0; j < kPivotRows; ++j)
#pragma unroll
                for (int e = 0; e < V; ++e) p[e] += uint32_t(j) < S.pivot_rows ? pv[j].f[e] : 0.f;
#pragma unroll
            for (int e = 0; e < V; ++e) piv[l.tx * V + e] = coarse(p[e] * S.inv_pivot_rows);
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < V; ++e) p[e] = piv[l.tx * V + e];
        for (uint32_t b = 0; b < batches; b += 2u) {
            if (b + 1u < batches) fetch(v1, i + step);
            add(v0, i);
            if (b + 1u < batches) {
                if (b + 2u < batches) fetch(v0, i + 2u * step);
                add(v1, i + step);
            }
            i += 2u * step;
        }
#pragma unroll
        for (int e = 0; e < V; ++e) {
            a[e] = float(A[e]);
            q[e] = float(Q[e]);
        }
    }
    write_partials<V>(a, q, lds, t, l, partial);
}

// Backward sums of Eq. 5 over all M rows: partial[k][c] = (sum dy, sum dy * (x - mean_c)).
// OUTSIDE: the kernel also writes dx on the rows that are NOT in S.  The second branch of Eq. 6, dx = gamma r dy,
// needs none of the sums, and dy of those rows is in registers here anyway; what is left for after the sums are
// the rows of S alone (nhwc_dx_rows_kernel).  Backward then has to move (3 + 2r) e bytes per element instead of (4 + r) e.
// KEEP: what the dx pass reads again is loaded without the non-temporal hint, so that it stays in the memory-side
// cache: 1 = dy in the blocks of the first `keep_splits` row shares (as many as fit; the dx pass loads and stores
// with the hint, so what is cached stays until it gets there), 2 = dy and x everywhere (S is most of the rows and
// both fit), 0 = neither (dx is written here).
template <typename T, int V, bool OUTSIDE, int KEEP>
__device__ __forceinline__ void reduce_partial_body(const T* __restrict__ x, const T* __restrict__ dy,
                                                    const float* __restrict__ mean, Partial* __restrict__ partial,
                                                    const Tiling& t, uint32_t M, T* __restrict__ dx,
                                                    const float* __restrict__ gamma, const float* __restrict__ invstd,
                                                    const RowBox& B, float* lds, uint32_t keep_splits) {
    const Lane l = lane_of(t);
    const uint32_t r0 = uint32_t(l.k) * t.rows_per_block;
    const uint32_t r1 = min(r0 + t.rows_per_block, M);
    const uint32_t TY = uint32_t(l.TY);
    float a[V], q[V], mu[V], sc[V];
    double A[V], Q[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
        a[e] = q[e] = mu[e] = sc[e] = 0.f;
        A[e] = Q[e] = 0.0;
    }
    if (l.live) {
#pragma unroll
        for (int e = 0; e < V; ++e) mu[e] = mean[l.cv * V + e];
        if (OUTSIDE) {
#pragma unroll
            for (int e = 0; e < V; ++e) sc[e] = gamma[l.cv * V + e] * invstd[l.cv * V + e];      // a = gamma r
        }
        const size_t col = size_t(l.cv) * V;
        auto walk = [&](auto keep_dy, auto keep_x) {
            constexpr bool KD = decltype(keep_dy)::value, KX = decltype(keep_x)::value;
            uint32_t r = r0 + uint32_t(l.ty);
            for (; r + TY < r1; r += 2u * TY) {
                Vec<T, V> g[2], v[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const size_t off = size_t(r + uint32_t(u) * TY) * t.C + col;
                    if (KD) g[u].load(dy + off); else g[u].load_nt(dy + off);
                    if (KX) v[u].load(x + off); else v[u].load_nt(x + off);
                }
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    A[e] += double(g[0].f[e] + g[1].f[e]);
                    Q[e] += double(fmaf(g[1].f[e], v[1].f[e] - mu[e], g[0].f[e] * (v[0].f[e] - mu[e])));
                }
                if (OUTSIDE) {
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const uint32_t row = r + uint32_t(u) * TY;
                        if (!row_in(B, row)) {
#pragma unroll
                            for (int e = 0; e < V; ++e) g[u].f[e] *= sc[e];
                            g[u].store_nt(dx + size_t(row) * t.C + col);
                        }
                    }
                }
            }
            for (; r < r1; r += TY) {
                const size_t off = size_t(r) * t.C + col;
                Vec<T, V> g, v;
                if (KD) g.load(dy + off); else g.load_nt(dy + off);
                if (KX) v.load(x + off); else v.load_nt(x + off);
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    A[e] += double(g.f[e]);
                    Q[e] += double(g.f[e] * (v.f[e] - mu[e]));
                }
                if (OUTSIDE && !row_in(B, r)) {
#pragma unroll
                    for (int e = 0; e < V; ++e) g.f[e] *= sc[e];
                    g.store_nt(dx + off);
                }
            }
        };
        if constexpr (KEEP == 2) {
            walk(std::true_type(), std::true_type());
        } else if constexpr (KEEP == 1) {
            if (uint32_t(l.k) < keep_splits) walk(std::true_type(), std::false_type());      // (the same for the whole block)
            else walk(std::false_type(), std::false_type());
        } else {
            walk(std::false_type(), std::false_type());
        }
#pragma unroll
        for (int e = 0; e < V; ++e) {
            a[e] = float(A[e]);
            q[e] = float(Q[e]);
        }
    }
    write_partials<V>(a, q, lds, t, l, partial);
}

template <typename T, int V, int KEEP>
__global__ __launch_bounds__(kBlock) void nhwc_reduce_partial_kernel(const T* __restrict__ x, const T* __restrict__ dy,
                                                                     const float* __restrict__ mean,
                                                                     Partial* __restrict__ partial, Tiling t, uint32_t M,
                                                                     uint32_t keep_splits) {
    __shared__ __align__(16) float lds[2 * kBlock * V];
    reduce_partial_body<T, V, false, KEEP>(x, dy, mean, partial, t, M, nullptr, nullptr, nullptr, RowBox{}, lds, keep_splits);
}

template <typename T, int V>
__global__ __launch_bounds__(kBlock) void nhwc_reduce_outside_kernel(const T* __restrict__ x, const T* __restrict__ dy,
                                                                     const float* __restrict__ mean,
                                                                     Partial* __restrict__ partial, Tiling t, uint32_t M,
                                                                     T* __restrict__ dx, const float* __restrict__ gamma,
                                                                     const float* __restrict__ invstd, RowBox B) {
    __shared__ __align__(16) float lds[2 * kBlock * V];
    reduce_partial_body<T, V, true, 0>(x, dy, mean, partial, t, M, dx, gamma, invstd, B, lds, 0u);
}

// Sums and dx outside S as above for 16-byte vectors, front to back: block k takes the chunks k, k + splits, ... of
// kSplitRows rows per row lane, so that the whole launch reads and writes one window that moves through the tensors, as a flat
// copy does.  Loads alone do not mind blocks that each walk a share of their own; with stores between them that costs a
// fifth of the rate (128x256x56x56 f32, the whole backward pass: shares 255 us, front to back 231; 4.9 and 6.0 TB/s).
// The loads of the next chunk are issued before this one is added up and stored, and neither loads nor stores hang on a
// condition, which would make each wait one for everything in flight: a row past the end is loaded as the last one and left out of
// the sums, and rows that must not be written (those, and the rows of S) are stored to an offset beyond the buffer, which
// the address check drops.  Rows are added in pairs in fp32, pairs in fp64, as in reduce_partial_body.
// CONTIG: S is one run of rows.  KEEP: the chunks that hold it come last and are loaded without the non-temporal hint, so that
// nhwc_dx_rows_kernel finds them in the memory-side cache.
constexpr int kSplitRows = 4;

template <typename T, int V, bool CONTIG, bool KEEP>
__global__ __launch_bounds__(kBlock, 2) void nhwc_reduce_outside_ordered_kernel(
    const T* __restrict__ x, const T* __restrict__ dy, const float* __restrict__ mean, Partial* __restrict__ partial, Tiling t,
    uint32_t M, T* __restrict__ dx, const float* __restrict__ gamma, const float* __restrict__ invstd, RowBox B, uint32_t s_lo,
    uint32_t s_rows) {
    typedef RawVec<T, V> RV;
    typedef typename RV::raw_t raw_t;
    typedef uint32_t store_t __attribute__((ext_vector_type(4)));
    __shared__ __align__(16) float lds[2 * kBlock * V];
    Lane l = lane_of(t);
    const uint32_t tiles = gridDim.x / uint32_t(t.splits);              // the tiles of a chunk side by side
    l.k = int(blockIdx.x / tiles);
    l.cv = int((blockIdx.x - uint32_t(l.k) * tiles) << t.log2_tx) + l.tx;
    l.live = l.cv < t.CV;
    const uint32_t TY = uint32_t(l.TY), step = uint32_t(kSplitRows) * TY, chunks = (M + step - 1u) / step, G = uint32_t(t.splits);
    const uint32_t pitch = uint32_t(t.C) * uint32_t(sizeof(T));
    // (lanes past the last channel vector repeat it and store nothing)
    const uint32_t cv = uint32_t(l.live ? l.cv : t.CV - 1), col = cv * uint32_t(V * sizeof(T));
    float mu[V], sc[V], a[V], q[V];
    double A[V], Q[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
        mu[e] = mean[cv * V + e];
        sc[e] = gamma[cv * V + e] * invstd[cv * V + e];                 // a = gamma r
        A[e] = Q[e] = 0.0;
    }
    raw_t g[2][kSplitRows], v[2][kSplitRows];
    auto load = [&](int at, uint32_t chunk, auto kept) __attribute__((always_inline)) {
        const uint32_t r0 = chunk * step, rows = min(step, M - r0);
        const char* xb = reinterpret_cast<const char*>(x + size_t(r0) * t.C);
        const char* gb = reinterpret_cast<const char*>(dy + size_t(r0) * t.C);
#pragma unroll
        for (int u = 0; u < kSplitRows; ++u) {
            const uint32_t off = min(uint32_t(l.ty) + uint32_t(u) * TY, rows - 1u) * pitch + col;
            const raw_t* pg = reinterpret_cast<const raw_t*>(gb + off);
            const raw_t* px = reinterpret_cast<const raw_t*>(xb + off);
            g[at][u] = decltype(kept)::value ? *pg : __builtin_nontemporal_load(pg);
            v[at][u] = decltype(kept)::value ? *px : __builtin_nontemporal_load(px);
        }
    };
    auto add = [&](int at, uint32_t chunk) __attribute__((always_inline)) {
        const uint32_t r0 = chunk * step, rows = min(step, M - r0);
        const auto out = __builtin_amdgcn_make_buffer_rsrc(dx + size_t(r0) * t.C, 0, int(rows * pitch), 0x00027000);
        float p1[V], p2[V];
#pragma unroll
        for (int u = 0; u < kSplitRows; ++u) {
            const uint32_t r = uint32_t(l.ty) + uint32_t(u) * TY, row = r0 + r;
            const bool live = r < rows;
            float fg[V], fx[V];
            RV::unpack(g[at][u], fg);
            RV::unpack(v[at][u], fx);
#pragma unroll
            for (int e = 0; e < V; ++e) {
                const float d = live ? fx[e] - mu[e] : 0.f, h = live ? fg[e] : 0.f;
                if (u % 2 == 0) {
                    p1[e] = h;
                    p2[e] = h * d;
                } else {
                    A[e] += double(p1[e] + h);
                    Q[e] += double(fmaf(h, d, p2[e]));
                }
                fg[e] *= sc[e];
            }
            const bool in = CONTIG ? row - s_lo < s_rows : row_in(B, row);
            const uint32_t off = live && l.live && !in ? r * pitch + col : 0x7FFFFFF0u;
            union {
                raw_t raw;
                store_t words;
            } w;
            w.raw = RV::pack(fg);
            __builtin_amdgcn_raw_buffer_store_b128(w.words, out, int(off), 0, 2);        // 2: non-temporal
        }
    };
    // The chunks chunk_of(i), i = first, first + G, ... below count.
    auto walk = [&](uint32_t first, uint32_t count, auto kept, auto&& chunk_of) __attribute__((always_inline)) {
        if (first >= count) return;
        auto next = [&](uint32_t i) { return chunk_of(min(i, count - 1u)); };
        load(0, next(first), kept);
        for (uint32_t i = first; i < count; i += 2u * G) {
            load(1, next(i + G), kept);
            __builtin_amdgcn_sched_barrier(0);
            add(0, next(i));
            load(0, next(i + 2u * G), kept);
            __builtin_amdgcn_sched_barrier(0);
            if (i + G < count) add(1, next(i + G));
        }
    };
    const uint32_t k = uint32_t(l.k);
    if constexpr (KEEP) {
        const uint32_t c0 = s_lo / step, held = (s_lo + s_rows - 1u) / step + 1u - c0, rest = chunks - held;
        walk(k, rest, std::false_type(), [&](uint32_t i) { return i < c0 ? i : i + held; });
        walk((k + G - rest % G) % G, held, std::true_type(), [&](uint32_t i) { return c0 + i; });      // (those with a chunk less first)
    } else {
        walk(k, chunks, std::false_type(), [&](uint32_t i) { return i; });
    }
#pragma unroll
    for (int e = 0; e < V; ++e) {
        a[e] = float(A[e]);
        q[e] = float(Q[e]);
    }
    write_partials<V>(a, q, lds, t, l, partial);
}

// Finalize kernels: a block takes kFinCh neighbouring channels; thread (ch, kl) adds the partials
// k = kl, kl + kFinK, ... of channel ch in fp64 (a wave reads whole 64-byte runs of partial[k][.]),
// then thread ch adds the kFinK lane sums in index order.
constexpr int kFinCh = 8;
constexpr int kFinK = kBlock / kFinCh;

// The channel of a thread, and whether it is the one that gets the channel's sums.
__device__ __forceinline__ int led_channel() { return blockIdx.x * kFinCh + int(threadIdx.x % kFinCh); }
__device__ __forceinline__ bool leads_channel(int C) { return threadIdx.x / kFinCh == 0 && led_channel() < C; }

// A thread's share of a channel's partial sums.
__device__ __forceinline__ void share_of_splits(const Partial* __restrict__ partial, int C, int splits, double& a, double& b) {
    const int c = led_channel(), kl = threadIdx.x / kFinCh;
    a = b = 0.0;
    if (c >= C) return;
    int k = kl;
    for (; k + 15 * kFinK < splits; k += 16 * kFinK) {     // sixteen loads in flight, added in index order
        Partial p[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) p[u] = partial[size_t(k + u * kFinK) * C + c];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            a += double(p[u].a);
            b += double(p[u].b);
        }
    }
    for (; k < splits; k += 8 * kFinK) {                    // (one by one: 68 shares took three round trips)
        Partial p[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) p[u] = partial[size_t(min(k + u * kFinK, splits - 1)) * C + c];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            a += k + u * kFinK < splits ? double(p[u].a) : 0.0;
            b += k + u * kFinK < splits ? double(p[u].b) : 0.0;
        }
    }
}

// Adds the shares (a, b) of a channel's threads, in order; the thread that leads the channel gets them and true.
__device__ __forceinline__ bool sum_shares(int C, double a, double b, double* lds, double& s1, double& s2) {
    const int ch = threadIdx.x % kFinCh, kl = threadIdx.x / kFinCh;
    lds[kl * kFinCh + ch] = a;
    lds[(kFinK + kl) * kFinCh + ch] = b;
    __syncthreads();
    if (!leads_channel(C)) return false;
    s1 = s2 = 0.0;
#pragma unroll 1
    for (int j = 0; j < kFinK; j += 8) {
        double va[8], vb[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            va[u] = lds[(j + u) * kFinCh + ch];
            vb[u] = lds[(kFinK + j + u) * kFinCh + ch];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            s1 += va[u];
            s2 += vb[u];
        }
    }
    return true;
}

// The pivot of channel c, the same expression as in nhwc_stats_partial_kernel.
template <typename T>
__device__ __forceinline__ float column_pivot(const T* __restrict__ x, const RowSet& S, int C, int c) {
    float pv[kPivotRows], psum = 0.f;
#pragma unroll
    for (int j = 0; j < kPivotRows; ++j)
        pv[j] = load_scalar<T>(x + size_t(sampled_row(S, min(uint32_t(j), S.pivot_rows - 1u))) * C + c);
#pragma unroll
    for (int j = 0; j < kPivotRows; ++j) psum += uint32_t(j) < S.pivot_rows ? pv[j] : 0.f;
    return coarse(psum * S.inv_pivot_rows);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void nhwc_stats_finalize_kernel(
    const T* __restrict__ x, const Partial* __restrict__ partial, RowSet S, int C, int splits, float eps, float momentum,
    float* __restrict__ save_mean, float* __restrict__ save_invstd, float* __restrict__ running_mean,
    float* __restrict__ running_var) {
    __shared__ double lds[2 * kBlock];
    const int c = led_channel();
    double s1, s2, a, b;
    float pivot_f = 0.f, rm = 0.f, rv = 0.f;                // (requested ahead: the loads overlap those of the sums)
    if (leads_channel(C)) {
        pivot_f = column_pivot(x, S, C, c);
        if (running_mean) rm = running_mean[c];
        if (running_var) rv = running_var[c];
    }
    share_of_splits(partial, C, splits, a, b);
    if (!sum_shares(C, a, b, lds, s1, s2)) return;
    const double pivot = double(pivot_f);
    const double m1 = s1 * S.inv_rows;
    const double mean = pivot + m1;
    double var = s2 * S.inv_rows - m1 * m1;      // biased (1/s), Eq. 3
    if (var < 0.0) var = 0.0;
    save_mean[c] = float(mean);
    save_invstd[c] = float(inv_sqrt(var + double(eps)));
    const double al = double(momentum);                       // Eq. 8
    if (running_mean) running_mean[c] = float((1.0 - al) * double(rm) + al * mean);
    if (running_var) running_var[c] = float((1.0 - al) * double(rv) + al * var);
}

// "VDN + sampling" (Eq. 4): the sums of the sampled real set S and of the virtual set V (the first n_v
// samples), each into its own E and Var by Eq. 3, then the blend.
template <typename T>
__global__ __launch_bounds__(kBlock) void nhwc_stats_finalize_mixed_kernel(
    const T* __restrict__ x, const Partial* __restrict__ partial_s, int splits_s, const Partial* __restrict__ partial_v,
    int splits_v, RowSet S, RowSet Vs, int C, float mix_beta, float eps, float momentum, float* __restrict__ save_mean,
    float* __restrict__ save_invstd, float* __restrict__ mean_parts, float* __restrict__ running_mean,
    float* __restrict__ running_var) {
    __shared__ double lds[4 * kBlock];
    const int c = led_channel();
    double a1, a2, v1, v2, as, bs, av, bv;
    float pivot_s = 0.f, pivot_v = 0.f, rm = 0.f, rv = 0.f;
    if (leads_channel(C)) {
        pivot_s = column_pivot(x, S, C, c);
        pivot_v = column_pivot(x, Vs, C, c);
        if (running_mean) rm = running_mean[c];
        if (running_var) rv = running_var[c];
    }
    share_of_splits(partial_s, C, splits_s, as, bs);
    share_of_splits(partial_v, C, splits_v, av, bv);
    const bool lead_s = sum_shares(C, as, bs, lds, a1, a2);
    const bool lead_v = sum_shares(C, av, bv, lds + 2 * kBlock, v1, v2);
    if (!lead_s || !lead_v) return;
    const double ms = a1 * S.inv_rows, mv = v1 * Vs.inv_rows;
    const double e_s = double(pivot_s) + ms;
    const double e_v = double(pivot_v) + mv;
    double var_s = a2 * S.inv_rows - ms * ms, var_v = v2 * Vs.inv_rows - mv * mv;
    if (var_s < 0.0) var_s = 0.0;
    if (var_v < 0.0) var_v = 0.0;
    const double bm = double(mix_beta);
    const double mean = bm * e_v + (1.0 - bm) * e_s;            // Eq. 4, X = E
    const double var = bm * var_v + (1.0 - bm) * var_s;         // Eq. 4, X = Var
    save_mean[c] = float(mean);
    save_invstd[c] = float(inv_sqrt(var + double(eps)));
    mean_parts[c] = float(e_v);
    mean_parts[C + c] = float(e_s);
    const double al = double(momentum);                         // Eq. 8
    if (running_mean) running_mean[c] = float((1.0 - al) * double(rm) + al * mean);
    if (running_var) running_var[c] = float((1.0 - al) * double(rv) + al * var);
}

__global__ __launch_bounds__(kBlock) void nhwc_reduce_finalize_kernel(const Partial* __restrict__ partial, int C,
                                                                      int splits, const float* __restrict__ invstd,
                                                                      float* __restrict__ dgamma,
                                                                      float* __restrict__ dbeta) {
    __shared__ double lds[2 * kBlock];
    const int c = led_channel();
    double s1, s2, a, b;
    const float r = leads_channel(C) ? invstd[c] : 0.f;
    share_of_splits(partial, C, splits, a, b);
    if (!sum_shares(C, a, b, lds, s1, s2)) return;
    dbeta[c] = float(s1);
    dgamma[c] = float(s2 * double(r));
}

// Eq. 1 on every element.  var_eps >= 0: `invstd` holds variances (inference, Appendix D).
template <typename T, int V>
__global__ __launch_bounds__(kBlock) void nhwc_normalize_kernel(const T* __restrict__ x, T* __restrict__ y,
                                                                const float* __restrict__ gamma,
                                                                const float* __restrict__ beta,
                                                                const float* __restrict__ mean,
                                                                const float* __restrict__ invstd, Tiling t, uint32_t M,
                                                                float var_eps) {
    const Lane l = lane_of(t);
    if (!l.live) return;
    const uint32_t r0 = uint32_t(l.k) * t.rows_per_block;
    const uint32_t r1 = min(r0 + t.rows_per_block, M);
    const uint32_t TY = uint32_t(l.TY);
    float sc[V], mu[V], be[V], rs[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {       // every load first: one round trip to memory, not one per channel
        const int c = l.cv * V + e;
        sc[e] = gamma[c];
        rs[e] = invstd[c];
        mu[e] = mean[c];
        be[e] = beta[c];
    }
    if (var_eps >= 0.f) {
#pragma unroll
        for (int e = 0; e < V; ++e) rs[e] = 1.0f / sqrtf(rs[e] + var_eps);
    }
#pragma unroll
    for (int e = 0; e < V; ++e) sc[e] *= rs[e];
    const size_t col = size_t(l.cv) * V;
    uint32_t r = r0 + uint32_t(l.ty);
    for (; r + 3u * TY < r1; r += 4u * TY) {
        Vec<T, V> v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u].load_nt(x + size_t(r + uint32_t(u) * TY) * t.C + col);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
#pragma unroll
            for (int e = 0; e < V; ++e) v[u].f[e] = fmaf(v[u].f[e] - mu[e], sc[e], be[e]);
            v[u].store_nt(y + size_t(r + uint32_t(u) * TY) * t.C + col);
        }
    }
    for (; r < r1; r += TY) {
        Vec<T, V> v;
        v.load_nt(x + size_t(r) * t.C + col);
#pragma unroll
        for (int e = 0; e < V; ++e) v.f[e] = fmaf(v.f[e] - mu[e], sc[e], be[e]);
        v.store_nt(y + size_t(r) * t.C + col);
    }
}

// Eq. 6 on every element: rows outside S scale dy, rows in S also read x and take the 1/s terms.
//   dx = a g                                   a  = gamma r
//   dx = a g - (k1 (x - mean) + k2)            k1 = a r dgamma / s,  k2 = a dbeta / s
template <typename T, int V>
__global__ __launch_bounds__(kBlock) void nhwc_dx_kernel(const T* __restrict__ x, const T* __restrict__ dy,
                                                         T* __restrict__ dx, const float* __restrict__ gamma,
                                                         const float* __restrict__ mean,
                                                         const float* __restrict__ invstd,
                                                         const float* __restrict__ dgamma,
                                                         const float* __restrict__ dbeta, RowBox B, Tiling t,
                                                         uint32_t M, float inv_s) {
    const Lane l = lane_of(t);
    if (!l.live) return;
    const uint32_t r0 = uint32_t(l.k) * t.rows_per_block;
    const uint32_t r1 = min(r0 + t.rows_per_block, M);
    const uint32_t TY = uint32_t(l.TY);
    float a[V], mu[V], k1[V], k2[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
        const int c = l.cv * V + e;
        const float r = invstd[c];
        a[e] = gamma[c] * r;
        mu[e] = mean[c];
        k1[e] = a[e] * inv_s * (dgamma[c] * r);
        k2[e] = a[e] * inv_s * dbeta[c];
    }
    const size_t col = size_t(l.cv) * V;
    uint32_t r = r0 + uint32_t(l.ty);
    for (; r + 3u * TY < r1; r += 4u * TY) {
        Vec<T, V> g[4], v[4];
        bool in[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t row = r + uint32_t(u) * TY;
            g[u].load_nt(dy + size_t(row) * t.C + col);
            in[u] = row_in(B, row);
            if (in[u]) v[u].load_nt(x + size_t(row) * t.C + col);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (in[u]) {
#pragma unroll
                for (int e = 0; e < V; ++e) g[u].f[e] = fmaf(a[e], g[u].f[e], -fmaf(k1[e], v[u].f[e] - mu[e], k2[e]));
            } else {
#pragma unroll
                for (int e = 0; e < V; ++e) g[u].f[e] *= a[e];
            }
            g[u].store_nt(dx + size_t(r + uint32_t(u) * TY) * t.C + col);
        }
    }
    for (; r < r1; r += TY) {
        Vec<T, V> g;
        g.load_nt(dy + size_t(r) * t.C + col);
        if (row_in(B, r)) {
            Vec<T, V> v;
            v.load_nt(x + size_t(r) * t.C + col);
#pragma unroll
            for (int e = 0; e < V; ++e) g.f[e] = fmaf(a[e], g.f[e], -fmaf(k1[e], v.f[e] - mu[e], k2[e]));
        } else {
#pragma unroll
            for (int e = 0; e < V; ++e) g.f[e] *= a[e];
        }
        g.store_nt(dx + size_t(r) * t.C + col);
    }
}

// Eq. 6, first branch, on the rows of S alone (sampled row i of the k-th share, as in the statistics kernel); the
// other rows were written by nhwc_reduce_outside_kernel.
template <typename T, int V, bool CONTIG>
__global__ __launch_bounds__(kBlock) void nhwc_dx_rows_kernel(const T* __restrict__ x, const T* __restrict__ dy,
                                                              T* __restrict__ dx, const float* __restrict__ gamma,
                                                              const float* __restrict__ mean,
                                                              const float* __restrict__ invstd,
                                                              const float* __restrict__ dgamma,
                                                              const float* __restrict__ dbeta, RowSet S, Tiling t,
                                                              float inv_s) {
    const Lane l = lane_of(t);
    if (!l.live) return;
    const uint32_t i0 = uint32_t(l.k) * t.rows_per_block;
    const uint32_t i1 = min(i0 + t.rows_per_block, S.rows);
    const uint32_t TY = uint32_t(l.TY);
    float a[V], mu[V], k1[V], k2[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
        const int c = l.cv * V + e;
        const float r = invstd[c];
        a[e] = gamma[c] * r;
        mu[e] = mean[c];
        k1[e] = a[e] * inv_s * (dgamma[c] * r);
        k2[e] = a[e] * inv_s * dbeta[c];
    }
    const size_t col = size_t(l.cv) * V;
    const uint32_t first = sampled_row(S, 0u);
    auto row_of = [&](uint32_t i) { return CONTIG ? first + i : sampled_row(S, i); };
    uint32_t i = i0 + uint32_t(l.ty);
    for (; i + 3u * TY < i1; i += 4u * TY) {
        Vec<T, V> g[4], v[4];
        size_t off[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            off[u] = size_t(row_of(i + uint32_t(u) * TY)) * t.C + col;
            g[u].load_nt(dy + off[u]);
            v[u].load_nt(x + off[u]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
#pragma unroll
            for (int e = 0; e < V; ++e) g[u].f[e] = fmaf(a[e], g[u].f[e], -fmaf(k1[e], v[u].f[e] - mu[e], k2[e]));
            g[u].store_nt(dx + off[u]);
        }
    }
    for (; i < i1; i += TY) {
        const size_t off = size_t(row_of(i)) * t.C + col;
        Vec<T, V> g, v;
        g.load_nt(dy + off);
        v.load_nt(x + off);
#pragma unroll
        for (int e = 0; e < V; ++e) g.f[e] = fmaf(a[e], g.f[e], -fmaf(k1[e], v.f[e] - mu[e], k2[e]));
        g.store_nt(dx + off);
    }
}

// Backward of Eq. 4: rows of the first n_v samples belong to the virtual set (weight w_v = mix_beta / s_v,
// centre E[x_v]), rows of S to the sampled real set (w_s = (1 - mix_beta) / s_s, centre E[x_s]):
//   dx = a g - a w (dbeta + r dgamma (x - E_set)),   dx = a g elsewhere.
template <typename T, int V>
__global__ __launch_bounds__(kBlock) void nhwc_dx_mixed_kernel(
    const T* __restrict__ x, const T* __restrict__ dy, T* __restrict__ dx, const float* __restrict__ gamma,
    const float* __restrict__ invstd, const float* __restrict__ dgamma, const float* __restrict__ dbeta,
    const float* __restrict__ centre_v, const float* __restrict__ centre_s, RowBox B, uint32_t virtual_rows, float w_v,
    float w_s, Tiling t, uint32_t M) {
    const Lane l = lane_of(t);
    if (!l.live) return;
    const uint32_t r0 = uint32_t(l.k) * t.rows_per_block;
    const uint32_t r1 = min(r0 + t.rows_per_block, M);
    const uint32_t TY = uint32_t(l.TY);
    float a[V], cv_[V], cs_[V], k1[V], k2[V];          // k1, k2 per unit weight
#pragma unroll
    for (int e = 0; e < V; ++e) {
        const int c = l.cv * V + e;
        const float r = invstd[c];
        a[e] = gamma[c] * r;
        cv_[e] = centre_v[c];
        cs_[e] = centre_s[c];
        k1[e] = a[e] * (dgamma[c] * r);
        k2[e] = a[e] * dbeta[c];
    }
    const size_t col = size_t(l.cv) * V;
    for (uint32_t r = r0 + uint32_t(l.ty); r < r1; r += TY) {
        Vec<T, V> g;
        g.load_nt(dy + size_t(r) * t.C + col);
        const bool virt = r < virtual_rows;
        if (virt || row_in(B, r)) {
            Vec<T, V> v;
            v.load_nt(x + size_t(r) * t.C + col);
            const float w = virt ? w_v : w_s;
#pragma unroll
            for (int e = 0; e < V; ++e) {
                const float centre = virt ? cv_[e] : cs_[e];
                g.f[e] = fmaf(a[e], g.f[e], -w * fmaf(k1[e], v.f[e] - centre, k2[e]));
            }
        } else {
#pragma unroll
            for (int e = 0; e < V; ++e) g.f[e] *= a[e];
        }
        g.store_nt(dx + size_t(r) * t.C + col);
    }
}

inline uint32_t ceil_div_u(uint32_t a, uint32_t b) { return uint32_t((uint64_t(a) + b - 1) / b); }

inline int column_vec(const Dims& d) { return (d.dtype == BNS_BF16 && d.C % 8 == 0) ? 8 : (d.C % 4 == 0) ? 4 : 1; }

// Blocks: enough to fill the device a few times over.  Reductions (blocks > 0, or the reduction
// default) keep at least four rows per row lane and a bounded number of partials per channel.
// split_bound (optional): the number of splits before the rows are dealt out evenly.  It never decreases when
// `rows` or `blocks` grow, and the final t.splits never exceeds it -- unlike t.splits itself, which the
// rounding of rows_per_block makes non-monotonic (924 rows -> 55 splits, 896 rows -> 56).
Tiling make_tiling(const Dims& d, uint32_t rows, int blocks = 0, bool elementwise = false,
                   uint32_t* split_bound = nullptr) {
    Tiling t;
    const int V = column_vec(d);
    t.C = d.C;
    t.CV = d.C / V;
    int l = 0;
    while ((1 << l) < t.CV && l < 6) ++l;
    t.log2_tx = l;
    const uint32_t tiles = uint32_t((t.CV + (1 << l) - 1) >> l);
    const uint32_t TY = uint32_t(kBlock >> l);
    uint32_t s;
    if (elementwise) {
        // short blocks of a few rows per row lane (the launch then streams through memory front to back
        // like a flat kernel); fewer rows per lane when that would leave compute units idle
        s = ceil_div_u(rows, TY * uint32_t(tuned(g_tuning.nhwc_ew_rows, kNhwcEwRows)));
        const uint32_t fill = ceil_div_u(uint32_t(kNhwcFill), tiles), cap = rows / TY;
        if (s < fill) s = fill < cap ? fill : cap;
    } else {
        if (blocks <= 0) blocks = tuned(g_tuning.nhwc_blocks, kNhwcBlocks);
        s = ceil_div_u(uint32_t(blocks), tiles);
        const uint32_t cap = rows / (TY * 4u);
        if (s > cap) s = cap;
        // a row lane adds its rows one after the other in fp32: keep that chain short
        const uint32_t lo = ceil_div_u(rows, TY * uint32_t(kNhwcMaxLaneRows));
        if (s < lo) s = lo;
        if (s > uint32_t(kNhwcMaxSplits)) s = kNhwcMaxSplits;
    }
    if (s < 1u) s = 1u;
    while (uint64_t(tiles) * s > 0x7FFFFFFFu) s = (s + 1u) / 2u;      // grid.x limit
    if (split_bound) *split_bound = s;
    t.rows_per_block = ceil_div_u(rows, s);
    t.splits = int32_t(ceil_div_u(rows, t.rows_per_block));     // no empty blocks
    return t;
}

inline uint32_t grid_of(const Tiling& t) {
    const uint32_t tiles = uint32_t((t.CV + (1 << t.log2_tx) - 1) >> t.log2_tx);
    return tiles * uint32_t(t.splits);
}

template <int V>
using VecTag = std::integral_constant<int, V>;

template <typename F>
hipError_t dispatch_nhwc(const Dims& d, F&& f) {
    const int V = column_vec(d);
    if (d.dtype == BNS_F32) return V == 4 ? f(float(), VecTag<4>()) : f(float(), VecTag<1>());
    if (V == 8) return f(bf16_t(), VecTag<8>());
    return V == 4 ? f(bf16_t(), VecTag<4>()) : f(bf16_t(), VecTag<1>());
}

template <typename T, int V>
hipError_t launch_stats_partial(const T* x, Partial* partial, const RowSet& S, const Tiling& t, hipStream_t st) {
    const dim3 grid(grid_of(t)), block(kBlock);
    // the normalization pass reads the rows of S again
    const bool keep = keep_for_next_pass(size_t(S.rows) * size_t(t.C) * sizeof(T));
    if (S.contiguous) {
        if (keep) BNS_LAUNCH((nhwc_stats_partial_kernel<T, V, true, true>), grid, block, 0, st, x, partial, S, t);
        else BNS_LAUNCH((nhwc_stats_partial_kernel<T, V, true, false>), grid, block, 0, st, x, partial, S, t);
    } else {
        if (keep) BNS_LAUNCH((nhwc_stats_partial_kernel<T, V, false, true>), grid, block, 0, st, x, partial, S, t);
        else BNS_LAUNCH((nhwc_stats_partial_kernel<T, V, false, false>), grid, block, 0, st, x, partial, S, t);
    }
    return hipGetLastError();
}

}  // namespace

size_t nhwc_partial_bytes(const Dims& d) {
    // the most splits make_tiling can choose for any row set of this shape and any block target
    uint32_t bound = 1;
    make_tiling(d, uint32_t(d.N) * uint32_t(d.HW), kNhwcBlocksMax, false, &bound);
    return (size_t(bound) * size_t(d.C) * sizeof(Partial) + 255) & ~size_t(255);
}

namespace {
// The partial sums of `t` must fit the workspace region the API sized with nhwc_partial_bytes.
inline bool fits_region(const Dims& d, const Tiling& t) {
    return size_t(t.splits) * size_t(d.C) * sizeof(Partial) <= nhwc_partial_bytes(d);
}
}  // namespace

hipError_t launch_nhwc_stats(const Dims& d, const bns_box& b, const void* x, Partial* partial, float eps, float momentum,
                             float* save_mean, float* save_invstd, float* running_mean, float* running_var,
                             hipStream_t st) {
    const RowSet S = make_rowset(d, b);
    const Tiling t = make_tiling(d, S.rows);
    if (!fits_region(d, t)) return hipErrorInvalidValue;
    return dispatch_nhwc(d, [&](auto ty, auto vt) {
        using T = decltype(ty);
        constexpr int V = decltype(vt)::value;
        hipError_t e = launch_stats_partial<T, V>(static_cast<const T*>(x), partial, S, t, st);
        if (e != hipSuccess) return e;
        BNS_LAUNCH((nhwc_stats_finalize_kernel<T>), dim3(ceil_div_u(uint32_t(d.C), kFinCh)), dim3(kBlock), 0, st,
                   static_cast<const T*>(x), partial, S, d.C, t.splits, eps, momentum, save_mean, save_invstd,
                   running_mean, running_var);
        return hipGetLastError();
    });
}

hipError_t launch_nhwc_normalize(const Dims& d, const void* x, const float* gamma, const float* beta, const float* mean,
                                 const float* invstd, void* y, hipStream_t st, float var_eps) {
    const uint32_t M = uint32_t(d.N) * uint32_t(d.HW);
    const Tiling t = make_tiling(d, M, 0, true);
    return dispatch_nhwc(d, [&](auto ty, auto vt) {
        using T = decltype(ty);
        constexpr int V = decltype(vt)::value;
        BNS_LAUNCH((nhwc_normalize_kernel<T, V>), dim3(grid_of(t)), dim3(kBlock), 0, st, static_cast<const T*>(x),
                   static_cast<T*>(y), gamma, beta, mean, invstd, t, M, var_eps);
        return hipGetLastError();
    });
}

hipError_t launch_nhwc_reduce(const Dims& d, const void* x, const void* dy, const float* mean, const float* invstd,
                              Partial* partial, float* dgamma, float* dbeta, bool x_again, hipStream_t st) {
    const uint32_t M = uint32_t(d.N) * uint32_t(d.HW);
    const Tiling t = make_tiling(d, M);
    if (!fits_region(d, t)) return hipErrorInvalidValue;
    // dy of as many row shares as fit is left in the memory-side cache for the dx pass (x too when that pass reads
    // most of it again and both fit)
    const size_t bytes = size_t(M) * size_t(d.C) * (d.dtype == BNS_F32 ? 4 : 2);
    const size_t share = size_t(t.rows_per_block) * size_t(d.C) * (d.dtype == BNS_F32 ? 4 : 2);
    const int reuse = g_tuning.cache_reuse;
    const uint32_t keep_splits =
        reuse == 2 ? 0u : reuse == 1 ? uint32_t(t.splits) : uint32_t(std::min<size_t>(size_t(t.splits), kKeepBytes / share));
    const int keep = keep_splits == 0u ? 0 : (x_again && keep_for_next_pass(2 * bytes)) ? 2 : 1;
    return dispatch_nhwc(d, [&](auto ty, auto vt) {
        using T = decltype(ty);
        constexpr int V = decltype(vt)::value;
        const dim3 grid(grid_of(t)), block(kBlock);
        const T* xp = static_cast<const T*>(x);
        const T* gp = static_cast<const T*>(dy);
        if (keep == 2) BNS_LAUNCH((nhwc_reduce_partial_kernel<T, V, 2>), grid, block, 0, st, xp, gp, mean, partial, t, M, keep_splits);
        else if (keep == 1) BNS_LAUNCH((nhwc_reduce_partial_kernel<T, V, 1>), grid, block, 0, st, xp, gp, mean, partial, t, M, keep_splits);
        else BNS_LAUNCH((nhwc_reduce_partial_kernel<T, V, 0>), grid, block, 0, st, xp, gp, mean, partial, t, M, keep_splits);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        BNS_LAUNCH(nhwc_reduce_finalize_kernel, dim3(ceil_div_u(uint32_t(d.C), kFinCh)), dim3(kBlock), 0, st,
                   partial, d.C, t.splits, invstd, dgamma, dbeta);
        return hipGetLastError();
    });
}

// Does a whole backward call that the single launch does not take use the reduction that writes dx outside S front to back?  It can
// where accesses are 16 bytes and a chunk's offsets stay below 2^30.  It is the faster side (us, streaming against this)
//   * where S is small, since the rows of S are read again and those outside are not: 128x256x56x56 f32 a patch of 1/16 248 / 224,
//     Batch Sampling 1/8 251 / 223, 1/4 258 / 241, 3/4 289 / 294; bf16 1/8 129 / 117, 1/4 132 / 122, 1/2 140 / 139;
//   * where few column lanes idle: 120x1024x24x24 f32 179 / 152, 100x480x45x45 (120 of 128 lanes) 247 / 230, 40x200x70x70 (50 of 64)
//     103.0 / 105.4, 100x328x45x45 (82 of 128) 194 / 206;
//   * beyond a few launches' worth of bytes: 32x256x28x28 f32 (26 MB) 25.0 / 24.4, 6x128x28x28 (2.4 MB) 11.8 / 12.9;
//   * where rows are whole segments of 64 bytes in one, two, four or eight column tiles: the blocks of a tile write their share of a row
//     long after the other tiles' blocks wrote theirs.  Of 2673 further layers drawn so (C up to 3200, 16-420 MB, S up to 1/4, 7/8 of the
//     lanes) it is 1.08 times as fast in the mean and none loses 5 %; of 1799 in five to seven tiles 591 do, 99x1480x18x18 f32 Batch
//     Sampling 143.5 / 158.9, 6x1152x99x99 f32 180 / 207, except where S is contiguous and no lane idles (f32, three, five, six tiles: 1.03,
//     115 layers, one; bf16, three: 1.01, five of 117);
//   * rows that start anywhere only where S is contiguous and there are at most two tiles (1.03, 129 layers, none): a patch
//     22x1128x45x45 f32 147 / 175.
bool nhwc_split_ordered(const Dims& d, const bns_box& b) {
    const int opt = g_tuning.nhwc_split_ordered;
    const size_t size = d.dtype == BNS_F32 ? 4 : 2, pitch = size_t(d.C) * size, M = size_t(d.N) * size_t(d.HW);
    if (opt == 2 || column_vec(d) * size != 16 || pitch * size_t(kBlock * kSplitRows) >= (size_t(1) << 30)) return false;
    if (opt == 1) return true;
    const RowSet S = make_rowset(d, b);
    const Tiling t = make_tiling(d, uint32_t(M));
    const size_t tiles = size_t((t.CV + (1 << t.log2_tx) - 1) >> t.log2_tx), lanes = tiles << t.log2_tx;
    if (4 * size_t(S.rows) > M || 8 * size_t(t.CV) < 7 * lanes || M * pitch < size_t(16) << 20) return false;
    if (pitch % 64) return tiles <= 2 && S.contiguous;
    return tiles <= 2 || tiles == 4 || tiles == 8 || (tiles <= 6 && d.dtype == BNS_F32 && S.contiguous && 100 * size_t(t.CV) >= 97 * lanes);
}

// The whole backward pass with dx split by Eq. 6's two branches: sums + dx outside S, finalize, dx on S.
hipError_t launch_nhwc_backward_split(const Dims& d, const bns_box& b, const void* x, const void* dy, const float* gamma,
                                      const float* mean, const float* invstd, Partial* partial, float* dgamma,
                                      float* dbeta, void* dx, bool ordered, hipStream_t st) {
    const uint32_t M = uint32_t(d.N) * uint32_t(d.HW);
    const Tiling t = make_tiling(d, M);      // the tiling of launch_nhwc_reduce: same partials, same sums, bit for bit (not `ordered`)
    if (!fits_region(d, t)) return hipErrorInvalidValue;
    const RowBox B = make_rowbox(d, b);
    const RowSet S = make_rowset(d, b);
    const Tiling ts = make_tiling(d, S.rows, 0, true);
    const uint32_t s_lo = (uint32_t(b.n0) * uint32_t(d.H) + uint32_t(b.h0)) * uint32_t(d.W) + uint32_t(b.w0);
    const double s = double(b.n_cnt) * double(b.h_cnt) * double(b.w_cnt);
    return dispatch_nhwc(d, [&](auto ty, auto vt) {
        using T = decltype(ty);
        constexpr int V = decltype(vt)::value;
        const T* xp = static_cast<const T*>(x);
        const T* gp = static_cast<const T*>(dy);
        T* op = static_cast<T*>(dx);
        const dim3 grid(grid_of(t)), block(kBlock);
        if constexpr (V * sizeof(T) == 16) {
            if (ordered) {
                // (a walk of its own for the rows of S costs a drained pipeline: a single sample of 128, 196 chunks for 512 blocks, 218 us
                // against 214; sixteen, six chunks per block, 223 against 232.  Not the "cache_reuse" option: the order of the sums depends on it)
                const uint32_t held = S.rows / (uint32_t(kSplitRows) * uint32_t(kBlock >> t.log2_tx));
                const bool keep = 2 * size_t(S.rows) * size_t(d.C) * sizeof(T) <= kKeepBytes && held >= 2u * uint32_t(t.splits);
                auto kernel = !S.contiguous ? &nhwc_reduce_outside_ordered_kernel<T, V, false, false>
                              : keep        ? &nhwc_reduce_outside_ordered_kernel<T, V, true, true>
                                            : &nhwc_reduce_outside_ordered_kernel<T, V, true, false>;
                BNS_LAUNCH((*kernel), grid, block, 0, st, xp, gp, mean, partial, t, M, op, gamma, invstd, B, s_lo, S.rows);
            }
        }
        if (!ordered)
            BNS_LAUNCH((nhwc_reduce_outside_kernel<T, V>), grid, block, 0, st, xp, gp, mean, partial, t, M, op, gamma, invstd, B);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        BNS_LAUNCH(nhwc_reduce_finalize_kernel, dim3(ceil_div_u(uint32_t(d.C), kFinCh)), dim3(kBlock), 0, st,
                   partial, d.C, t.splits, invstd, dgamma, dbeta);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (S.contiguous)
            BNS_LAUNCH((nhwc_dx_rows_kernel<T, V, true>), dim3(grid_of(ts)), dim3(kBlock), 0, st, static_cast<const T*>(x),
                       static_cast<const T*>(dy), static_cast<T*>(dx), gamma, mean, invstd, dgamma, dbeta, S, ts,
                       float(1.0 / s));
        else
            BNS_LAUNCH((nhwc_dx_rows_kernel<T, V, false>), dim3(grid_of(ts)), dim3(kBlock), 0, st, static_cast<const T*>(x),
                       static_cast<const T*>(dy), static_cast<T*>(dx), gamma, mean, invstd, dgamma, dbeta, S, ts,
                       float(1.0 / s));
        return hipGetLastError();
    });
}

hipError_t launch_nhwc_dx(const Dims& d, const bns_box& b, const void* x, const void* dy, const float* gamma,
                          const float* mean, const float* invstd, const float* dgamma, const float* dbeta, void* dx,
                          hipStream_t st) {
    const uint32_t M = uint32_t(d.N) * uint32_t(d.HW);
    const Tiling t = make_tiling(d, M, 0, true);
    const RowBox B = make_rowbox(d, b);
    const double s = double(b.n_cnt) * double(b.h_cnt) * double(b.w_cnt);
    return dispatch_nhwc(d, [&](auto ty, auto vt) {
        using T = decltype(ty);
        constexpr int V = decltype(vt)::value;
        BNS_LAUNCH((nhwc_dx_kernel<T, V>), dim3(grid_of(t)), dim3(kBlock), 0, st, static_cast<const T*>(x),
                   static_cast<const T*>(dy), static_cast<T*>(dx), gamma, mean, invstd, dgamma, dbeta, B, t, M,
                   float(1.0 / s));
        return hipGetLastError();
    });
}

// Eq. 4 forward statistics: `partial` holds two regions of nhwc_partial_bytes(d) each (set S, then set V).
hipError_t launch_nhwc_stats_mixed(const Dims& d, const bns_box& b, int n_v, const void* x, Partial* partial,
                                   float mix_beta, float eps, float momentum, float* save_mean, float* save_invstd,
                                   float* mean_parts, float* running_mean, float* running_var, hipStream_t st) {
    const RowSet S = make_rowset(d, b);
    const bns_box vb{0, n_v, 0, d.H, 0, d.W};
    const RowSet Vs = make_rowset(d, vb);
    const Tiling ts = make_tiling(d, S.rows), tv = make_tiling(d, Vs.rows);
    if (!fits_region(d, ts) || !fits_region(d, tv)) return hipErrorInvalidValue;
    Partial* partial_v = reinterpret_cast<Partial*>(reinterpret_cast<char*>(partial) + nhwc_partial_bytes(d));
    return dispatch_nhwc(d, [&](auto ty, auto vt) {
        using T = decltype(ty);
        constexpr int V = decltype(vt)::value;
        hipError_t e = launch_stats_partial<T, V>(static_cast<const T*>(x), partial, S, ts, st);
        if (e != hipSuccess) return e;
        if ((e = launch_stats_partial<T, V>(static_cast<const T*>(x), partial_v, Vs, tv, st)) != hipSuccess) return e;
        BNS_LAUNCH((nhwc_stats_finalize_mixed_kernel<T>), dim3(ceil_div_u(uint32_t(d.C), kFinCh)), dim3(kBlock), 0,
                   st, static_cast<const T*>(x), partial, ts.splits, partial_v, tv.splits, S, Vs, d.C, mix_beta, eps,
                   momentum, save_mean, save_invstd, mean_parts, running_mean, running_var);
        return hipGetLastError();
    });
}

hipError_t launch_nhwc_dx_mixed(const Dims& d, const bns_box& b, int n_v, float mix_beta, const void* x, const void* dy,
                                const float* gamma, const float* invstd, const float* dgamma, const float* dbeta,
                                const float* mean_parts, void* dx, hipStream_t st) {
    const uint32_t M = uint32_t(d.N) * uint32_t(d.HW);
    const Tiling t = make_tiling(d, M, 0, true);
    const RowBox B = make_rowbox(d, b);
    const float w_s = float((1.0 - double(mix_beta)) / (double(b.n_cnt) * double(b.h_cnt) * double(b.w_cnt)));
    const float w_v = float(double(mix_beta) / (double(n_v) * double(d.HW)));
    return dispatch_nhwc(d, [&](auto ty, auto vt) {
        using T = decltype(ty);
        constexpr int V = decltype(vt)::value;
        BNS_LAUNCH((nhwc_dx_mixed_kernel<T, V>), dim3(grid_of(t)), dim3(kBlock), 0, st, static_cast<const T*>(x),
                   static_cast<const T*>(dy), static_cast<T*>(dx), gamma, invstd, dgamma, dbeta, mean_parts,
                   mean_parts + d.C, B, uint32_t(n_v) * uint32_t(d.HW), w_v, w_s, t, M);
        return hipGetLastError();
    });
}

}  // namespace bns
