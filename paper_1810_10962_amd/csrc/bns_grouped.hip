// Single-launch kernels for N x C x H x W tensors with small planes: a block owns a GROUP of adjacent channels.
//
// The planes of G adjacent channels of one sample are one contiguous run of G * HW elements, so the tensor is a matrix
// of N rows (samples) by C * HW columns, and a block takes the columns of its G channels and every row.  A thread holds
// a fixed vector of columns and walks down the rows: it works out once, for the whole launch, which channels its V
// elements belong to (at most two, since HW >= V), which of them lie in the patch and which statistics they need;
// the loop over the rows has no division and no membership test but "is this sample in S".  The channel stays in
// registers between its sums and its element-wise pass (forward: x, 2e bytes per element; backward: dy and x, 3e), and
// nothing crosses blocks, so there is nothing to wait for.
//
// What it is for: the kernels of bns_fused.hip address one plane at a time.  With planes of 49 elements that means
// accesses of one element per lane (49 is no multiple of a vector, so planes start anywhere) and 98 or 196 bytes
// per plane that share their cache lines with the neighbours' planes.  A group's run is vector accesses from end to end:
// G is chosen so that it is a whole number of vectors where possible; where it is not, accesses are element-aligned (the
// memory system takes 128-bit accesses at any element) and the last vector of a run is moved back so that it ends with
// the run (the elements it shares with the vector before it are left out of the sums and stored twice with the same bits).
//
// Bound by memory: one read of each input, one write of the output, and by what a launch of one round costs (load, two
// block barriers, store).  64x2048x7x7, Batch Sampling, us forward / backward: bf16 8.7 / 10.4 (2.9 / 3.7 TB/s; with shuffles and divisions 9.95 / 11.4) against
// 14.3 / 22.3 with the other kernels, f32 12.3 / 15.7 (4.2 / 4.9 TB/s) against 22.3 / 33.0.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "bns_device.hpp"
#include "bns_fused_device.hpp"
#include "bns_internal.hpp"

namespace bns {

namespace {

constexpr int kGroupMaxChannels = 64;

struct GroupArgs {
    const void* x;
    const void* dy;
    void* out;
    const float* gamma;
    const float* beta;
    float* save_mean;
    float* save_invstd;
    float* running_mean;
    float* running_var;
    float* dgamma;
    float* dbeta;
    float* mean_parts;      // Eq. 4: [E_v per channel][E_s per channel]
    IndexParams ip;
    FastDiv tx_div, hw_div, w_div;
    int32_t N, C, HW, W, G;
    int32_t whole;          // S takes whole planes
    int32_t TY;             // rows taken at a time: threads / column vectors of a group
    int32_t n_v;            // Eq. 4: samples of the virtual set
    float mix_beta, w_s, w_v, eps, momentum;
    double inv_s64, inv_s_v;    // 1 / points of S, of the virtual set
};

// 128-bit (64-bit) accesses at element alignment: planes of an odd number of elements start anywhere.
template <typename T, int V>
struct ElemVec : RawVec<T, V> {
    typedef typename RawVec<T, V>::raw_t raw_t;
    typedef raw_t unaligned_t __attribute__((aligned(sizeof(T))));
    static __device__ __forceinline__ raw_t ld(const T* p) {
        return __builtin_nontemporal_load(reinterpret_cast<const unaligned_t*>(p));
    }
    static __device__ __forceinline__ void st(T* p, raw_t r) {
        __builtin_nontemporal_store(r, reinterpret_cast<unaligned_t*>(p));
    }
};

// What a thread knows about its columns.
template <int V>
struct Columns {
    int tx, ty;
    int c0, channels;       // the block's channels
    uint32_t col;           // first column, within the group's run
    int ch0;                // channel of the first column, within the group
    int bnd;                // elements e < bnd belong to ch0, the others to ch0 + 1
    uint32_t own;           // elements that no other thread holds (bit e)
    uint32_t in;            // elements inside the rows and columns of their channel's patch
    bool live;

    __device__ __forceinline__ Columns(const GroupArgs& A) {
        const uint32_t t = threadIdx.x;
        ty = int(fdiv(t, A.tx_div));
        tx = int(t) - ty * int(A.tx_div.d);
        c0 = int(blockIdx.x) * A.G;
        channels = min(A.G, A.C - c0);
        const uint32_t run = uint32_t(channels) * uint32_t(A.HW);
        live = ty < A.TY && uint32_t(tx) * V < run;             // (the last group may be narrower)
        const uint32_t first = live ? uint32_t(tx) * V : 0u;
        col = min(first, run - V);
        ch0 = int(fdiv(col, A.hw_div));
        bnd = int(uint32_t(ch0 + 1) * uint32_t(A.HW) - col);
        own = (~0u << (first - col)) & ((1u << V) - 1u);
        in = ~0u;
        if (A.whole) return;
        in = 0u;
        bns_box b = box_of_channel(A.ip, c0 + ch0);
        uint32_t pos = col - uint32_t(ch0) * uint32_t(A.HW);
        uint32_t h = fdiv(pos, A.w_div), w = pos - h * uint32_t(A.W);
#pragma unroll
        for (int e = 0; e < V; ++e) {
            if (e == bnd) {
                b = box_of_channel(A.ip, c0 + ch0 + 1);
                h = w = 0u;
            }
            in |= uint32_t(in_hw(b, h, w)) << e;
            if (++w == uint32_t(A.W)) {
                w = 0u;
                ++h;
            }
        }
    }
};

// A thread's way down its rows: the byte offset of the next one from the group's first element (one addition per row; worked out by
// multiplication, and together with the divisions that whole planes do not need, 64x2048x7x7 bf16 lost 0.7 us of 9.7 to it).
struct RowsDown {
    int n;
    size_t off;
    template <typename T>
    static __device__ __forceinline__ RowsDown from(int row, size_t nstride, uint32_t col) {
        return RowsDown{row, (size_t(uint32_t(row)) * nstride + col) * sizeof(T)};
    }
    __device__ __forceinline__ void next(int rows, size_t bytes) {
        n += rows;
        off += bytes;
    }
};
template <typename T>
__device__ __forceinline__ T* down(T* base, size_t off) {
    typedef typename std::conditional<std::is_const<T>::value, const char, char>::type byte_t;
    return reinterpret_cast<T*>(reinterpret_cast<byte_t*>(base) + off);
}

// Per-thread sums of V columns -> one (ch0, ch0 + 1) pair of sums per thread in LDS.  `mask`: the elements that count.
template <int V, int NT>
__device__ __forceinline__ void columns_to_lds(const float (&a)[V], const float (&q)[V], uint32_t mask, int bnd, float4* part) {
    float4 p = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < V; ++e) {
        const bool counts = (mask >> e) & 1u;                   // (a select: a masked NaN must not reach the sum)
        p.x += counts && e < bnd ? a[e] : 0.f;
        p.y += counts && e < bnd ? q[e] : 0.f;
        p.z += counts && e >= bnd ? a[e] : 0.f;
        p.w += counts && e >= bnd ? q[e] : 0.f;
    }
    part[threadIdx.x] = p;
}

// Lane l of wave w finishes channel w + l * (waves of the block): channel_of is that channel, channel_totals leaves its
// two sums there.
template <int NT>
__device__ __forceinline__ int channel_of() {
    return int(threadIdx.x / kWave) + int(threadIdx.x % kWave) * (NT / kWave);
}

template <int V, int NT>
__device__ __forceinline__ void channel_totals(const GroupArgs& A, int channels, const float4* part, double& t1, double& t2) {
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    const uint32_t HW = uint32_t(A.HW), run = uint32_t(channels) * HW;
    t1 = t2 = 0.0;
    int turn = 0;
    for (int g = wave; g < channels; g += NT / kWave, ++turn) {
        const uint32_t lo = uint32_t(g) * HW / V, hi = (uint32_t(g + 1) * HW - 1u) / V;    // column vectors that hold it
        const uint32_t cnt = hi - lo + 1u, total = cnt * uint32_t(A.TY);                  // (at most two blocks' worth of threads)
        const float per = __builtin_amdgcn_rcpf(float(cnt));                              // (i + 0.5 stays clear of whole rows)
        const uint32_t starts = uint32_t(g) * HW;
        double s1 = 0.0, s2 = 0.0;
        for (uint32_t i = uint32_t(lane); i < total; i += kWave) {
            const uint32_t row = uint32_t((float(i) + 0.5f) * per), tx = lo + (i - row * cnt);
            const float4 p = part[row * A.tx_div.d + tx];
            const bool first = min(tx * V, run - V) >= starts;      // the vector's first column is of this channel
            s1 += double(first ? p.x : p.z);
            s2 += double(first ? p.y : p.w);
        }
        s1 = wave_sum(s1);
        s2 = wave_sum(s2);
        if (lane == turn) {
            t1 = s1;
            t2 = s2;
        }
    }
}

// Waves per SIMD that the registers have to allow: 128 of them hold up to 16 vectors and what the elements need (8 in the forward pass of
// Eq. 4), so that a compute unit takes two blocks of 512 threads.
constexpr int group_waves(int vectors, bool mixed_forward) { return vectors > (mixed_forward ? 8 : 16) ? 2 : 4; }

template <typename T, int V, int K, int NT, bool MIXED>
__global__ __launch_bounds__(NT, group_waves(K, MIXED)) void grouped_forward_kernel(GroupArgs A) {
    touch_arguments<GroupArgs>();
    typedef ElemVec<T, V> EV;
    __shared__ float4 part[(MIXED ? 2 : 1) * NT];
    __shared__ float4 consts[kGroupMaxChannels];
    const Columns<V> me(A);
    const int t = channel_of<NT>();
    const size_t nstride = size_t(A.C) * A.HW;
    const T* xg = static_cast<const T*>(A.x) + size_t(me.c0) * A.HW;
    T* yg = static_cast<T*>(A.out) + size_t(me.c0) * A.HW;

    // The pivots (first sampled element of a channel) of the thread's channels, and what the thread that finishes
    // channel t needs, are requested ahead of the vectors.
    const int n0 = A.ip.shared.n0, n1 = n0 + A.ip.shared.n_cnt;
    const int next = min(me.ch0 + 1, me.channels - 1);
    auto pivot_of = [&](int g) {
        const bns_box b = box_of_channel(A.ip, me.c0 + g);
        return load_scalar<T>(xg + size_t(b.n0) * nstride + size_t(g) * A.HW + size_t(b.h0) * A.W + b.w0);
    };
    const float p0 = pivot_of(me.ch0), p1 = pivot_of(next);
    const float v0 = MIXED ? load_scalar<T>(xg + size_t(me.ch0) * A.HW) : 0.f;
    const float v1 = MIXED ? load_scalar<T>(xg + size_t(next) * A.HW) : 0.f;
    float pivot = 0.f, pivot_v = 0.f, ga = 0.f, be = 0.f, rm = 0.f, rv = 0.f;
    const bool leads = t < me.channels;
    if (leads) {
        const int c = me.c0 + t;
        pivot = pivot_of(t);
        if (MIXED) pivot_v = load_scalar<T>(xg + size_t(t) * A.HW);
        ga = A.gamma[c];
        be = A.beta[c];
        if (A.running_mean) rm = A.running_mean[c];
        if (A.running_var) rv = A.running_var[c];
    }
    typename EV::raw_t v[K];
    // (each phase works its addresses out anew: see opaque)
    const size_t hop = size_t(A.TY) * nstride * sizeof(T), last = (size_t(A.N - 1) * nstride + me.col) * sizeof(T);
    RowsDown at = RowsDown::from<T>(int(opaque(uint32_t(me.ty))), nstride, me.col);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (k * A.TY < A.N) v[k] = EV::ld(down(xg, at.n < A.N ? at.off : last));
        at.next(A.TY, hop);
    }
    float a[V], q[V], av[MIXED ? V : 1], qv[MIXED ? V : 1];
#pragma unroll
    for (int e = 0; e < V; ++e) a[e] = q[e] = 0.f;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int n = k * A.TY + me.ty;
        if (k * A.TY < n1 && n >= n0 && n < n1) {
            float f[V];
            EV::unpack(v[k], f);
#pragma unroll
            for (int e = 0; e < V; ++e) {
                const float d = f[e] - (e < me.bnd ? p0 : p1);
                a[e] += d;
                q[e] = fmaf(d, d, q[e]);
            }
        }
    }
    columns_to_lds<V, NT>(a, q, me.live ? me.own & me.in : 0u, me.bnd, part);
    if constexpr (MIXED) {                                      // the virtual set: every column of samples [0, n_v)
#pragma unroll
        for (int e = 0; e < V; ++e) av[e] = qv[e] = 0.f;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (k * A.TY < A.n_v && k * A.TY + me.ty < A.n_v) {
                float f[V];
                EV::unpack(v[k], f);
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const float d = f[e] - (e < me.bnd ? v0 : v1);
                    av[e] += d;
                    qv[e] = fmaf(d, d, qv[e]);
                }
            }
        }
        columns_to_lds<V, NT>(av, qv, me.live ? me.own : 0u, me.bnd, part + NT);
    }
    __syncthreads();
    double s1, s2, u1 = 0.0, u2 = 0.0;
    channel_totals<V, NT>(A, me.channels, part, s1, s2);
    if constexpr (MIXED) channel_totals<V, NT>(A, me.channels, part + NT, u1, u2);
    if (leads) {                                                // Eq. 3, Eq. 4, Eq. 8: one thread per channel
        const int c = me.c0 + t;
        const double m1 = s1 * A.inv_s64;
        double mean = double(pivot) + m1;
        double var = s2 * A.inv_s64 - m1 * m1;
        if (!(var >= 0.0)) var = (var != var) ? var : 0.0;      // clamp rounding; keep NaN visible
        if constexpr (MIXED) {
            const double mv = u1 * A.inv_s_v;
            const double e_v = double(pivot_v) + mv;
            double var_v = u2 * A.inv_s_v - mv * mv;
            if (!(var_v >= 0.0)) var_v = (var_v != var_v) ? var_v : 0.0;
            A.mean_parts[c] = float(e_v);
            A.mean_parts[A.C + c] = float(mean);
            const double bm = double(A.mix_beta);
            mean = bm * e_v + (1.0 - bm) * mean;
            var = bm * var_v + (1.0 - bm) * var;
        }
        const float mu = float(mean);
        const float r = float(inv_sqrt(var + double(A.eps)));
        A.save_mean[c] = mu;
        A.save_invstd[c] = r;
        const double al = double(A.momentum);
        if (A.running_mean) A.running_mean[c] = float((1.0 - al) * double(rm) + al * mean);
        if (A.running_var) A.running_var[c] = float((1.0 - al) * double(rv) + al * var);
        consts[t] = float4{mu, ga * r, be, 0.f};
    }
    __syncthreads();
    if (!me.live) return;
    const float4 k0 = consts[me.ch0], k1 = consts[next];
    float mu[V], sc[V], sh[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
        mu[e] = e < me.bnd ? k0.x : k1.x;
        sc[e] = e < me.bnd ? k0.y : k1.y;
        sh[e] = e < me.bnd ? k0.z : k1.z;
    }
    at = RowsDown::from<T>(int(opaque(uint32_t(me.ty))), nstride, me.col);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (at.n < A.N) {
            float f[V];
            opaque_raw(v[k]);
            EV::unpack(v[k], f);
#pragma unroll
            for (int e = 0; e < V; ++e) f[e] = fmaf(f[e] - mu[e], sc[e], sh[e]);
            EV::st(down(yg, at.off), EV::pack(f));
        }
        at.next(A.TY, hop);
    }
}

template <typename T, int V, int K, int NT, bool MIXED>
__global__ __launch_bounds__(NT, group_waves(2 * K, false)) void grouped_backward_kernel(GroupArgs A) {
    touch_arguments<GroupArgs>();
    typedef ElemVec<T, V> EV;
    __shared__ float4 part[NT];
    __shared__ float4 consts[(MIXED ? 2 : 1) * kGroupMaxChannels];
    const Columns<V> me(A);
    const int t = channel_of<NT>();
    const size_t nstride = size_t(A.C) * A.HW;
    const T* xg = static_cast<const T*>(A.x) + size_t(me.c0) * A.HW;
    const T* gg = static_cast<const T*>(A.dy) + size_t(me.c0) * A.HW;
    T* dg = static_cast<T*>(A.out) + size_t(me.c0) * A.HW;

    const int next = min(me.ch0 + 1, me.channels - 1);
    const float m0 = A.save_mean[me.c0 + me.ch0], m1 = A.save_mean[me.c0 + next];
    float mean = 0.f, r = 0.f, ga = 0.f, e_v = 0.f, e_s = 0.f;
    const bool leads = t < me.channels;
    const int n0 = A.ip.shared.n0, n1 = n0 + A.ip.shared.n_cnt;
    if (leads) {
        const int c = me.c0 + t;
        mean = A.save_mean[c];
        r = A.save_invstd[c];
        ga = A.gamma[c];
        if (MIXED) {
            e_v = A.mean_parts[c];
            e_s = A.mean_parts[A.C + c];
        }
    }
    typename EV::raw_t g[K], x[K];
    const size_t hop = size_t(A.TY) * nstride * sizeof(T), last = (size_t(A.N - 1) * nstride + me.col) * sizeof(T);
    RowsDown at = RowsDown::from<T>(int(opaque(uint32_t(me.ty))), nstride, me.col);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (k * A.TY < A.N) {
            const size_t off = at.n < A.N ? at.off : last;
            g[k] = EV::ld(down(gg, off));
            x[k] = EV::ld(down(xg, off));
        }
        at.next(A.TY, hop);
    }
    float a[V], q[V];
#pragma unroll
    for (int e = 0; e < V; ++e) a[e] = q[e] = 0.f;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (k * A.TY < A.N && k * A.TY + me.ty < A.N) {
            float fg[V], fx[V];
            EV::unpack(g[k], fg);
            EV::unpack(x[k], fx);
#pragma unroll
            for (int e = 0; e < V; ++e) {
                a[e] += fg[e];
                q[e] = fmaf(fg[e], fx[e] - (e < me.bnd ? m0 : m1), q[e]);
            }
        }
    }
    columns_to_lds<V, NT>(a, q, me.live ? me.own : 0u, me.bnd, part);
    __syncthreads();
    double t1, t2;
    channel_totals<V, NT>(A, me.channels, part, t1, t2);
    if (leads) {                                                // Eq. 5; the constants of Eq. 6
        const int c = me.c0 + t;
        const float dbeta = float(t1);
        const float dgamma = float(t2 * double(r));
        A.dbeta[c] = dbeta;
        A.dgamma[c] = dgamma;
        const float ar = ga * r;
        consts[t] = float4{ar, ar * A.w_s * dbeta, ar * A.w_s * dgamma * r, MIXED ? e_s : mean};
        if (MIXED) consts[kGroupMaxChannels + t] = float4{0.f, ar * A.w_v * dbeta, ar * A.w_v * dgamma * r, e_v};
    }
    __syncthreads();
    if (!me.live) return;
    const float4 s0 = consts[me.ch0], s1 = consts[next];
    at = RowsDown::from<T>(int(opaque(uint32_t(me.ty))), nstride, me.col);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int n = at.n;
        if (n < A.N) {
            float f[V];
            opaque_raw(g[k]);
            EV::unpack(g[k], f);
            if (MIXED && n < A.n_v) {
                const float4 w0 = consts[kGroupMaxChannels + me.ch0], w1 = consts[kGroupMaxChannels + next];
                float fx[V];
                opaque_raw(x[k]);
                EV::unpack(x[k], fx);
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const bool lo = e < me.bnd;
                    f[e] = fmaf(lo ? s0.x : s1.x, f[e],
                                -fmaf(lo ? w0.z : w1.z, fx[e] - (lo ? w0.w : w1.w), lo ? w0.y : w1.y));
                }
            } else if (n >= n0 && n < n1) {
                float fx[V];
                opaque_raw(x[k]);
                EV::unpack(x[k], fx);
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const bool lo = e < me.bnd;
                    const float corr = fmaf(lo ? s0.z : s1.z, fx[e] - (lo ? s0.w : s1.w), lo ? s0.y : s1.y);
                    f[e] = fmaf(lo ? s0.x : s1.x, f[e], (me.in >> e) & 1u ? -corr : 0.f);
                }
            } else {
#pragma unroll
                for (int e = 0; e < V; ++e) f[e] *= e < me.bnd ? s0.x : s1.x;
            }
            EV::st(down(dg, at.off), EV::pack(f));
        }
        at.next(A.TY, hop);
    }
}

// (threads per block, vectors per thread and tensor)
struct GroupVariant {
    int nt, k;
};
constexpr GroupVariant kGroupVariants[] = {{256, 4}, {256, 8}, {512, 8}, {512, 16}};
constexpr int kNumGroupVariants = sizeof(kGroupVariants) / sizeof(kGroupVariants[0]);

template <typename T, int V, int K, int NT>
void launch_variant(bool backward, bool mixed, const GroupArgs& A, dim3 grid, hipStream_t st) {
    const dim3 block(NT);
    if (backward) {
        if (mixed) BNS_LAUNCH((grouped_backward_kernel<T, V, K, NT, true>), grid, block, 0, st, A);
        else BNS_LAUNCH((grouped_backward_kernel<T, V, K, NT, false>), grid, block, 0, st, A);
    } else {
        if (mixed) BNS_LAUNCH((grouped_forward_kernel<T, V, K, NT, true>), grid, block, 0, st, A);
        else BNS_LAUNCH((grouped_forward_kernel<T, V, K, NT, false>), grid, block, 0, st, A);
    }
}

template <typename T, int V>
void launch_any(int variant, bool backward, bool mixed, const GroupArgs& A, dim3 grid, hipStream_t st) {
    switch (variant) {
        case 0: return launch_variant<T, V, 4, 256>(backward, mixed, A, grid, st);
        case 1: return launch_variant<T, V, 8, 256>(backward, mixed, A, grid, st);
        case 2: return launch_variant<T, V, 8, 512>(backward, mixed, A, grid, st);
        default: return launch_variant<T, V, 16, 512>(backward, mixed, A, grid, st);
    }
}

}  // namespace

hipError_t launch_grouped(const Dims& d, const IndexParams& ip, bool backward, const FusedIo& io, float eps, float momentum,
                          hipStream_t st, int cus, const FusedMix* mix) {
    const int V = d.dtype == BNS_F32 ? 4 : 8;
    const int opt = g_tuning.grouped, opt_g = g_tuning.grouped_channels;
    if (d.HW < V || opt == 2 || cus <= 0) return hipErrorNotSupported;
    // Channels per group: about one block per compute unit, also where two fit (64x2048x7x7 bf16, forward / backward: groups of 8, 256 blocks,
    // 8.3 / 10.0 us; of 4, 9.3 / 10.5; of 2, 10.3 / 15.1; of 16, 9.6 / 12.9; 64x512x7x7: of 2, 256 blocks, 5.5 / 6.0; of 1, 6.4 / 6.6; of 8, 6.8 / 8.0), whole vectors per run
    // (multiples of `unit` channels) if that leaves as many blocks, fewer when the rows of a group would not fit the
    // largest block.  Block: the smallest that holds the group.
    const int unit = d.HW % V == 0 ? 1 : d.HW % (V / 2) == 0 ? 2 : (V == 8 && d.HW % 2 == 0) ? 4 : V;
    const int64_t room = int64_t(kGroupVariants[kNumGroupVariants - 1].nt) * kGroupVariants[kNumGroupVariants - 1].k;
    int64_t G = opt_g > 0 ? opt_g : (d.C + cus - 1) / cus;
    G = std::min<int64_t>({G, room * V / (int64_t(d.HW) * d.N), kGroupMaxChannels, d.C});
    int best_v = -1;
    for (; G >= 1 && best_v < 0; --G) {
        if (G > unit && G % unit != 0 && opt_g <= 0) continue;
        const int64_t lanes = (G * d.HW + V - 1) / V;
        for (int v = 0; v < kNumGroupVariants && best_v < 0; ++v) {
            const GroupVariant gv = kGroupVariants[v];
            if (lanes <= gv.nt && int64_t(gv.nt / lanes) * gv.k >= d.N && (opt < 3 || v == opt - 3)) best_v = v;
        }
        if (best_v >= 0) break;
    }
    if (best_v < 0) return hipErrorNotSupported;
    const int best_g = int(G);
    // A run of more than half a block's threads leaves the others without work (3x700x33x33 f32: 273 of 512 threads, forward
    // 11.4 us against 8.6 with one element per access).  With three and more channels in a run the other kernels have more blocks than
    // the device holds at once, and this is the faster side backward up to 16 MB (1.2 in the mean of 62 drawn layers, 4x852x17x17 f32 5.8
    // against 21.6) and forward where planes are whole vectors (asked when those take several rounds or have very many blocks: 1.5 in the mean of 23,
    // 10x832x28x28 f32 11.0 against 20.1).  Eq. 4: 1.11 forward, 11 layers, 1.24 backward, 14.
    const int64_t bytes = int64_t(d.N) * d.C * d.HW * (V == 8 ? 2 : 4);
    const bool crowded = G >= 3 && (backward ? bytes < 16000000 : d.vec > 1);
    if (opt == 0 && (G * d.HW + V - 1) / V > 256 && !crowded) return hipErrorNotSupported;
    // Forward, planes that are no whole vectors: a group of fewer than 1536 vectors leaves most of its 512 threads one row or none, and the
    // kernels of bns_fused.hip, a small block per channel, take 1 / 1.13 (140 layers) and 1 / 1.21 (84) of the time: 62x200x7x7 f32 5.3 against 4.4.
    // (A patch costs those more: 12x1349x11x9 f32, 1188 vectors, 8.6 against 11.0.  Eq. 4, other / grouped: up to 1024 vectors 0.76 to 0.95 by size, 177 layers, none
    // above 1; 1024 to 1536 0.92, 21 layers; beyond 1.14, 45.)
    const bool patch = ip.shared.h_cnt != d.H || ip.shared.w_cnt != d.W;
    // (In more than four channels to a compute unit those no longer fit at once: 26x1632x7x7 f32, 1274 vectors, 7.5 against 8.9.)
    if (opt == 0 && !backward && d.vec == 1 && d.C <= 4 * cus && int64_t(d.N) * ((G * d.HW + V - 1) / V) < (patch && !mix ? 1024 : 1536)) return hipErrorNotSupported;
    // Backward: a channel of up to 64 vectors fits one wave of its own (1.18 and 1.26 times as fast, 53 and 48 layers, none slower: 2x528x10x10
    // bf16 5.2 against 3.6; beyond 1.2 MB it is, 12x1952x7x5 bf16 6.2 against 8.5), one of more than 1024 fills a block of 512 threads, which pays
    // in small tensors (1.05 and 1.10, 68 and 46 layers).  Eq. 4: up to 64 vectors 0.86 to 0.92, 92 layers; more than 1024 up to these sizes 0.95, 25; beyond them and
    // between 1.04 to 1.47, by size.
    const int64_t vectors = int64_t(d.N) * ((d.HW + V - 1) / V);
    if (opt == 0 && backward && ((vectors <= 64 && bytes <= 1200000) || (vectors > 1024 && bytes <= (d.vec > 1 ? 4000000 : 1800000))))
        return hipErrorNotSupported;
    // Few channels would fill only part of the device with large blocks; the kernels of bns_fused.hip share a channel (backward, us:
    // 128x64x16x16 f32 11.2 against 11.6, 100x60x12x12 bf16 8.5 against 8.9, 102x64x23x23 bf16 11.0 against 19.3).
    const int blocks = (d.C + best_g - 1) / best_g;
    if (opt == 0 && blocks < cus / 2 && best_v >= 2) return hipErrorNotSupported;
    // More blocks than compute units, planes of whole vectors.  Two of these blocks share a unit (one, backward or Eq. 4 with 16 vectors per thread: tall).
    // The other kernels' time over this one's, layers drawn and timed both ways, geometric means f32 / bf16 (layers below 0.97):
    //   forward, tall, 257 to 512 blocks 1.40 (3 of 78) / 1.58 (2 of 75); 513 to 1024 1.09 (14 of 71) / 1.12 (11 of 76), a patch 1.19 (1 of 20) / 1.55 (none of
    //   24); beyond, 0.94 / 1.05.  (99x560x16x16 bf16, all points, 280 blocks, 13.0 against 15.2 us; 91x1552x20x19 bf16, 776 blocks, 49.3 against 63.4.)
    //   Eq. 4 forward, 257 to 512 blocks 1.43 / 1.10 (6), beyond 1.11 / 0.91.
    //   backward, whole full-width vectors that begin on cache lines (fp32) or any (bf16), where the pipelined kernel is the other: tall, 257 to 384 1.10 / 0.96,
    //   385 to 512 1.16 / 1.15 (none below), beyond 0.98 / 0.94 (128x1024x16x16 39.1 against 42.5 us in bf16, 74.3 against 80.0); not tall, 513 to
    //   1024 1.11 / 1.08, beyond 1.01 / 0.97.
    //   backward, others, tall: 257 to 320 1.03 / 0.99 (61x288x28x28 bf16 40.8 against 41.7), 321 to 512 1.20 / 1.24, 513 to 640 1.00 / 1.06, then 1.07 / 1.08.
    const bool tall = best_v == 3, lines = d.vec == V && !mix && (V == 8 || d.HW * 4 % 128 == 0);
    if (opt == 0 && d.vec > 1 && best_v >= 2 && blocks > cus) {
        const bool part = blocks % cus != 0 && blocks % cus < cus / 2;         // a last round of one block per unit leaves most of them idle
        const bool other = !backward ? (mix ? V == 8 && (blocks > 2 * cus || part) : blocks > (patch ? 4 : 2) * cus)
                           : lines   ? (tall ? blocks > 2 * cus || (V == 8 && 2 * blocks < 3 * cus) : blocks > 4 * cus)
                                     : tall && (4 * blocks < 5 * cus || (blocks > 2 * cus && part));
        if (other) return hipErrorNotSupported;
    }
    // Calls that take 5 us whatever they do: working out the columns costs more there than it saves (forward, us: 8x224x5x5 f32
    // 4.8 against 5.4, 37x96x9x9 bf16 5.7 against 6.3; backward, 6x144x7x7 bf16 5.0 against 5.4).  Just above the lines the median gain is
    // nil: forward, 1.0 to 1.3 MB, 1.00 (30 tensors), backward, bf16, 0.3 to 0.5 MB, 1.06 (66); fp32 below 0.1 MB 1.03 (54).
    if (opt == 0 && bytes < (backward ? (V == 8 ? 300000 : 0) : 1000000) && !mix) return hipErrorNotSupported;
    const GroupVariant gv = kGroupVariants[best_v];
    const uint32_t lanes = uint32_t((long(best_g) * d.HW + V - 1) / V);
    GroupArgs A;
    A.x = io.x;
    A.dy = io.dy;
    A.out = io.out;
    A.gamma = io.gamma;
    A.beta = io.beta;
    A.save_mean = io.save_mean;
    A.save_invstd = io.save_invstd;
    A.running_mean = io.running_mean;
    A.running_var = io.running_var;
    A.dgamma = io.dgamma;
    A.dbeta = io.dbeta;
    A.mean_parts = mix ? mix->mean_parts : nullptr;
    A.ip = ip;
    A.tx_div = make_fastdiv(lanes);
    A.hw_div = make_fastdiv(uint32_t(d.HW));
    A.w_div = make_fastdiv(uint32_t(d.W));
    A.N = d.N;
    A.C = d.C;
    A.HW = d.HW;
    A.W = d.W;
    A.G = best_g;
    A.whole = ip.shared.h_cnt == d.H && ip.shared.w_cnt == d.W;
    A.TY = gv.nt / int(lanes);
    const bns_box& b = ip.shared;
    const double points = double(b.n_cnt) * double(b.h_cnt) * double(b.w_cnt);
    A.n_v = mix ? mix->n_v : 0;
    const double virtual_points = mix ? double(mix->n_v) * double(d.HW) : 1.0;
    A.inv_s64 = 1.0 / points;
    A.inv_s_v = 1.0 / virtual_points;
    A.mix_beta = mix ? mix->mix_beta : 0.f;
    A.w_s = mix ? float((1.0 - double(mix->mix_beta)) / points) : float(1.0 / points);
    A.w_v = mix ? float(double(mix->mix_beta) / virtual_points) : 0.f;
    A.eps = eps;
    A.momentum = momentum;
    const dim3 grid(uint32_t((d.C + best_g - 1) / best_g));
    if (d.dtype == BNS_F32) launch_any<float, 4>(best_v, backward, mix != nullptr, A, grid, st);
    else launch_any<bf16_t, 8>(best_v, backward, mix != nullptr, A, grid, st);
    return hipGetLastError();
}

}  // namespace bns
