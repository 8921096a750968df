// Single-launch kernels for large N x C x H x W tensors: one block of 512 threads per compute unit, whose register file
// holds the block's whole share of a channel.
//
// A team of T blocks owns a channel, as in bns_fused.hip, and exchanges its sums through the same stamped slots; the
// fewest blocks that hold a channel form a team, so that a tensor takes one or two rounds and most of the time is one long
// run of loads followed by one long run of stores.  Such runs reach the rate of a flat copy whatever the order of the
// planes: a stand-alone probe (bytes only, 64x256x56x56) took 34 / 50 us forward / backward in bf16 with a channel per block
// (flat passes over the same bytes 34 / 48) and 72 / 103 us in fp32 with two rounds of pairs of blocks (flat 64 / 96).
// What that needs:
//   * addresses that cost next to nothing.  A thread's vectors lie T * 512 vectors apart; it walks them with a byte offset
//     and a place in the plane (two additions and a wrap), in every phase anew, instead of dividing or keeping an
//     offset per vector (the same probe with a division per vector that the compiler then kept in registers: 160 us);
//   * loads that never wait for one another: backward reads x in two batches of a few vectors, each requested together with
//     the vectors of dy that it will meet, and what the dx pass needs again of x (the vectors that touch S) is parked in LDS,
//     the first kPark of each thread; beyond that it is read again.  Where S is most of the tensor the KEEPX flavour holds
//     x beside dy, half as many vectors of each;
//   * loads without conditions: in the place of vectors past the end of the channel its first one is loaded, left out of the
//     sums and never stored.
// Sums: a few vectors at a time in fp32, everything beyond in fp64 (only the pair that crosses blocks is rounded to fp32).
#include <hip/hip_runtime.h>

#include "bns_device.hpp"
#include "bns_fused_device.hpp"
#include "bns_internal.hpp"
#include "bns_resident_plan.hpp"

namespace bns {

namespace {

constexpr int kResWaves = kResThreads / kWave;
constexpr int kPark = 17;           // vectors of x per thread that LDS holds (and a place for those that are not kept): 144 of the 160 KiB

struct ResidentArgs {
    FusedArgs f;
    uint32_t stride;        // bytes from a sample to the next
    uint32_t dn, dr, dc;    // step of a thread through the channel: bytes of whole samples, vectors within a plane, within a row
    uint32_t end;           // of the samples, in bytes
    uint32_t s_lo, s_len;   // samples of S, in bytes
    uint32_t v_len;         // samples of the virtual set (Eq. 4), in bytes
};

// How S cuts a plane: not at all; a patch, rows of any length; a patch, rows that are a whole number of vectors.
enum PatchKind { kWholePlanes = 0, kPatch = 1, kPatchRows = 2 };

// Where a thread is: byte offset of its sample from the channel's first element, vector within the plane, and (kPatchRows) vector
// within the row.
struct Walk {
    uint32_t nb, r, c;
};

template <typename T, int V, int PATCH>
struct Walker {
    const ResidentArgs& A;
    bns_box b;
    uint32_t r_lo, r_len, c_lo, c_len;      // kPatchRows: vectors of the plane and of the row that touch the patch; kPatch: elements
    __device__ __forceinline__ explicit Walker(const ResidentArgs& a) : A(a) {}
    __device__ __forceinline__ void channel(int c) {
        b = box_of_channel(A.f.ip, c);
        if constexpr (PATCH == kPatchRows) {
            const uint32_t wv = A.f.wv_div.d;
            r_lo = uint32_t(b.h0) * wv;
            r_len = uint32_t(b.h_cnt) * wv;
            c_lo = uint32_t(b.w0) / V;
            c_len = uint32_t(b.w0 + b.w_cnt - 1) / V - c_lo + 1u;
        } else if constexpr (PATCH == kPatch) {
            r_lo = uint32_t(b.h0) * uint32_t(A.f.W) - uint32_t(V - 1);
            r_len = uint32_t(b.h_cnt) * uint32_t(A.f.W) + uint32_t(V - 1);
        }
    }
    __device__ __forceinline__ Walk start(int j) const {
        const uint32_t i = uint32_t(j) * kResThreads + threadIdx.x, n = fdiv(i, A.f.hwv_div);
        Walk w = {n * A.stride, i - n * A.f.hwv_div.d, 0u};
        if constexpr (PATCH == kPatchRows) w.c = w.r - fdiv(w.r, A.f.wv_div) * A.f.wv_div.d;
        return w;
    }
    // (opaque: each phase walks anew instead of keeping one offset per vector alive)
    __device__ __forceinline__ void next(Walk& w) const {
        if constexpr (PATCH == kPatchRows) asm volatile("" : "+v"(w.nb), "+v"(w.r), "+v"(w.c));
        else asm volatile("" : "+v"(w.nb), "+v"(w.r));
        w.r += A.dr;
        w.nb += A.dn;
        const bool wrap = w.r >= A.f.hwv_div.d;
        w.r -= wrap ? A.f.hwv_div.d : 0u;
        w.nb += wrap ? A.stride : 0u;
        if constexpr (PATCH == kPatchRows) {                // (planes are whole rows: their wrap does not move the column)
            w.c += A.dc;
            w.c -= w.c >= A.f.wv_div.d ? A.f.wv_div.d : 0u;
        }
    }
    // The same for loads, which need no place within the row.
    __device__ __forceinline__ void next_load(Walk& w) const {
        asm volatile("" : "+v"(w.nb), "+v"(w.r));
        w.r += A.dr;
        w.nb += A.dn;
        const bool wrap = w.r >= A.f.hwv_div.d;
        w.r -= wrap ? A.f.hwv_div.d : 0u;
        w.nb += wrap ? A.stride : 0u;
    }
    __device__ __forceinline__ uint32_t element(const Walk& w) const { return plane_offset<T, V>(w.r, A.f.HW); }
    // (all lanes past the end read the channel's first vector: one line, whatever the number of such loads)
    __device__ __forceinline__ uint32_t load_at(const Walk& w) const { return exists(w) ? store_at(w) : 0u; }
    __device__ __forceinline__ uint32_t store_at(const Walk& w) const { return w.nb + element(w) * uint32_t(sizeof(T)); }
    __device__ __forceinline__ bool exists(const Walk& w) const { return w.nb < A.end; }
    // Does the vector touch S?  (kPatch: its rows do.)
    __device__ __forceinline__ bool touches(const Walk& w) const {
        bool t = w.nb - A.s_lo < A.s_len;
        if constexpr (PATCH == kPatchRows) t = t && w.r - r_lo < r_len && w.c - c_lo < c_len;
        if constexpr (PATCH == kPatch) t = t && element(w) - r_lo < r_len;
        return t;
    }
    // Which elements of a vector that touches S lie in it (bit e).
    __device__ __forceinline__ uint32_t in_patch(const Walk& w) const {
        if constexpr (PATCH == kPatchRows) {                // a run of columns
            const int32_t col = int32_t(w.c) * V;
            const int32_t lo = max(b.w0 - col, 0), hi = min(b.w0 + b.w_cnt - col, V);
            return (1u << hi) - (1u << lo);
        }
        uint32_t m = 0u;
        const uint32_t e0 = element(w);
        uint32_t h = fdiv(e0, A.f.w_div), c = e0 - h * uint32_t(A.f.W);
#pragma unroll
        for (int e = 0; e < V; ++e) {
            m |= uint32_t(in_hw(b, h, c)) << e;
            if (++c == uint32_t(A.f.W)) {
                c = 0u;
                ++h;
            }
        }
        return m;
    }
    // Leading elements that the vector before this one holds already: the last vector of a plane that is no whole number of them.
    __device__ __forceinline__ uint32_t shared(const Walk& w) const {
        return Odd<T>::value ? shared_elements<T, V>(w.r, A.f.HW) : 0u;
    }
};

// d if bit e of m is set, else 0 (a NaN that is masked out must not reach a sum).
__device__ __forceinline__ float masked(float d, uint32_t m, int e) {
    return __uint_as_float(__float_as_uint(d) & uint32_t(__builtin_amdgcn_sbfe(int(m), e, 1)));
}

// The sums of the elements of a vector that lie in a set, about a pivot.
template <typename T, int V, int PATCH>
__device__ __forceinline__ void add_in_set(const Walker<T, V, PATCH>& at, const Walk& w, bool hit, const float (&f)[V], float pivot,
                                           float& s1, float& s2) {
    const uint32_t skip = at.shared(w);
    if (PATCH == kWholePlanes && !(Odd<T>::value && __builtin_amdgcn_ballot_w64(skip != 0u))) {
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const float d = hit ? f[e] - pivot : 0.f;
            s1 += d;
            s2 = fmaf(d, d, s2);
        }
    } else {
        uint32_t m = ~0u << skip;
        if constexpr (PATCH != kWholePlanes) m &= at.in_patch(w);
        m = hit ? m : 0u;
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const float d = masked(f[e] - pivot, m, e);
            s1 += d;
            s2 = fmaf(d, d, s2);
        }
    }
}

// Block-wide sums, the same bits in every thread.
__device__ __forceinline__ void block_total(double& a, double& b, double* red) {
    a = wave_sum(a);
    b = wave_sum(b);
    const int wave = threadIdx.x / kWave;
    __syncthreads();                                        // red[] may still be read from the previous use
    if (threadIdx.x % kWave == 0) {
        red[wave] = a;
        red[kResWaves + wave] = b;
    }
    __syncthreads();
    a = red[0];
    b = red[kResWaves];
#pragma unroll
    for (int w = 1; w < kResWaves; ++w) {
        a += red[w];
        b += red[kResWaves + w];
    }
}

// Totals over the team.  A team of one keeps its fp64 sums; otherwise fp32 pairs cross blocks and are added in member order.
__device__ __forceinline__ bool gather(const FusedArgs& F, uint32_t* words, int first_block, uint32_t it, double& a, double& b,
                                       float* team_lds, double* bc) {
    if (F.T == 1) return true;
    double ta, tb;
    const bool ok = team_collect<kResThreads>(F, words, first_block, it, float(a), float(b), ta, tb, team_lds, bc);
    a = ta;
    b = tb;
    return ok;
}

// ---------------------------------------------------------------------------------------
// Forward: Eq. 3, Eq. 8, Eq. 1
// ---------------------------------------------------------------------------------------
template <typename T, int V, int K, int PATCH>
__global__ __launch_bounds__(kResThreads, 2) void resident_forward_kernel(ResidentArgs A) {
    typedef RawVec<T, V> RV;
    __shared__ double red[2 * kResWaves], bc[2];
    __shared__ float team_lds[2 * kMaxTeam];
    __shared__ uint32_t words[3];
    touch_arguments<ResidentArgs>();
    const FusedArgs& F = A.f;
    Walker<T, V, PATCH> at(A);
    const int team = int(fdiv(blockIdx.x, F.team_div)), j = int(blockIdx.x) - team * F.T;
    const T* x = static_cast<const T*>(F.x);
    T* y = static_cast<T*>(F.out);
    const unsigned long long state = stamp_request(F);

    uint32_t it = 0;
    for (int c = team; c < F.cg; c += F.num_teams, ++it) {
        at.channel(c);
        const T* xc = x + size_t(c) * F.HW;
        T* yc = y + size_t(c) * F.HW;
        const Walk w0 = at.start(j);
        const float pivot = load_scalar<T>(at_byte(xc, A.s_lo) + size_t(at.b.h0) * F.W + at.b.w0);     // first sampled element
        const float gamma = F.gamma[c], beta = F.beta[c];   // (no wait here: these are used behind the loads)

        // Loads run kAhead vectors ahead of the sums: a wave that issued all of them first would find most of its vectors there
        // by the time its last load is accepted, and add them up with nothing left in flight.
        typename RV::raw_t v[K];
        Walk wl = w0, w = w0;                               // of the loads, of the sums
        constexpr int kAhead = K < 20 ? K : 20, kGroup = 7; // kGroup: vectors added up in fp32
        auto load = [&](int k) {
            v[k] = RV::ld(at_byte(xc, at.load_at(wl)));
            at.next_load(wl);
        };
#pragma unroll
        for (int k = 0; k < kAhead; ++k) load(k);
        double d1 = 0.0, d2 = 0.0;
#pragma unroll
        for (int k0 = 0; k0 < K; k0 += kGroup) {
            float s1 = 0.f, s2 = 0.f;
#pragma unroll
            for (int k = k0 + kAhead; k < k0 + kAhead + kGroup && k < K; ++k) load(k);
#pragma unroll
            for (int k = k0; k < k0 + kGroup && k < K; ++k) {
                const bool hit = at.touches(w);
                if (__builtin_amdgcn_ballot_w64(hit)) {     // (the whole wave or none of it)
                    float f[V];
                    opaque_raw(v[k]);
                    RV::unpack(v[k], f);
                    add_in_set<T, V, PATCH>(at, w, hit, f, pivot, s1, s2);
                }
                at.next(w);
            }
            d1 += double(s1);
            d2 += double(s2);
            asm volatile("" : "+v"(d1), "+v"(d2));          // (the sums keep pace with the loads)
        }
        if (it == 0) stamp_accept(F, state, words);
        block_total(d1, d2, red);
        team_publish(F, read_stamp(F, words), team * F.T, j, it, float(d1), float(d2));
        const bool arrived = gather(F, words, team * F.T, it, d1, d2, team_lds, bc);
        const double m1 = d1 * F.inv_s64;
        const double mean = double(pivot) + m1;
        double var = d2 * F.inv_s64 - m1 * m1;
        if (!(var >= 0.0)) var = (var != var) ? var : 0.0;  // clamp rounding; keep NaN visible
        const float mu = float(mean);
        const float r = float(inv_sqrt(var + double(F.eps)));
        if (j == 0 && threadIdx.x == 0) {
            F.save_mean[c] = mu;
            F.save_invstd[c] = r;
            const double al = double(F.momentum);
            // (a wait for a team-mate that ran out leaves NaN statistics; the moving averages then stay as they are)
            if (F.running_mean && arrived) F.running_mean[c] = float((1.0 - al) * double(F.running_mean[c]) + al * mean);
            if (F.running_var && arrived) F.running_var[c] = float((1.0 - al) * double(F.running_var[c]) + al * var);
        }
        const float sc = settled(gamma) * r, be = settled(beta);
        w = w0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            float f[V];
            opaque_raw(v[k]);
            RV::unpack(v[k], f);
#pragma unroll
            for (int e = 0; e < V; ++e) f[e] = fmaf(f[e] - mu, sc, be);
            if (at.exists(w)) RV::st(at_byte(yc, at.store_at(w)), RV::pack(f));
            at.next(w);
        }
    }
    team_done(F, j, read_stamp(F, words));
}

// ---------------------------------------------------------------------------------------
// Backward: the sums of Eq. 5, Eq. 6
// ---------------------------------------------------------------------------------------
template <typename T, int V, int K, int PATCH, bool KEEPX, bool MIXED>
__global__ __launch_bounds__(kResThreads, 2) void resident_backward_kernel(ResidentArgs A) {
    typedef RawVec<T, V> RV;
    typedef typename RV::raw_t raw_t;
    __shared__ raw_t park[KEEPX ? 1 : (kPark + 1) * kResThreads];
    __shared__ double red[2 * kResWaves], bc[2];
    __shared__ float team_lds[2 * kMaxTeam];
    __shared__ float consts[2][2];
    __shared__ uint32_t words[3];
    touch_arguments<ResidentArgs>();
    const FusedArgs& F = A.f;
    Walker<T, V, PATCH> at(A);
    const int team = int(fdiv(blockIdx.x, F.team_div)), j = int(blockIdx.x) - team * F.T;
    const T* x = static_cast<const T*>(F.x);
    const T* dy = static_cast<const T*>(F.dy);
    T* dx = static_cast<T*>(F.out);
    const unsigned long long state = stamp_request(F);

    uint32_t it = 0;
    for (int c = team; c < F.cg; c += F.num_teams, ++it) {
        at.channel(c);
        const T* xc = x + size_t(c) * F.HW;
        const T* gc = dy + size_t(c) * F.HW;
        T* dc = dx + size_t(c) * F.HW;
        float mu = F.save_mean[c], r = F.save_invstd[c], ga = F.gamma[c];       // (no wait here: used behind the first loads)
        const Walk w0 = at.start(j);

        raw_t g[K], xk[KEEPX ? K : 1];
        double d1 = 0.0, d2 = 0.0;
        uint32_t parked = 0;
        Walk wl = w0, w = w0;                               // of the loads, of the sums
        // What came with the mean waits in LDS, behind the barriers of the sums: held in registers, these two and the start of the walk
        // sent 12 to 52 bytes of these kernels through scratch memory.  Not where registers suffice: with ten vectors of each tensor in
        // flight the branch costs a pause (64x256x56x56 bf16, everything, 54.3 -> 56.5 us).
        constexpr bool kStash = !KEEPX || (PATCH == kPatch && V == 8);
        float* held = consts[it & 1u];                      // (a slow wave may still read those of the channel before)
        auto keep_constants = [&]() {
            if (kStash && threadIdx.x == 0) {
                held[0] = r;
                held[1] = ga;
            }
        };
        // The sums of one vector.
        auto add = [&](const raw_t& gv, const raw_t& xv, float& s1, float& s2) {
            float fg[V], fx[V];
            RV::unpack(gv, fg);
            RV::unpack(xv, fx);
            if constexpr (Odd<T>::value) {
                const uint32_t skip = at.shared(w);
#pragma unroll
                for (int e = 0; e < V - 1; ++e)
                    if (uint32_t(e) < skip) fg[e] = 0.f, fx[e] = mu;
            }
            float t1 = 0.f, t2 = 0.f;
#pragma unroll
            for (int e = 0; e < V; ++e) {
                t1 += fg[e];
                t2 = fmaf(fg[e], fx[e] - mu, t2);
                if (V == 8 && !KEEPX && e % 2 == 1) asm volatile("" : "+v"(t1), "+v"(t2));      // (two elements at a time: registers)
            }
            const bool ok = at.exists(w);
            s1 += ok ? t1 : 0.f;
            s2 += ok ? t2 : 0.f;
            if (V == 8) asm volatile("" : "+v"(s1), "+v"(s2));
        };
        if constexpr (KEEPX) {
            constexpr int kAhead = 10, kGroup = 3;          // as in the forward kernel
            auto load = [&](int k) {
                const uint32_t off = at.load_at(wl);
                g[k] = RV::ld(at_byte(gc, off));
                xk[k] = RV::ld(at_byte(xc, off));
                at.next_load(wl);
            };
#pragma unroll
            for (int k = 0; k < kAhead; ++k) load(k);
            mu = settled(mu);
            keep_constants();
#pragma unroll
            for (int k0 = 0; k0 < K; k0 += kGroup) {
                float s1 = 0.f, s2 = 0.f;
#pragma unroll
                for (int k = k0 + kAhead; k < k0 + kAhead + kGroup && k < K; ++k) load(k);
#pragma unroll
                for (int k = k0; k < k0 + kGroup && k < K; ++k) {
                    opaque_raw(xk[k]);
                    add(g[k], xk[k], s1, s2);
                    at.next(w);
                }
                d1 += double(s1);
                d2 += double(s2);
                asm volatile("" : "+v"(d1), "+v"(d2));
            }
            if (it == 0) stamp_accept(F, state, words);
        } else {
            constexpr int XB = V == 8 ? 2 : 3;              // vectors of x per batch, two batches in flight
            raw_t b0[XB], b1[XB];
            auto batch = [&](raw_t(&xb)[XB], int k0) {
#pragma unroll
                for (int u = 0; u < XB; ++u)
                    if (k0 + u < K) {
                        const uint32_t off = at.load_at(wl);
                        g[k0 + u] = RV::ld(at_byte(gc, off));
                        xb[u] = RV::ld(at_byte(xc, off));
                        at.next_load(wl);
                    }
            };
            auto use = [&](raw_t(&xb)[XB], int k0) {
                float s1 = 0.f, s2 = 0.f;
#pragma unroll
                for (int u = 0; u < XB; ++u)
                    if (k0 + u < K) {
                        opaque_raw(xb[u]);
                        add(g[k0 + u], xb[u], s1, s2);
                        const bool hit = at.touches(w);
                        // (stored whether it is needed or not: no branch)
                        park[(hit ? min(parked, uint32_t(kPark)) : uint32_t(kPark)) * kResThreads + threadIdx.x] = xb[u];
                        parked += hit ? 1u : 0u;
                        at.next(w);
                    }
                d1 += double(s1);
                d2 += double(s2);
                asm volatile("" : "+v"(d1), "+v"(d2));      // (the sums keep pace with the loads, or the registers run out)
            };
            batch(b0, 0);
            mu = settled(mu);
            keep_constants();
#pragma unroll
            for (int k0 = 0; k0 < K; k0 += 2 * XB) {
                if (k0 + XB < K) batch(b1, k0 + XB);
                use(b0, k0);
                if (k0 + 2 * XB < K) batch(b0, k0 + 2 * XB);
                if (k0 + XB < K) use(b1, k0 + XB);
            }
            if (it == 0) stamp_accept(F, state, words);
        }
        block_total(d1, d2, red);
        team_publish(F, read_stamp(F, words), team * F.T, j, it, float(d1), float(d2));
        gather(F, words, team * F.T, it, d1, d2, team_lds, bc);

        r = kStash ? held[0] : settled(r);
        ga = kStash ? held[1] : settled(ga);
        const float dbeta = float(d1);
        const float dgamma = float(d2 * double(r));
        if (j == 0 && threadIdx.x == 0) {
            F.dbeta[c] = dbeta;
            F.dgamma[c] = dgamma;
        }
        const float a = ga * r;
        const float wgt_s = MIXED ? F.w_s : F.inv_s;
        const float k1 = a * wgt_s * dbeta, k2 = a * wgt_s * dgamma * r;
        const float centre = MIXED ? F.mean_parts[F.C + c] : mu;
        const float k1v = MIXED ? a * F.w_v * dbeta : 0.f, k2v = MIXED ? a * F.w_v * dgamma * r : 0.f;
        const float centre_v = MIXED ? F.mean_parts[c] : 0.f;
        parked = 0;
        w = at.start(int(opaque(uint32_t(j))));             // (not kept, either)
#pragma unroll
        for (int k = 0; k < K; ++k) {
            float f[V];
            opaque_raw(g[k]);
            if constexpr (KEEPX) opaque_raw(xk[k]);
            RV::unpack(g[k], f);
            const bool hit = at.touches(w), virt = MIXED && w.nb < A.v_len;
            if (!(hit || virt)) {
#pragma unroll
                for (int e = 0; e < V; ++e) f[e] *= a;
            } else {
                float fx[V];
                if constexpr (KEEPX) {
                    RV::unpack(xk[k], fx);
                } else {
                    raw_t xr;
                    if (parked < uint32_t(kPark)) xr = park[parked * kResThreads + threadIdx.x];
                    else xr = RV::ld(at_byte(xc, at.store_at(w)));
                    RV::unpack(xr, fx);
                    ++parked;
                }
                const uint32_t m = PATCH != kWholePlanes && !virt ? at.in_patch(w) : ~0u;
                const float q1 = virt ? k1v : k1, q2 = virt ? k2v : k2, ce = virt ? centre_v : centre;
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const float corr = fmaf(q2, fx[e] - ce, q1);
                    f[e] = fmaf(a, f[e], PATCH == kWholePlanes ? -corr : -masked(corr, m, e));
                }
            }
            if (at.exists(w)) RV::st(at_byte(dc, at.store_at(w)), RV::pack(f));
            at.next(w);
        }
    }
    team_done(F, j, read_stamp(F, words));
}

template <typename T, int V, int PATCH>
const void* resident_ptr(bool backward, bool keep_x, bool mixed) {
    constexpr bool f32 = V == 4, odd = Odd<T>::value, general = PATCH == kPatch;
    constexpr int kForward = resident_vectors(f32, odd, general, false, false), kBig = resident_vectors(f32, odd, general, true, false),
                  kPair = resident_vectors(f32, odd, general, true, true);
    if (!backward) return reinterpret_cast<const void*>(&resident_forward_kernel<T, V, kForward, PATCH>);
    return mixed    ? reinterpret_cast<const void*>(&resident_backward_kernel<T, V, kPair, PATCH, true, true>)
           : keep_x ? reinterpret_cast<const void*>(&resident_backward_kernel<T, V, kPair, PATCH, true, false>)
                    : reinterpret_cast<const void*>(&resident_backward_kernel<T, V, kBig, PATCH, false, false>);
}

const void* resident_kernel(const Dims& d, const ResidentChoice& c, bool backward, bool mixed) {
    const bool x = c.keep_x, rows = c.patch && !c.general;
    if (d.dtype == BNS_F32) {
        if (c.odd) return c.patch ? resident_ptr<f32_odd, 4, kPatch>(backward, x, mixed) : resident_ptr<f32_odd, 4, kWholePlanes>(backward, x, mixed);
        return rows      ? resident_ptr<float, 4, kPatchRows>(backward, x, mixed)
               : c.patch ? resident_ptr<float, 4, kPatch>(backward, x, mixed)
                         : resident_ptr<float, 4, kWholePlanes>(backward, x, mixed);
    }
    if (c.odd) return c.patch ? resident_ptr<bf16_odd, 8, kPatch>(backward, x, mixed) : resident_ptr<bf16_odd, 8, kWholePlanes>(backward, x, mixed);
    return rows      ? resident_ptr<bf16_t, 8, kPatchRows>(backward, x, mixed)
           : c.patch ? resident_ptr<bf16_t, 8, kPatch>(backward, x, mixed)
                     : resident_ptr<bf16_t, 8, kWholePlanes>(backward, x, mixed);
}

}  // namespace

hipError_t launch_resident(const Dims& d, const IndexParams& ip, bool backward, const FusedIo& io, float eps, float momentum,
                           void* header, void* slots, size_t slot_bytes, hipStream_t st, int cus, const FusedMix* mix,
                           bool may_create_event) {
    const ResidentChoice choice = resident_choice(d, ip, backward, mix != nullptr, g_tuning.resident, cus);
    if (!choice.take) return hipErrorNotSupported;
    const uint32_t e = d.dtype == BNS_F32 ? 4u : 2u, hwv = choice.plane_vectors;
    const int V = choice.vector;
    const bns_box& b = ip.shared;
    const uint64_t tot = uint64_t(d.N) * hwv;
    const int64_t T = choice.plan.T, teams = choice.plan.teams, rounds = choice.plan.rounds;
    const int K = choice.held;
    const void* kernel = resident_kernel(d, choice, backward, mix != nullptr);
    // offsets within the tensor are 32-bit, those of vectors past the end of a channel included
    const uint64_t stride = uint64_t(d.C) * uint64_t(d.HW) * e;
    const uint64_t step = uint64_t(T) * kResThreads;
    if ((step * uint64_t(K + 1) / hwv + 2) * stride >= (uint64_t(1) << 32)) return hipErrorNotSupported;
    if (T > 1 && size_t(teams * T) * 2 * 2 * sizeof(unsigned long long) > slot_bytes)
        return hipErrorNotSupported;

    ResidentArgs A;
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
    F.ip = ip;
    F.hwv_div = make_fastdiv(hwv);
    F.w_div = make_fastdiv(uint32_t(d.W));
    F.wv_div = make_fastdiv(uint32_t(std::max(d.W / V, 1)));       // (used when W is a multiple of V)
    F.C = d.C;
    F.W = d.W;
    F.HW = d.HW;
    F.cg = d.C;
    F.T = int32_t(T);
    F.team_div = make_fastdiv(uint32_t(T));
    F.num_teams = int32_t(teams);
    F.tot = uint32_t(tot);
    F.stamp_advance = uint32_t(rounds) + 1u;
    F.stamp_seed = next_stamp_seed();
    const int spin = g_tuning.test_spin_limit;
    F.spin_limit = spin > 0 ? uint32_t(spin) : kSpinLimit;
    F.mute = g_tuning.test_mute_exchange;
    F.eps = eps;
    F.momentum = momentum;
    const double points = double(b.n_cnt) * double(b.h_cnt) * double(b.w_cnt);
    F.inv_s64 = 1.0 / points;
    F.inv_s = float(F.inv_s64);
    F.inv_s_v = 1.0;
    A.v_len = 0;
    if (mix) {
        F.n_v = mix->n_v;
        F.mix_beta = mix->mix_beta;
        const double virtual_points = double(mix->n_v) * double(d.HW);
        F.inv_s_v = 1.0 / virtual_points;
        F.w_v = float(double(mix->mix_beta) / virtual_points);
        F.w_s = float((1.0 - double(mix->mix_beta)) / points);
        F.mean_parts = mix->mean_parts;
        A.v_len = uint32_t(uint64_t(mix->n_v) * stride);
    }
    A.stride = uint32_t(stride);
    A.dn = uint32_t(step / hwv * stride);
    A.dr = uint32_t(step % hwv);
    A.dc = uint32_t(step % hwv % F.wv_div.d);
    A.end = uint32_t(uint64_t(d.N) * stride);
    A.s_lo = uint32_t(uint64_t(b.n0) * stride);
    A.s_len = uint32_t(uint64_t(b.n_cnt) * stride);
    (backward ? t_last_fused_backward : t_last_fused_forward) = backward ? 5 : 4;
    t_last_team[backward] = F.T;
    t_last_variant[backward] = 0;
    void* params[] = {&A};
    return launch_waiting(kernel, dim3(uint32_t(teams * T)), dim3(kResThreads), params, T > 1, may_create_event, st);
}

}  // namespace bns
