// Device-side building blocks: 128-bit vector access for fp32 / bf16 storage,
// wave64 and block reductions, and division by launch-uniform divisors.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bns {

constexpr int kWave = 64;     // gfx950 wavefront
constexpr int kBlock = 256;   // threads per block in every kernel (4 waves)

// ---------------------------------------------------------------------------
// Division of a 32-bit dividend (< 2^31) by a divisor fixed for the launch:
// round-up multiplier method (Granlund & Montgomery 1994).  q = (mulhi(n, mul) + n) >> shift.
// ---------------------------------------------------------------------------
struct FastDiv {
    uint32_t mul, shift, d;
};

inline FastDiv make_fastdiv(uint32_t d) {  // host; d >= 1
    FastDiv f;
    f.d = d;
    uint32_t l = 0;
    while ((uint64_t(1) << l) < d) ++l;     // ceil(log2 d)
    f.shift = l;
    f.mul = uint32_t(((uint64_t(1) << 32) * ((uint64_t(1) << l) - d)) / d + 1);
    return f;
}

__host__ __device__ __forceinline__ uint32_t fdiv(uint32_t n, const FastDiv& f) {
    return (uint32_t((uint64_t(n) * f.mul) >> 32) + n) >> f.shift;
}

// 1 / sqrt(x) in fp64, within two units in the last place: the hardware's estimate (some 23 bits) and one step of third order,
// x (y (1 + e / 2 + 3 e^2 / 8))^2 = 1 + O(e^3) with e = 1 - x y^2.  x = 0, infinity and NaN keep the estimate (infinity, 0, NaN).
// A dozen instructions where a square root and a division are some 90, each a few nanoseconds in blocks of 512 threads that all wait
// for them (64-bit and 32-bit instructions issue at one rate).
__device__ __forceinline__ double inv_sqrt(double x) {
    const double y = __builtin_amdgcn_rsq(x), e = fma(-x * y, y, 1.0);
    return x > 0.0 && x < __builtin_inf() ? fma(y * e, fma(e, 0.375, 0.5), y) : y;
}

// Requests every cache line of the kernel's arguments at once.  A kernel with some hundred bytes of them otherwise fetches them line by
// line, each where it is first needed and with a wait of its own: 0.2 us a line, where nothing else is going on yet.
template <typename Args>
__device__ __forceinline__ void touch_arguments() {
    typedef const uint32_t __attribute__((address_space(4))) word_t;
    const word_t* p = (const word_t*)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr int kLines = int((sizeof(Args) + 63) / 64);
    static_assert(kLines <= 12, "one operand each");
    uint32_t w[12];
#pragma unroll
    for (int i = 0; i < 12; ++i) w[i] = p[16 * (i < kLines ? i : 0)];
    asm volatile("" ::"s"(w[0]), "s"(w[1]), "s"(w[2]), "s"(w[3]), "s"(w[4]), "s"(w[5]), "s"(w[6]), "s"(w[7]), "s"(w[8]), "s"(w[9]),
                 "s"(w[10]), "s"(w[11]));
}

// ---------------------------------------------------------------------------
// Storage types.  bf16 is handled as raw 16-bit patterns: widening is a shift,
// narrowing is the hardware conversion (round to nearest, ties to even; NaN stays NaN).
// ---------------------------------------------------------------------------
struct bf16_t {
    uint16_t bits;
};

__device__ __forceinline__ float bf16_to_f32(uint32_t b) { return __uint_as_float(b << 16); }

// Two floats -> two bf16 packed in one dword (lo in bits 0..15): v_cvt_pk_bf16_f32 on gfx950.
typedef __bf16 bf16x2_native __attribute__((ext_vector_type(2)));
typedef float f32x2_native __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    const f32x2_native v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_native));
}
__device__ __forceinline__ uint32_t f32_to_bf16(float f) { return pack_bf16x2(f, 0.f) & 0xFFFFu; }

// Vec<T, V>: V consecutive elements of storage type T, moved with one access of
// V * sizeof(T) bytes and exposed as V floats.
template <typename T, int V>
struct Vec;

template <>
struct Vec<float, 1> {
    float f[1];
    __device__ __forceinline__ void load(const float* p) { f[0] = *p; }
    __device__ __forceinline__ void load_nt(const float* p) { f[0] = __builtin_nontemporal_load(p); }
    __device__ __forceinline__ void store(float* p) const { *p = f[0]; }
    __device__ __forceinline__ void store_nt(float* p) const { __builtin_nontemporal_store(f[0], p); }
};

template <>
struct Vec<float, 4> {
    float f[4];
    typedef float v4 __attribute__((ext_vector_type(4)));
    __device__ __forceinline__ void load(const float* p) {
        v4 v = *reinterpret_cast<const v4*>(p);
        f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
    }
    __device__ __forceinline__ void load_nt(const float* p) {
        v4 v = __builtin_nontemporal_load(reinterpret_cast<const v4*>(p));
        f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
    }
    __device__ __forceinline__ void store(float* p) const {
        v4 v = {f[0], f[1], f[2], f[3]};
        *reinterpret_cast<v4*>(p) = v;
    }
    __device__ __forceinline__ void store_nt(float* p) const {
        v4 v = {f[0], f[1], f[2], f[3]};
        __builtin_nontemporal_store(v, reinterpret_cast<v4*>(p));
    }
};

template <>
struct Vec<bf16_t, 1> {
    float f[1];
    __device__ __forceinline__ void load(const bf16_t* p) { f[0] = bf16_to_f32(p->bits); }
    __device__ __forceinline__ void load_nt(const bf16_t* p) { load(p); }
    __device__ __forceinline__ void store(bf16_t* p) const { p->bits = uint16_t(f32_to_bf16(f[0])); }
    __device__ __forceinline__ void store_nt(bf16_t* p) const { store(p); }
};

template <>
struct Vec<bf16_t, 4> {
    float f[4];
    typedef uint32_t u2 __attribute__((ext_vector_type(2)));
    __device__ __forceinline__ void unpack(u2 v) {
        f[0] = bf16_to_f32(v.x & 0xFFFFu); f[1] = __uint_as_float(v.x & 0xFFFF0000u);
        f[2] = bf16_to_f32(v.y & 0xFFFFu); f[3] = __uint_as_float(v.y & 0xFFFF0000u);
    }
    __device__ __forceinline__ u2 pack() const {
        u2 v;
        v.x = pack_bf16x2(f[0], f[1]);
        v.y = pack_bf16x2(f[2], f[3]);
        return v;
    }
    __device__ __forceinline__ void load(const bf16_t* p) { unpack(*reinterpret_cast<const u2*>(p)); }
    __device__ __forceinline__ void load_nt(const bf16_t* p) {
        unpack(__builtin_nontemporal_load(reinterpret_cast<const u2*>(p)));
    }
    __device__ __forceinline__ void store(bf16_t* p) const { *reinterpret_cast<u2*>(p) = pack(); }
    __device__ __forceinline__ void store_nt(bf16_t* p) const {
        __builtin_nontemporal_store(pack(), reinterpret_cast<u2*>(p));
    }
};

template <>
struct Vec<bf16_t, 8> {
    float f[8];
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    __device__ __forceinline__ void unpack(u4 v) {
        f[0] = bf16_to_f32(v.x & 0xFFFFu); f[1] = __uint_as_float(v.x & 0xFFFF0000u);
        f[2] = bf16_to_f32(v.y & 0xFFFFu); f[3] = __uint_as_float(v.y & 0xFFFF0000u);
        f[4] = bf16_to_f32(v.z & 0xFFFFu); f[5] = __uint_as_float(v.z & 0xFFFF0000u);
        f[6] = bf16_to_f32(v.w & 0xFFFFu); f[7] = __uint_as_float(v.w & 0xFFFF0000u);
    }
    __device__ __forceinline__ u4 pack() const {
        u4 v;
        v.x = pack_bf16x2(f[0], f[1]);
        v.y = pack_bf16x2(f[2], f[3]);
        v.z = pack_bf16x2(f[4], f[5]);
        v.w = pack_bf16x2(f[6], f[7]);
        return v;
    }
    __device__ __forceinline__ void load(const bf16_t* p) { unpack(*reinterpret_cast<const u4*>(p)); }
    __device__ __forceinline__ void load_nt(const bf16_t* p) {
        unpack(__builtin_nontemporal_load(reinterpret_cast<const u4*>(p)));
    }
    __device__ __forceinline__ void store(bf16_t* p) const { *reinterpret_cast<u4*>(p) = pack(); }
    __device__ __forceinline__ void store_nt(bf16_t* p) const {
        __builtin_nontemporal_store(pack(), reinterpret_cast<u4*>(p));
    }
};

// The same elements in planes that are no whole number of vectors (and so may start at any element): a plane then has
// ceil(HW / V) vectors, accessed at element alignment, and the last one is moved back so that it ends with the plane.  The
// elements it shares with the vector before it are left out of sums (the first `skip`) and written twice with the same bits.
struct f32_odd {
    float v;
};
struct bf16_odd {
    uint16_t bits;
};
template <typename T>
struct Odd {
    static constexpr bool value = false;
};
template <>
struct Odd<f32_odd> {
    static constexpr bool value = true;
};
template <>
struct Odd<bf16_odd> {
    static constexpr bool value = true;
};
// First element, within its plane, of vector i of a plane of HW elements.
template <typename T, int V>
__device__ __forceinline__ uint32_t plane_offset(uint32_t i, int HW) {
    return Odd<T>::value ? min(i * V, uint32_t(HW) - V) : i * V;
}

// Elements that vector i shares with the one before it.
template <typename T, int V>
__device__ __forceinline__ uint32_t shared_elements(uint32_t i, int HW) {
    return i * V - plane_offset<T, V>(i, HW);
}

template <>
struct Vec<f32_odd, 4> {
    float f[4];
    typedef float v4 __attribute__((ext_vector_type(4)));
    typedef v4 v4e __attribute__((aligned(4)));
    __device__ __forceinline__ void set(v4 v) { f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w; }
    __device__ __forceinline__ void load(const f32_odd* p) { set(*reinterpret_cast<const v4e*>(p)); }
    __device__ __forceinline__ void load_nt(const f32_odd* p) { set(__builtin_nontemporal_load(reinterpret_cast<const v4e*>(p))); }
    __device__ __forceinline__ void store(f32_odd* p) const { *reinterpret_cast<v4e*>(p) = v4{f[0], f[1], f[2], f[3]}; }
    __device__ __forceinline__ void store_nt(f32_odd* p) const {
        const v4 v = {f[0], f[1], f[2], f[3]};
        __builtin_nontemporal_store(v, reinterpret_cast<v4e*>(p));
    }
};
template <>
struct Vec<bf16_odd, 8> : Vec<bf16_t, 8> {
    typedef u4 u4e __attribute__((aligned(2)));
    __device__ __forceinline__ void load(const bf16_odd* p) { unpack(*reinterpret_cast<const u4e*>(p)); }
    __device__ __forceinline__ void load_nt(const bf16_odd* p) { unpack(__builtin_nontemporal_load(reinterpret_cast<const u4e*>(p))); }
    __device__ __forceinline__ void store(bf16_odd* p) const { *reinterpret_cast<u4e*>(p) = pack(); }
    __device__ __forceinline__ void store_nt(bf16_odd* p) const { __builtin_nontemporal_store(pack(), reinterpret_cast<u4e*>(p)); }
};

template <typename T>
__device__ __forceinline__ float load_scalar(const T* p);
template <>
__device__ __forceinline__ float load_scalar<f32_odd>(const f32_odd* p) { return p->v; }
template <>
__device__ __forceinline__ float load_scalar<bf16_odd>(const bf16_odd* p) { return bf16_to_f32(p->bits); }
template <>
__device__ __forceinline__ float load_scalar<float>(const float* p) { return *p; }
template <>
__device__ __forceinline__ float load_scalar<bf16_t>(const bf16_t* p) { return bf16_to_f32(p->bits); }

// ---------------------------------------------------------------------------
// Reductions, in a fixed order.  Block: one value per wave through
// LDS, then the first wave adds the four in index order.
// ---------------------------------------------------------------------------
// Inclusive scan with data-parallel-primitive moves (shifts of 1, 2, 4, 8 lanes inside each row of 16, then the last lane of row 0 / row 2
// broadcast into the next row, then lane 31 into the upper half), after which lane 63 holds the total: a balanced tree, neighbours
// first.  A butterfly of cross-lane shuffles is one, too (distant lanes first, so its bits differ), but goes through LDS and needs lane-index registers
// (64x2048x7x7 bf16, the sums of a group of channels 0.8 -> 0.5 us).
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_or_zero(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, ROWS, 0xf, true));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_or_zero(double x) {
    typedef int pair_t __attribute__((ext_vector_type(2)));
    pair_t w = __builtin_bit_cast(pair_t, x);
    w.x = __builtin_amdgcn_update_dpp(0, w.x, CTRL, ROWS, 0xf, true);
    w.y = __builtin_amdgcn_update_dpp(0, w.y, CTRL, ROWS, 0xf, true);
    return __builtin_bit_cast(double, w);
}
__device__ __forceinline__ float last_lane(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), kWave - 1));
}
__device__ __forceinline__ double last_lane(double x) {
    typedef int pair_t __attribute__((ext_vector_type(2)));
    pair_t w = __builtin_bit_cast(pair_t, x);
    w.x = __builtin_amdgcn_readlane(w.x, kWave - 1);
    w.y = __builtin_amdgcn_readlane(w.y, kWave - 1);
    return __builtin_bit_cast(double, w);
}
// Sum over the 64 lanes of a wave (all of them active), returned as a wave-uniform value; float or double.
template <typename F>
__device__ __forceinline__ F wave_sum(F v) {
    v += dpp_or_zero<0x111, 0xf>(v);    // row_shr:1
    v += dpp_or_zero<0x112, 0xf>(v);    // row_shr:2
    v += dpp_or_zero<0x114, 0xf>(v);    // row_shr:4
    v += dpp_or_zero<0x118, 0xf>(v);    // row_shr:8
    v += dpp_or_zero<0x142, 0xa>(v);    // row_bcast:15 into rows 1, 3
    v += dpp_or_zero<0x143, 0xc>(v);    // row_bcast:31 into rows 2, 3
    return last_lane(v);
}

// Sum of two values over a block of NT threads; result valid in thread 0.  `lds` holds
// 2 * (NT / kWave) floats.
template <int NT = kBlock>
__device__ __forceinline__ void block_sum2(float& a, float& b, float* lds) {
    a = wave_sum(a);
    b = wave_sum(b);
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    constexpr int nw = NT / kWave;
    if (lane == 0) {
        lds[wave] = a;
        lds[nw + wave] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        float sa = lds[0], sb = lds[nw];
#pragma unroll
        for (int w = 1; w < nw; ++w) {
            sa += lds[w];
            sb += lds[nw + w];
        }
        a = sa;
        b = sb;
    }
}

}  // namespace bns
