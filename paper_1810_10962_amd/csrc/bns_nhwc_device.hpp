// Pieces shared by the kernels for the N x H x W x C layout: the rows of S, as a list and as a membership test.
#pragma once
#include <hip/hip_runtime.h>

#include "bns_device.hpp"
#include "bns_internal.hpp"

namespace bns {
namespace {

struct RowSet {                 // the rows of S: sampled row i -> (n, ph, pw) -> row
    int32_t n0, h0, w0;
    int32_t H, W;
    FastDiv patch_div;          // h_cnt * w_cnt
    FastDiv pw_div;             // w_cnt
    uint32_t rows;              // n_cnt * h_cnt * w_cnt
    uint32_t pivot_rows;        // min(kPivotRows, rows)
    float inv_pivot_rows;
    double inv_rows;            // 1 / rows
    bool contiguous;            // sampled row i = sampled row 0 + i
};

// The one-pass variance is taken about a pivot p_c close to the mean: sum (x - p)^2 / s - (sum (x - p) / s)^2
// loses (1 + 2 k^2) digits' worth for a pivot k standard deviations off.  p_c = mean of the first few
// sampled rows (added in row order, the same expression in the partial and the finalize kernel).
constexpr int kPivotRows = 8;

// The pivot keeps only its upper 16 bits (a bf16 pattern): x - p is then exact for bf16 data and
// carries no low bits that every addition would round the same way.
__device__ __forceinline__ float coarse(float p) { return __uint_as_float(__float_as_uint(p) & 0xFFFF0000u); }

// Accumulation.  A thread adds up to a thousand rows.  Adding them one by one into an fp32 sum loses
// n * eps / 4 of the result when the addends share their low bits (constant dy, activations on a grid,
// exact zeros after a ReLU): every addition then rounds the same way and the errors add up instead of
// averaging out.  So the rows of one unrolled iteration are added in fp32 and each group's sum goes
// into an fp64 accumulator (one fp64 add per group and channel: far below the fp64 rate).

__host__ __device__ __forceinline__ uint32_t sampled_row(const RowSet& s, uint32_t i) {
    const uint32_t n = fdiv(i, s.patch_div);
    const uint32_t r = i - n * s.patch_div.d;
    const uint32_t ph = fdiv(r, s.pw_div);
    const uint32_t pw = r - ph * s.pw_div.d;
    return ((uint32_t(s.n0) + n) * uint32_t(s.H) + uint32_t(s.h0) + ph) * uint32_t(s.W) + uint32_t(s.w0) + pw;
}

struct RowBox {                 // membership of a row in S
    uint32_t n0, n1, h0, h1, w0, w1;
    FastDiv hw_div, w_div;
};

__device__ __forceinline__ bool row_in(const RowBox& b, uint32_t row) {
    const uint32_t n = fdiv(row, b.hw_div);
    const uint32_t rem = row - n * b.hw_div.d;
    const uint32_t h = fdiv(rem, b.w_div);
    const uint32_t w = rem - h * b.w_div.d;
    return n >= b.n0 && n < b.n1 && h >= b.h0 && h < b.h1 && w >= b.w0 && w < b.w1;
}

inline RowSet make_rowset(const Dims& d, const bns_box& b) {
    RowSet s;
    s.n0 = b.n0;
    s.h0 = b.h0;
    s.w0 = b.w0;
    s.H = d.H;
    s.W = d.W;
    s.patch_div = make_fastdiv(uint32_t(b.h_cnt) * uint32_t(b.w_cnt));
    s.pw_div = make_fastdiv(uint32_t(b.w_cnt));
    s.rows = uint32_t(b.n_cnt) * uint32_t(b.h_cnt) * uint32_t(b.w_cnt);
    s.pivot_rows = s.rows < uint32_t(kPivotRows) ? s.rows : uint32_t(kPivotRows);
    s.inv_pivot_rows = 1.0f / float(s.pivot_rows);
    s.inv_rows = 1.0 / double(s.rows);
    s.contiguous = (b.w_cnt == d.W && (b.h_cnt == d.H || b.n_cnt == 1)) || (b.n_cnt == 1 && b.h_cnt == 1);
    return s;
}

inline RowBox make_rowbox(const Dims& d, const bns_box& b) {
    RowBox B;
    B.n0 = uint32_t(b.n0);
    B.n1 = uint32_t(b.n0 + b.n_cnt);
    B.h0 = uint32_t(b.h0);
    B.h1 = uint32_t(b.h0 + b.h_cnt);
    B.w0 = uint32_t(b.w0);
    B.w1 = uint32_t(b.w0 + b.w_cnt);
    B.hw_div = make_fastdiv(uint32_t(d.HW));
    B.w_div = make_fastdiv(uint32_t(d.W));
    return B;
}

}  // namespace
}  // namespace bns
