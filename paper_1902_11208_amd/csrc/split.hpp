// fp32 values as sums of three bf16 values, for products on the bf16 MFMA.
//
// A float has 24 significant bits; hi = rne_bf16(v), mid = rne_bf16(v - hi),
// lo = rne_bf16(v - hi - mid) carry 8 each (both differences are exact), so
// v = hi + mid + lo exactly (down to about 1e-33, where lo falls below bf16's
// range). Of the nine products of two such sums the six largest are kept (hi
// hi, hi mid, mid hi, hi lo, lo hi, mid mid); the dropped ones reach 2^-25 of
// the product each, 2^-24 together: an ulp at most. They accumulate in fp32.
// One 16x16x32 bf16 MFMA takes 16 cycles, so 32 reduction values cost 96 cycles
// in this form against 256 as eight 16x16x4 fp32 MFMAs.
//
// A value beyond the largest bf16 has no such form, an infinite one least of all
// (its products are NaN whatever the sum is): a unit that met one is run again
// without pieces (wave_plain.hpp).
#pragma once

#include "common.hpp"

namespace mdl {

template <typename T>
struct Pieces {
    static constexpr int N = 1;
};
template <>
struct Pieces<float> {
    static constexpr int N = 3;
};

// Two floats of at most the largest bf16 (or NaN) to packed pieces, first value in the low halves.
__device__ __forceinline__ void split2(float a, float b, uint32_t (&p)[3]) {
    p[0] = f2bf2(a, b);
    a -= __uint_as_float(p[0] << 16);
    b -= __uint_as_float(p[0] & 0xffff0000u);
    p[1] = f2bf2(a, b);
    a -= __uint_as_float(p[1] << 16);
    b -= __uint_as_float(p[1] & 0xffff0000u);
    p[2] = f2bf2(a, b);
}

constexpr float BF16_LARGEST = 3.3895313892515355e38f;

// Eight reduction values of one operand slot as MFMA operands.
template <typename T>
__device__ __forceinline__ void make_op(const float (&v)[8], bf16x8 (&o)[Pieces<T>::N]) {
    if constexpr (Pieces<T>::N == 3) {
        uint32_t w[3][4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint32_t p[3];
            split2(v[2 * e], v[2 * e + 1], p);
#pragma unroll
            for (int k = 0; k < 3; ++k) w[k][e] = p[k];
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) o[k] = as_bf16x8(make_uint4(w[k][0], w[k][1], w[k][2], w[k][3]));
    } else {
        // the values are bf16 already: exact
        o[0] = as_bf16x8(make_uint4(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]), f2bf2(v[4], v[5]), f2bf2(v[6], v[7])));
    }
}

// acc[t] + low[t] += a[t][ks] b over one K step, for every tile t, consecutive
// MFMAs on different accumulators. The products of fp32 pieces below the
// leading one go to `low`: added there they are rounded at their own size, and
// the leading sum takes one rounding per 32 reduction values (error of the
// layer's output against 64 bits at H = 32, with the bias added afterwards:
// 1.5e-7; 1.7e-7 on the fp32 MFMA, 2.1e-7 with one accumulator from the bias).
// Types of one piece leave `low` alone.
template <int P, int TILES, int KS>
__device__ __forceinline__ void mma_tiles(const bf16x8 (&a)[TILES][KS][P], int ks, const bf16x8 (&b)[P],
                                          floatx4 (&acc)[TILES], floatx4 (&low)[TILES]) {
    if constexpr (P == 3) {
        constexpr int pa[5] = {1, 0, 2, 0, 1}, pb[5] = {1, 2, 0, 1, 0};
#pragma unroll
        for (int k = 0; k < 5; ++k)
#pragma unroll
            for (int t = 0; t < TILES; ++t) low[t] = mfma_bf16(a[t][ks][pa[k]], b[pb[k]], low[t]);
    }
#pragma unroll
    for (int t = 0; t < TILES; ++t) acc[t] = mfma_bf16(a[t][ks][0], b[0], acc[t]);
}

// Neighbouring rows of a tile sit in neighbouring lanes (16 rows per DPP row).
// Lane n takes lane n - 1's value (n + 1's), lane 0 (15) keeps `edge`.
__device__ __forceinline__ float row_above(float v, float edge) {
    return __int_as_float(
        __builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), 0x111, 0xf, 0xf, false));
}
__device__ __forceinline__ float row_below(float v, float edge) {
    return __int_as_float(
        __builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), 0x101, 0xf, 0xf, false));
}
// Rotations within the sixteen lanes: lane 0 takes lane 15's value (lane 15 lane 0's).
__device__ __forceinline__ float last_to_first(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x121, 0xf, 0xf, false));
}
__device__ __forceinline__ float first_to_last(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x12f, 0xf, 0xf, false));
}

}  // namespace mdl
