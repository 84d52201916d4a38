// A unit of the fp32 wavefronts by plain FMAs over the layer's own operands.
//
// A value beyond the largest bf16 has no pieces (split.hpp), so a wavefront kernel that
// met one (an input, weight, cell state or gate gradient) runs its unit again
// here: inf * 0 and inf - inf give NaN, a sum with infinities of one sign keeps
// it. Every value passes through memory, every thread takes (cell, hidden unit)
// pairs of the diagonal; speed does not matter. Calls of their own: inlined,
// their registers change how the kernels' loops are scheduled (forward, H 16,
// 16 images of 16 rows: 203 -> 226 us).
#pragma once

#include "common.hpp"
#include "wave.hpp"

namespace mdl {

// Activations of a cell; with memory-state matrices the states feed the gates,
// and the library functions are as exact as the arithmetic around them.
template <bool MEM>
__device__ __forceinline__ float cell_sigm(float z) {
    return MEM ? 1.0f / (1.0f + __expf(-z)) : sigm_fast(z);
}
template <bool MEM>
__device__ __forceinline__ float cell_tanh(float z) {
    return MEM ? tanhf(z) : tanh_fast(z);
}

// A kernel's argument struct (its only argument) where the launch put it.
template <typename A>
using KernArgs = const __attribute__((address_space(4))) A;
template <typename A>
__device__ __forceinline__ KernArgs<A>* kern_args() {
    return (KernArgs<A>*)__builtin_amdgcn_kernarg_segment_ptr();
}

// Activated gates of hidden unit j of local cell (y, x) of a unit in direction
// d from the inputs, outputs and cell states in memory.
template <int H, bool MEM, typename A>
__device__ __forceinline__ void plain_gates(const A& a, const RectD& R, int d, int y, int x, int j, const float* Y,
                                            float (&g)[5]) {
    const float* const wx = static_cast<const float*>(a.wx) + (int64_t)d * 5 * H * a.c_in;
    const float* const u = static_cast<const float*>(a.u) + (int64_t)d * 5 * H * 2 * H;
    const float* const v = static_cast<const float*>(a.v) + (MEM ? (int64_t)d * 3 * H * 2 * H : 0);
    const float* const b = static_cast<const float*>(a.b) + d * 5 * H;
    const float* const xp = a.xf + canvas_index(R, d, y, x, a.canvas_w) * a.c_in;
#pragma unroll
    for (int t = 0; t < 5; ++t) g[t] = b[t * H + j];
#pragma clang loop unroll(disable)
    for (int k = 0; k < a.c_in; ++k)
#pragma unroll
        for (int t = 0; t < 5; ++t) g[t] = fmaf(wx[(t * H + j) * a.c_in + k], xp[k], g[t]);
#pragma clang loop unroll(disable)
    for (int side = 0; side < 2; ++side) {  // left predecessor, top predecessor
        const int py = y - side, px = x - (1 - side);
        const bool has = py >= 0 && px >= 0;
        const int64_t p = has ? canvas_index(R, d, py, px, a.canvas_w) * (4 * H) + d * H : 0;
#pragma clang loop unroll(disable)
        for (int k = 0; k < H; ++k) {
            const float h = has ? Y[p + k] : 0.0f, c = MEM && has ? a.c[p + k] : 0.0f;
#pragma unroll
            for (int t = 0; t < 5; ++t) {
                g[t] = fmaf(u[(t * H + j) * 2 * H + side * H + k], h, g[t]);
                if (MEM && t < 3) g[t] = fmaf(v[(t * H + j) * 2 * H + side * H + k], c, g[t]);
            }
        }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) g[t] = cell_sigm<MEM>(g[t]);
    g[4] = cell_tanh<MEM>(g[4]);
}

// Diagonals [sb, se) of a unit, the state of diagonal sb - 1 in memory.
template <int H, bool MEM>
__device__ __attribute__((noinline)) void plain_fwd_unit(KernArgs<FwdArgs>* args, int unit, int sb, int se) {
    FwdArgs a;
    __builtin_memcpy(&a, (const void*)args, sizeof(a));
    if (a.now) a = step_args(a);
    const int d = unit & 3;
    const RectD R = reinterpret_cast<const RectD*>(a.rects)[unit >> 2];
    float *const Z = static_cast<float*>(a.z), *const Y = static_cast<float*>(a.y);
#pragma clang loop unroll(disable)
    for (int s = sb; s < se; ++s) {
        __syncthreads();  // the previous diagonal is in memory
        const int ylo = max(0, s - R.w + 1), yhi = min(R.h - 1, s);
#pragma clang loop unroll(disable)
        for (int i = threadIdx.x; i < (yhi - ylo + 1) * H; i += blockDim.x) {
            const int y = ylo + i / H, x = s - y, j = i % H;
            const int64_t p = canvas_index(R, d, y, x, a.canvas_w);
            float g[5];
            plain_gates<H, MEM>(a, R, d, y, x, j, Y, g);
            const int64_t o = p * (4 * H) + d * H + j;
            const float cl = x > 0 ? a.c[canvas_index(R, d, y, x - 1, a.canvas_w) * (4 * H) + d * H + j] : 0.0f;
            const float ct = y > 0 ? a.c[canvas_index(R, d, y - 1, x, a.canvas_w) * (4 * H) + d * H + j] : 0.0f;
            const bool valid = a.mask[p] != 0;
            const float c = g[0] * g[4] + g[1] * cl + g[2] * ct;
            a.c[o] = valid ? c : 0.0f;
            Y[o] = valid ? g[3] * cell_tanh<MEM>(c) : 0.0f;
            if (!valid) g[0] = -1.0f;  // marks a masked cell for the backward
#pragma unroll
            for (int t = 0; t < 5; ++t) Z[p * (20 * H) + d * 5 * H + t * H + j] = g[t];
        }
    }
}


// A backward unit from its last diagonal, the gates computed again from the
// forward's outputs and cell states (the workspace may hold gate gradients in
// their place by now). pass: scratch of 4 H `rows` floats (the rectangle's rows at
// least), what a cell hands over to its predecessors' states, by diagonal
// parity, side and row.
template <int H, bool MEM>
__device__ __attribute__((noinline)) void plain_bwd_unit(KernArgs<BwdArgs>* args, int unit, float* pass, int rows) {
    BwdArgs a;
    __builtin_memcpy(&a, (const void*)args, sizeof(a));
    const int d = unit & 3;
    const RectD R = reinterpret_cast<const RectD*>(a.rects)[unit >> 2];
    float* const Z = static_cast<float*>(a.z);
    const float *const DY = static_cast<const float*>(a.dy), *const Y = static_cast<const float*>(a.y);
    const float* const U = static_cast<const float*>(a.u) + (int64_t)d * 5 * H * 2 * H;
    const float* const V = static_cast<const float*>(a.v) + (MEM ? (int64_t)d * 3 * H * 2 * H : 0);
#pragma clang loop unroll(disable)
    for (int s = R.h + R.w - 2; s >= 0; --s) {
        __syncthreads();  // the following diagonal is in memory
        const int ylo = max(0, s - R.w + 1), yhi = min(R.h - 1, s);
        float *const mine = pass + (s & 1) * 2 * rows * H, *const next = pass + ((s & 1) ^ 1) * 2 * rows * H;
#pragma clang loop unroll(disable)
        for (int i = threadIdx.x; i < (yhi - ylo + 1) * H; i += blockDim.x) {
            const int y = ylo + i / H, x = s - y, j = i % H;
            const int64_t p = canvas_index(R, d, y, x, a.canvas_w), o = p * (4 * H) + d * H + j;
            float dh = DY[o], dc = 0.0f;
#pragma clang loop unroll(disable)
            for (int side = 0; side < 2; ++side) {  // right successor, lower successor
                const int sy = y + side, sx = x + 1 - side;
                if (sy >= R.h || sx >= R.w) continue;
                const float* da = Z + canvas_index(R, d, sy, sx, a.canvas_w) * (20 * H) + d * 5 * H;
                dc += next[(side * rows + sy) * H + j];
#pragma clang loop unroll(disable)
                for (int k = 0; k < 5 * H; ++k) {
                    dh = fmaf(U[k * 2 * H + side * H + j], da[k], dh);
                    if (MEM && k < 3 * H) dc = fmaf(V[k * 2 * H + side * H + j], da[k], dc);
                }
            }
            float g[5];
            plain_gates<H, MEM>(a, R, d, y, x, j, Y, g);
            const float tc = cell_tanh<MEM>(a.c[o]);
            dc += dh * g[3] * (1.0f - tc * tc);
            const float cl = x > 0 ? a.c[canvas_index(R, d, y, x - 1, a.canvas_w) * (4 * H) + d * H + j] : 0.0f;
            const float ct = y > 0 ? a.c[canvas_index(R, d, y - 1, x, a.canvas_w) * (4 * H) + d * H + j] : 0.0f;
            const bool live = a.mask[p] != 0;
            const float da[5] = {dc * g[4] * g[0] * (1.0f - g[0]), dc * cl * g[1] * (1.0f - g[1]),
                                 dc * ct * g[2] * (1.0f - g[2]), dh * tc * g[3] * (1.0f - g[3]),
                                 dc * g[0] * (1.0f - g[4] * g[4])};
#pragma unroll
            for (int t = 0; t < 5; ++t) Z[p * (20 * H) + d * 5 * H + t * H + j] = live ? da[t] : 0.0f;
            mine[y * H + j] = live ? dc * g[1] : 0.0f;
            mine[(rows + y) * H + j] = live ? dc * g[2] : 0.0f;
        }
    }
}

}  // namespace mdl
