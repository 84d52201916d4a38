// What the wavefront kernels share: launch arguments, the unit queue, vector
// access to a lane's consecutive hidden units, and the store sink.
#pragma once

#include <climits>
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"
#include "split.hpp"

namespace mdl {

// W consecutive values of storage type T.
template <typename T, int W>
struct Vec;
template <>
struct Vec<float, 1> {
    using R = float;
    static __device__ __forceinline__ float get(const R& v, int) { return v; }
    static __device__ __forceinline__ R pack(const float (&v)[1]) { return v[0]; }
};
template <>
struct Vec<float, 2> {
    using R = floatx2;
    static __device__ __forceinline__ float get(const R& v, int k) { return v[k]; }
    static __device__ __forceinline__ R pack(const float (&v)[2]) { return R{v[0], v[1]}; }
};
template <>
struct Vec<float, 4> {
    using R = floatx4;
    static __device__ __forceinline__ float get(const R& v, int k) { return v[k]; }
    static __device__ __forceinline__ R pack(const float (&v)[4]) { return R{v[0], v[1], v[2], v[3]}; }
};
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
template <>
struct Vec<bf16_t, 1> {
    using R = bf16_t;
    static __device__ __forceinline__ float get(const R& v, int) { return bf2f(v); }
    static __device__ __forceinline__ R pack(const float (&v)[1]) { return f2bf(v[0]); }
};
template <>
struct Vec<bf16_t, 2> {
    using R = uint32_t;
    static __device__ __forceinline__ float get(const R& v, int k) {
        return __uint_as_float(k ? (v & 0xffff0000u) : (v << 16));
    }
    static __device__ __forceinline__ R pack(const float (&v)[2]) { return f2bf2(v[0], v[1]); }
};
template <>
struct Vec<bf16_t, 4> {
    using R = u32x2;
    static __device__ __forceinline__ float get(const R& v, int k) {
        const uint32_t w = v[k >> 1];
        return __uint_as_float((k & 1) ? (w & 0xffff0000u) : (w << 16));
    }
    static __device__ __forceinline__ R pack(const float (&v)[4]) { return R{f2bf2(v[0], v[1]), f2bf2(v[2], v[3])}; }
};
template <typename T, int W>
__device__ __forceinline__ typename Vec<T, W>::R ldw(const T* p) {
    return *reinterpret_cast<const typename Vec<T, W>::R*>(p);
}
template <typename T, int W>
__device__ __forceinline__ void stw(T* p, const float (&v)[W]) {
    *reinterpret_cast<typename Vec<T, W>::R*>(p) = Vec<T, W>::pack(v);
}

// A wavefront kernel and its workgroup size.
struct WaveKernel {
    const void* fn = nullptr;
    int threads = 0;
};

struct FwdArgs {
    const int32_t* units;  // unit = rect*4 + direction, in launch order
    const int32_t* rects;  // [n_rects][4]
    const uint8_t* mask;   // [n_cells]
    const void* u;         // [4][5H][2H]
    const void* v;         // [4][3H][2H] memory-state matrices, or NULL
    const void* wx;        // [4][5H][c_in]
    const void* b;         // [4][5H]
    const void* x;         // inputs per cell: bf16 [c_in], or the fp32 inputs as bf16 pieces [3][32 CK]
    const float* xf;       // the fp32 inputs themselves
    const int* xinf;       // per rectangle: one of its fp32 inputs has no pieces (where x is pieces)
    int c_in;
    void* z;               // [n_cells][20H]: pre-activations in where the projection ran apart; gates out
    float* c;              // [n_cells][4H] cell state
    void* y;               // [n_cells][4H] output
    int canvas_w;
    int s0, s1;            // local diagonals [s0, s1) of every unit
    unsigned* queue;       // next unit to take (zeroed before the launch), or NULL: unit = block
    int n_units;
    const StepTensors* now;  // per-diagonal launches: wx, b, x and xf are read from here
};

// The arguments of a per-diagonal launch with the tensors of this call.
__device__ __forceinline__ FwdArgs step_args(FwdArgs a) {
    using G = const __attribute__((address_space(1))) char*;  // keeps the loads global
    const StepTensors t = *a.now;
    a.wx = (const void*)(G)t.wx;
    a.b = (const void*)(G)t.b;
    a.x = (const void*)(G)t.x;
    a.xf = (const float*)(G)t.xf;
    return a;
}


struct BwdArgs {
    const int32_t* units;  // unit = rect*4 + direction, in launch order
    const int32_t* rects;  // [n_rects][4]
    const uint8_t* mask;   // [n_cells] (wide bf16 layers, plain_bwd_unit)
    const void* u;         // [4][5H][2H]
    const void* v;         // [4][3H][2H] memory-state matrices, or NULL
    void* z;               // [n_cells][20H]: gates in (other layers: a masked cell's input gates are negative), dZ out
    const float* c;        // [n_cells][4H] cell state
    const void* dy;        // [n_cells][4H] upstream gradient
    const void* wx;        // the forward's operands, for plain_bwd_unit
    const void* b;
    const float* xf;
    int c_in;
    const void* y;
    int canvas_w;
    unsigned* queue;       // next unit to take (zeroed before the launch), or NULL: unit = block
    int n_units;
};

// Target of the stores of lanes whose cell is outside the diagonal: every lane
// stores on every path, so the number of memory operations in flight is the
// same on all paths and the compiler waits for exactly the loads it needs (a
// skipped store would make it wait for everything). 1536 bytes per lane (room
// for a cell's gates of one direction), shared by workgroups eight apart;
// never read. Internal to a translation unit: one whose kernels all stage their
// rows keeps none.
constexpr int WAVE_SINK_LANE = 96;  // 16-byte slots per lane
static __device__ __attribute__((aligned(256))) uint4 g_sink[8 * 64 * WAVE_SINK_LANE];

__device__ __forceinline__ char* sink_ptr() {
    return reinterpret_cast<char*>(&g_sink[((blockIdx.x & 7) * 64 + (threadIdx.x & 63)) * WAVE_SINK_LANE]);
}

// An LDS array of a kernel, the same for every body of it (K: the kernel's
// configuration, ID: which array).
template <typename A, typename K, int ID>
__device__ __forceinline__ A& lds_array() {
    __shared__ __attribute__((aligned(16))) A a;
    return a;
}

// Runs f(integral_constant<TA>) with the number of the wave group's tiles, of
// its TPG, that hold rows of the unit's rectangle: tiles below it are not
// computed, so a short rectangle in a launch for taller ones costs its own
// tiles only (255 images of 12 rows and one of 64, training: fp32 H 32 4.1 ->
// 1.8 ms, H 64 13.0 -> 6.5, memory H 32 10.4 -> 3.5). Every body has the same
// barriers.
template <int TPG, int FIRST, typename F>
__device__ __forceinline__ void with_tiles(int n, const F& f) {
    if constexpr (TPG > FIRST) {
        if (n < TPG) return with_tiles<TPG - 1, FIRST>(n, f);
    }
    f(std::integral_constant<int, TPG>{});
}

// Units of a launch: workgroup b runs unit b, or, with a queue, a fixed number
// of workgroups per CU take units in launch order (longest first) until none
// is left; the last workgroup out zeroes the queue again.
template <typename A, typename F>
__device__ __forceinline__ void for_units(const A& a, const F& run) {
    __shared__ int slot;
    for (;;) {
        int k = (int)blockIdx.x;
        if (a.queue) {
            lds_barrier();  // the previous unit's LDS reads are done
            if (threadIdx.x == 0) slot = (int)atomicAdd(a.queue, 1u);
            lds_barrier();
            k = __builtin_amdgcn_readfirstlane(slot);
        }
        if (k >= a.n_units) break;
        run(a.units[k]);
        if (!a.queue) return;
    }
    if (threadIdx.x == 0) {
        __threadfence();
        if (atomicAdd(a.queue + 1, 1u) == gridDim.x - 1) {
            __threadfence();
            atomicExch(a.queue, 0u);
            atomicExch(a.queue + 1, 0u);
        }
    }
}

}  // namespace mdl
