// Anti-diagonal wavefront recurrence of the four-direction 2D MDLSTM
// (Section III cell; Section IV-A: after input skewing every cell of an
// anti-diagonal depends only on the previous anti-diagonal; Section V: state
// from predecessors outside the cell's rectangle or with mask 0 is blocked).
//
// One workgroup runs one unit = (rectangle, scan direction) and walks its
// h + w - 1 local anti-diagonals. Cells of a diagonal are indexed by local
// row y: the left predecessor is row y of the previous diagonal, the top
// predecessor row y - 1.
//
// Here: the forward and backward of wide bf16 layers (H = 128), the layout
// pass and the launches; the other shapes are wave_fwd.hpp and wave_bwd.hpp.
#include <algorithm>
#include <climits>
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"
#include "wave_bwd.hpp"
#include "wave_fwd.hpp"

namespace mdl {

namespace {

// A-operand values of one reduction slot from global memory: element stride
// `es` between consecutive k.
template <int NSTEP>
__device__ __forceinline__ void load_slot(const bf16_t* __restrict__ base, int64_t es, bool ok,
                                          bf16x8 (&v)[NSTEP]) {
#pragma unroll
    for (int ks = 0; ks < NSTEP; ++ks) {
        uint32_t w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t lo = ok ? base[(8 * ks + 2 * e) * es] : 0;
            const uint32_t hi = ok ? base[(8 * ks + 2 * e + 1) * es] : 0;
            w[e] = lo | (hi << 16);
        }
        v[ks] = as_bf16x8(make_uint4(w[0], w[1], w[2], w[3]));
    }
}

constexpr int WIDE_WAVES = 8;  // waves per unit of the wide kernels, sixteen hidden units each (H = 128)

}  // namespace

// ---------------------------------------------------------------------------
// Forward for wide layers (bf16, H = 128: four quads per wave, where the
// staged kernel's LDS buffers do not fit and its registers spill).
//
// Lane 16q + n of wave w owns the four consecutive hidden units
// u0 = 16w + 4q .. u0 + 3 of cell n of a tile. The rows of own MFMA tile k
// are ordered (unit offset jj, gate) -> U row gate*H + 16w + 4jj + k, so the
// lane ends with the four sigmoid gates of unit u0 + k in tile k; the rows of
// the candidate tile are the wave's sixteen units in order, so its register
// k is the candidate of unit u0 + k. No value crosses lanes: the cell update
// follows each tile's MFMAs without a barrier, both neighbours' cell states
// come from LDS, and pre-activations arrive as 8-byte vectors. Tiles of a
// diagonal run one after another (the accumulators of one tile only), their
// pre-activations loaded two tiles ahead. The diagonal's gates, outputs and
// cell states are left in LDS and, after a barrier, written back by the whole
// workgroup as contiguous 16-byte chunks (a lane's own values would be
// 8-byte pieces of sixteen canvas rows per store).
// ---------------------------------------------------------------------------
template <int H, int NT, typename T>
__device__ __forceinline__ void wave_fwd_big(const FwdArgs& a, const int unit) {
    using Op = bf16x8;
    constexpr int G = 5 * H, KRUN = H / 2, NSTEP = KRUN / 8, NTH = 512;
    constexpr int ROWS = NT * 16 + 1;            // row 0: zero row above local row 0
    constexpr int HP = H + 16 / (int)sizeof(T);  // padded LDS row pitches
    constexpr int CP = H + 4;
    constexpr int GP = G + 16 / (int)sizeof(T);
    // 16-byte chunks of a cell's outputs: gates, output, cell state
    constexpr int QZ = G * (int)sizeof(T) / 16, QY = H * (int)sizeof(T) / 16, QC = H * 4 / 16;
    constexpr int QF = QZ + QY + QC, NPS = NT * 16 * QF / NTH;
    static_assert(NT * 16 * QF % NTH == 0, "store passes");
    __shared__ __attribute__((aligned(16))) T hbuf[2][ROWS][HP];
    // Cell states of the previous diagonal, overwritten row by row by the
    // current one: the tiles run from the bottom up, so a tile never
    // overwrites a row that a later tile of the diagonal still reads (a
    // lane's hidden units are its wave's columns, read before written).
    __shared__ __attribute__((aligned(16))) float cbuf[ROWS][CP];
    __shared__ __attribute__((aligned(16))) T gst[NT * 16][GP];  // activated gates of the diagonal

    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int q = lane >> 4, n16 = lane & 15;
    const int u0 = 16 * w + 4 * q;
    const int d = unit & 3;
    const RectD R = reinterpret_cast<const RectD*>(a.rects)[unit >> 2];
    const T* __restrict__ U = static_cast<const T*>(a.u) + (int64_t)d * G * 2 * H;
    T* __restrict__ Z = static_cast<T*>(a.z);
    T* __restrict__ Y = static_cast<T*>(a.y);
    float* __restrict__ Cs = a.c;
    const int steps = R.h + R.w - 1;
    const int sb = a.s0, se = min(a.s1, steps);
    if (sb >= se) return;

    for (int i = threadIdx.x; i < 2 * ROWS * HP; i += blockDim.x) (&hbuf[0][0][0])[i] = T(0);
    for (int i = threadIdx.x; i < ROWS * CP; i += blockDim.x) (&cbuf[0][0])[i] = 0.0f;
    if (sb > 0) {  // state of diagonal sb - 1 from the previous launch's outputs
        lds_barrier();  // every zero written before the read-back fills the same rows
        const int pb = (sb & 1) ^ 1;
        for (int i = threadIdx.x; i < NT * 16 * H; i += blockDim.x) {
            const int yy = i / H, j = i - yy * H, xx = sb - 1 - yy;
            if (yy < R.h && xx >= 0 && xx < R.w) {
                const int64_t p = canvas_index(R, d, yy, xx, a.canvas_w);
                hbuf[pb][yy + 1][j] = Y[p * (4 * H) + d * H + j];
                cbuf[yy + 1][j] = Cs[p * (4 * H) + d * H + j];
            }
        }
    }

    Op Aown[4][NSTEP], Ag[NSTEP];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int row = (n16 & 3) * H + 16 * w + 4 * (n16 >> 2) + k;
        load_slot<NSTEP>(U + (int64_t)row * 2 * H + q * KRUN, 1, true, Aown[k]);
    }
    load_slot<NSTEP>(U + (int64_t)(4 * H + 16 * w + n16) * 2 * H + q * KRUN, 1, true, Ag);
    __builtin_amdgcn_s_waitcnt(0);

    const DiagMap M(R, d, a.canvas_w);
    const uint8_t* mrow = a.mask + M.c0;
    const T* const zb = Z + M.c0 * (4 * G) + d * G + u0;  // the lane's pre-activations at idx = 0

    // Outputs of diagonal s, staged in LDS, written back as contiguous 16-byte
    // chunks (pass ps, thread t: chunk (ps * 512 + t) % QF of cell row slot
    // (ps * 512 + t) / QF); every thread stores in every pass (rows outside
    // the diagonal repeat its nearest cell, which writes the same bytes twice).
    char* const zd = reinterpret_cast<char*>(Z + d * G) + M.c0 * (4 * G * (int)sizeof(T));
    char* const yd = reinterpret_cast<char*>(Y + d * H) + M.c0 * (4 * H * (int)sizeof(T));
    char* const cd = reinterpret_cast<char*>(Cs + d * H) + M.c0 * (16 * H);
    auto write_back = [&](int s) {
        const int ylo = max(0, s - R.w + 1), yhi = min(R.h - 1, s);
        const int cur = s & 1, sxs = M.sx * s;
        constexpr int GR = 4;  // passes per LDS round trip (registers)
        static_assert(NPS % GR == 0, "pass groups");
#pragma unroll
        for (int p0 = 0; p0 < NPS; p0 += GR) {
            u32x4 v[GR];
#pragma unroll
            for (int k = 0; k < GR; ++k) {
                const int i = (p0 + k) * NTH + (int)threadIdx.x, r = i % QF;
                const int cell = min(max(i / QF, ylo), yhi);
                const u32x4* src = r < QZ        ? reinterpret_cast<const u32x4*>(&gst[cell][0]) + r
                                   : r < QZ + QY ? reinterpret_cast<const u32x4*>(&hbuf[cur][cell + 1][0]) + (r - QZ)
                                                 : reinterpret_cast<const u32x4*>(&cbuf[cell + 1][0]) + (r - QZ - QY);
                v[k] = *src;
            }
#pragma unroll
            for (int k = 0; k < GR; ++k) {
                const int i = (p0 + k) * NTH + (int)threadIdx.x, r = i % QF;
                const int64_t idx = sxs + min(max(i / QF, ylo), yhi) * M.ky;
                char* dst = r < QZ        ? zd + idx * (4 * G * (int)sizeof(T)) + 16 * r
                            : r < QZ + QY ? yd + idx * (4 * H * (int)sizeof(T)) + 16 * (r - QZ)
                                          : cd + idx * (16 * H) + 16 * (r - QZ - QY);
                *reinterpret_cast<u32x4*>(dst) = v[k];
            }
        }
    };

    // Pre-activations (5 gates x 4 units) and mask byte of the lane's cell of
    // tile nt of diagonal s; past the last diagonal, or for rows outside the
    // diagonal, a valid cell of the rectangle is read instead (fixed number of
    // loads on every path).
    auto load = [&](int s, int nt, uint2 (&zr)[5], uint32_t& m) {
        const int sc = min(s, se - 1);
        const int ylo = max(0, sc - R.w + 1), yhi = min(R.h - 1, sc);
        const int idx = M.sx * sc + min(max(16 * nt + n16, ylo), yhi) * M.ky;
        const T* zp = zb + (int64_t)idx * (4 * G);
#pragma unroll
        for (int t = 0; t < 5; ++t) zr[t] = *reinterpret_cast<const uint2*>(zp + t * H);
        m = mrow[idx];
    };
    // Next tile of the walk: the next active tile up the diagonal, else the
    // bottom active tile of the next one.
    auto advance = [&](int& s, int& nt) {
        const int ylo = max(0, s - R.w + 1);
        if (16 * nt > ylo) {
            --nt;
        } else {
            ++s;
            nt = min(R.h - 1, s) >> 4;
        }
    };
    auto tile = [&](int s, int nt, const uint2 (&zr)[5], uint32_t m) {
        const int cur = s & 1, prv = cur ^ 1;
        const int ylo = max(0, s - R.w + 1), yhi = min(R.h - 1, s);
        const int yy = 16 * nt + n16;
        const T* brow = (q < 2) ? &hbuf[prv][yy + 1][q * KRUN] : &hbuf[prv][yy][(q - 2) * KRUN];
        floatx4 acc[4], ag = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < NSTEP; ++ks) {
            const Op b = as_bf16x8(*reinterpret_cast<const uint4*>(brow + ks * 8));
            ag = mfma_bf16(Ag[ks], b, ag);
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[k] = mfma_bf16(Aown[k][ks], b, acc[k]);
        }
        const float4 cl = *reinterpret_cast<const float4*>(&cbuf[yy + 1][u0]);
        const float4 ct = *reinterpret_cast<const float4*>(&cbuf[yy][u0]);
        const float clv[4] = {cl.x, cl.y, cl.z, cl.w}, ctv[4] = {ct.x, ct.y, ct.z, ct.w};
        const bool live = yy >= ylo && yy <= yhi && m != 0;
        float gv[5][4], hv[4], cv[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float zv[5];
#pragma unroll
            for (int t = 0; t < 5; ++t) {
                const uint32_t wd = (k < 2) ? zr[t].x : zr[t].y;
                zv[t] = __uint_as_float((k & 1) ? (wd & 0xffff0000u) : (wd << 16));
            }
            gv[0][k] = sigm_fast(acc[k][0] + zv[0]);
            gv[1][k] = sigm_fast(acc[k][1] + zv[1]);
            gv[2][k] = sigm_fast(acc[k][2] + zv[2]);
            gv[3][k] = sigm_fast(acc[k][3] + zv[3]);
            gv[4][k] = tanh_fast(ag[k] + zv[4]);
            const float cn = gv[0][k] * gv[4][k] + gv[1][k] * clv[k] + gv[2][k] * ctv[k];
            const float hn = gv[3][k] * tanh_fast(cn);
            cv[k] = live ? cn : 0.0f;
            hv[k] = live ? hn : 0.0f;
        }
        auto pack = [](const float (&v)[4]) {
            return make_uint2(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]));
        };
        *reinterpret_cast<uint2*>(&hbuf[cur][yy + 1][u0]) = pack(hv);
        *reinterpret_cast<float4*>(&cbuf[yy + 1][u0]) = make_float4(cv[0], cv[1], cv[2], cv[3]);
#pragma unroll
        for (int t = 0; t < 5; ++t) *reinterpret_cast<uint2*>(&gst[yy][t * H + u0]) = pack(gv[t]);
        if (16 * nt <= ylo) {  // top tile of the diagonal: publish it, write it back
            lds_barrier();
            write_back(s);
            lds_barrier();
        }
    };

    lds_barrier();
    uint2 z0[5], z1[5];
    uint32_t m0, m1;
    int s = sb, nt = min(R.h - 1, sb) >> 4;
    int ls = s, lnt = nt;
    load(ls, lnt, z0, m0);
    advance(ls, lnt);
    load(ls, lnt, z1, m1);
    advance(ls, lnt);
    for (;;) {
        tile(s, nt, z0, m0);
        load(ls, lnt, z0, m0);
        advance(ls, lnt);
        advance(s, nt);
        if (s >= se) break;
        tile(s, nt, z1, m1);
        load(ls, lnt, z1, m1);
        advance(ls, lnt);
        advance(s, nt);
        if (s >= se) break;
    }
}

// ---------------------------------------------------------------------------
// Backward for wide layers (bf16, H = 128), with the forward's lane mapping:
// lane 16q + n of wave w owns units u0 = 16w + 4q .. u0 + 3 of cell n of a
// tile. The wave computes the two U^T da output tiles of its own units, the
// left-predecessor part (rows u0 + r) and the top-predecessor part
// (rows H + u0 + r), so the left part lands in the lane that needs it on the
// next diagonal (the cell's left predecessor is on the same row) and stays in
// registers; the top part and dc f_T go one row up through LDS, within the
// wave. Only the gate gradients cross waves (all of them are the reduction
// operand), so a diagonal runs as segments [A(t0)] [B(t0) A(t1)] ... [B(t1)]
// with a barrier after each: A = gate-gradient update of a tile, B = its
// U^T da products on MFMA.
// ---------------------------------------------------------------------------
template <int H, int NT, typename T>
__device__ __forceinline__ void wave_bwd_big(const BwdArgs& a, const int unit) {
    using Op = bf16x8;
    constexpr int G = 5 * H, KRUNB = G / 4, NSTEPB = KRUNB / 8;
    constexpr int GP = G + 16 / (int)sizeof(T);  // padded LDS row pitches
    constexpr int CP = H + 4;
    __shared__ __attribute__((aligned(16))) T dabuf[NT * 16][GP];
    // per cell row: the top-predecessor part of U^T da, and dc f_T (row NT*16 stays zero)
    __shared__ __attribute__((aligned(16))) float gtop[NT * 16 + 1][CP];
    __shared__ __attribute__((aligned(16))) float dct[NT * 16 + 1][CP];

    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int q = lane >> 4, n16 = lane & 15;
    const int u0 = 16 * w + 4 * q;
    const int d = unit & 3;
    const RectD R = reinterpret_cast<const RectD*>(a.rects)[unit >> 2];
    const T* __restrict__ U = static_cast<const T*>(a.u) + (int64_t)d * G * 2 * H;
    T* __restrict__ Z = static_cast<T*>(a.z);
    const T* __restrict__ DY = static_cast<const T*>(a.dy);
    const float* __restrict__ Cs = a.c;
    const int steps = R.h + R.w - 1;

    for (int i = threadIdx.x; i < NT * 16 * GP; i += blockDim.x) (&dabuf[0][0])[i] = T(0);
    for (int i = threadIdx.x; i < (NT * 16 + 1) * CP; i += blockDim.x) {
        (&gtop[0][0])[i] = 0.0f;
        (&dct[0][0])[i] = 0.0f;
    }
    // A operands: U^T rows k = u-part + 16w + n16 (column k of U); slot q
    // holds gate rows q*KRUNB + 8 ks + e.
    Op A[2][NSTEPB];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
        load_slot<NSTEPB>(U + (int64_t)(q * KRUNB) * 2 * H + tt * H + 16 * w + n16, 2 * H, true, A[tt]);
    floatx4 gl[NT], dcl[NT];  // left-successor parts of dh and dc, per tile row
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) gl[nt] = dcl[nt] = floatx4{0.f, 0.f, 0.f, 0.f};
    __builtin_amdgcn_s_waitcnt(0);

    const DiagMap M(R, d, a.canvas_w);
    const uint8_t* mrow = a.mask + M.c0;
    T* const zb = Z + M.c0 * (4 * G) + d * G + u0;
    const T* const dyb = DY + M.c0 * (4 * H) + d * H + u0;
    const float* const cb = Cs + M.c0 * (4 * H) + d * H + u0;

    struct In {
        uint2 g[5], dy;
        float4 c, cl, ct;
        uint32_t m;
    };
    // Inputs of the lane's cell of tile nt of diagonal s (rows outside the
    // diagonal read its nearest cell; a missing predecessor reads the cell).
    auto load = [&](int s, int nt, In& in) {
        const int ylo = max(0, s - R.w + 1), yhi = min(R.h - 1, s);
        const int yc = min(max(16 * nt + n16, ylo), yhi), xc = s - yc;
        const int idx = M.sx * s + yc * M.ky;
        const int il = xc > 0 ? idx - M.sx : idx;
        const int it = yc > 0 ? idx - M.sx - M.ky : idx;
        const T* zp = zb + (int64_t)idx * (4 * G);
#pragma unroll
        for (int t = 0; t < 5; ++t) in.g[t] = *reinterpret_cast<const uint2*>(zp + t * H);
        in.dy = *reinterpret_cast<const uint2*>(dyb + (int64_t)idx * (4 * H));
        in.c = *reinterpret_cast<const float4*>(cb + (int64_t)idx * (4 * H));
        in.cl = *reinterpret_cast<const float4*>(cb + (int64_t)il * (4 * H));
        in.ct = *reinterpret_cast<const float4*>(cb + (int64_t)it * (4 * H));
        in.m = mrow[idx];
    };
    auto bf = [](const uint2& v, int k) {
        const uint32_t wd = (k < 2) ? v.x : v.y;
        return __uint_as_float((k & 1) ? (wd & 0xffff0000u) : (wd << 16));
    };
    auto pack = [](const float (&v)[4]) {
        return make_uint2(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]));
    };
    // Phase A of tile nt: gate gradients of the lane's four units.
    auto phase_a = [&](int s, int nt, const In& in) {
        const int ylo = max(0, s - R.w + 1), yhi = min(R.h - 1, s);
        const int yy = 16 * nt + n16;
        const bool inr = yy >= ylo && yy <= yhi;
        const bool live = inr && in.m != 0;
        const bool hasl = s - yy > 0, hast = yy > 0;
        const float4 gt4 = *reinterpret_cast<const float4*>(&gtop[yy + 1][u0]);
        const float4 dt4 = *reinterpret_cast<const float4*>(&dct[yy + 1][u0]);
        const float gtv[4] = {gt4.x, gt4.y, gt4.z, gt4.w}, dtv[4] = {dt4.x, dt4.y, dt4.z, dt4.w};
        const float cv4[4] = {in.c.x, in.c.y, in.c.z, in.c.w};
        const float cl4[4] = {in.cl.x, in.cl.y, in.cl.z, in.cl.w};
        const float ct4[4] = {in.ct.x, in.ct.y, in.ct.z, in.ct.w};
        float da[5][4], ndl[4], ndt[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float gi = bf(in.g[0], k), gfl = bf(in.g[1], k), gft = bf(in.g[2], k), go = bf(in.g[3], k),
                        gg = bf(in.g[4], k);
            const float cL = hasl ? cl4[k] : 0.0f, cT = hast ? ct4[k] : 0.0f;
            const float dh = bf(in.dy, k) + gl[nt][k] + gtv[k];
            const float tc = tanh_fast(cv4[k]);
            const float dc = dcl[nt][k] + dtv[k] + dh * go * (1.0f - tc * tc);
            da[0][k] = live ? dc * gg * gi * (1.0f - gi) : 0.0f;
            da[1][k] = live ? dc * cL * gfl * (1.0f - gfl) : 0.0f;
            da[2][k] = live ? dc * cT * gft * (1.0f - gft) : 0.0f;
            da[3][k] = live ? dh * tc * go * (1.0f - go) : 0.0f;
            da[4][k] = live ? dc * gi * (1.0f - gg * gg) : 0.0f;
            ndl[k] = live ? dc * gfl : 0.0f;
            ndt[k] = live ? dc * gft : 0.0f;
        }
        dcl[nt] = floatx4{ndl[0], ndl[1], ndl[2], ndl[3]};
        *reinterpret_cast<float4*>(&dct[yy][u0]) = make_float4(ndt[0], ndt[1], ndt[2], ndt[3]);
#pragma unroll
        for (int t = 0; t < 5; ++t) *reinterpret_cast<uint2*>(&dabuf[yy][t * H + u0]) = pack(da[t]);
        {
            T* const zp = inr ? zb + (int64_t)(M.sx * s + yy * M.ky) * (4 * G) : reinterpret_cast<T*>(sink_ptr());
#pragma unroll
            for (int t = 0; t < 5; ++t) *reinterpret_cast<uint2*>(zp + t * H) = pack(da[t]);
        }
    };
    // Phase B of tile nt: U^T da of its cells for the wave's units.
    auto phase_b = [&](int nt) {
        const T* brow = &dabuf[16 * nt + n16][q * KRUNB];
        floatx4 al = floatx4{0.f, 0.f, 0.f, 0.f}, at = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < NSTEPB; ++ks) {
            const Op b = as_bf16x8(*reinterpret_cast<const uint4*>(brow + ks * 8));
            al = mfma_bf16(A[0][ks], b, al);
            at = mfma_bf16(A[1][ks], b, at);
        }
        gl[nt] = al;
        *reinterpret_cast<float4*>(&gtop[16 * nt + n16][u0]) = make_float4(at[0], at[1], at[2], at[3]);
    };

    // The inputs of the next tile's phase A are loaded right after the
    // current one (one register set), so they are in flight across the
    // barrier and the next segment's MFMAs.
    In in;
    load(steps - 1, max(0, steps - R.w) >> 4, in);
    lds_barrier();
    for (int s = steps - 1; s >= 0; --s) {
        const int ylo = max(0, s - R.w + 1), yhi = min(R.h - 1, s);
        const int t0 = ylo >> 4, t1 = yhi >> 4;
#pragma unroll
        for (int k = 0; k <= NT; ++k) {
            const bool pa = k < NT && k >= t0 && k <= t1;      // A(k) in this segment
            const bool pb = k >= 1 && k - 1 >= t0 && k - 1 <= t1;  // B(k - 1) in this segment
            if (pb) phase_b(k - 1);
            if (pa) {
                phase_a(s, k, in);
                if (k < t1) load(s, k + 1, in);
                else load(max(s - 1, 0), max(0, s - R.w) >> 4, in);  // first tile of the next diagonal
            }
            if (pa || pb) lds_barrier();
        }
    }
}

// ---------------------------------------------------------------------------
// Kernels. With a queue, a fixed number of workgroups per CU take units in
// launch order (longest first) from a counter until none is left, so a long
// unit shares its CU with fewer others than when every unit has its own
// workgroup from the start; without one, workgroup b runs unit b.
// ---------------------------------------------------------------------------
// One unit per workgroup where the units are at most one per CU (forward) or two
// (backward): the loop over the queue costs registers (forward, three tiles: 9
// spilled against none, 256 units of 48 rows 4565 against 4422 us; backward
// sixteen more spilled, 512 units 22.5 against 21.7 ms).
template <int H, int NT, typename T, bool QUEUE>
__global__ void __launch_bounds__((64 * WIDE_WAVES)) k_wave_fwd(FwdArgs a) {
    if constexpr (QUEUE) for_units(a, [&](int unit) { wave_fwd_big<H, NT, T>(a, unit); });
    else wave_fwd_big<H, NT, T>(a, a.units[blockIdx.x]);
}

template <int H, int NT, typename T, bool QUEUE>
__global__ void __launch_bounds__((64 * WIDE_WAVES)) k_wave_bwd(BwdArgs a) {
    if constexpr (QUEUE) for_units(a, [&](int unit) { wave_bwd_big<H, NT, T>(a, unit); });
    else wave_bwd_big<H, NT, T>(a, a.units[blockIdx.x]);
}

template <bool QUEUE>
static WaveKernel wide_fwd_kernel(int nt) {
    constexpr int th = 64 * WIDE_WAVES;
    switch (nt) {
        case 1: return {reinterpret_cast<const void*>(&k_wave_fwd<128, 1, bf16_t, QUEUE>), th};
        case 2: return {reinterpret_cast<const void*>(&k_wave_fwd<128, 2, bf16_t, QUEUE>), th};
        case 3: return {reinterpret_cast<const void*>(&k_wave_fwd<128, 3, bf16_t, QUEUE>), th};
        case 4: return {reinterpret_cast<const void*>(&k_wave_fwd<128, 4, bf16_t, QUEUE>), th};
        default: return {};
    }
}

template <bool QUEUE>
static WaveKernel wide_bwd_kernel(int nt) {
    constexpr int th = 64 * WIDE_WAVES;
    switch (nt) {
        case 1: return {reinterpret_cast<const void*>(&k_wave_bwd<128, 1, bf16_t, QUEUE>), th};
        case 2: return {reinterpret_cast<const void*>(&k_wave_bwd<128, 2, bf16_t, QUEUE>), th};
        case 3: return {reinterpret_cast<const void*>(&k_wave_bwd<128, 3, bf16_t, QUEUE>), th};
        case 4: return {reinterpret_cast<const void*>(&k_wave_bwd<128, 4, bf16_t, QUEUE>), th};
        default: return {};
    }
}

// ---------------------------------------------------------------------------
// Dispatch over hidden size, tiles per diagonal and storage type.
// ---------------------------------------------------------------------------
// The forward kernel of a shape. bf16 H = 128 has its own kernel: its operands
// alone take 160 registers a lane at eight waves (here the one without a queue).
static WaveKernel fwd_kernel_of(const LayerGeom& g, int nt, bool memory, bool one_step) {
    const int ck = fwd_fused_steps(g);
    if (memory)
        return g.dtype != 0      ? WaveKernel{}
               : g.hidden == 16 ? fwd_kernel_mem_h16(nt, ck)
               : g.hidden == 32 ? fwd_kernel_mem_h32(nt, ck)
                                 : WaveKernel{};
    if (g.dtype == 0) {
        switch (g.hidden) {
            case 4: return fwd_kernel_f32_h4(nt, ck, one_step);
            case 8: return fwd_kernel_f32_h8(nt, ck, one_step);
            case 16: return fwd_kernel_f32_h16(nt, ck, one_step);
            case 32: return fwd_kernel_f32_h32(nt, ck, one_step);
            case 64: return fwd_kernel_f32_h64(nt, ck, one_step);
            default: return {};
        }
    }
    switch (g.hidden) {
        case 32: return fwd_kernel_bf16_h32(nt, ck, one_step);
        case 64: return fwd_kernel_bf16_h64(nt, ck, one_step);
        case 128: return wide_fwd_kernel<false>(nt);
        default: return {};
    }
}

// K steps of 32 input channels that the forward wavefront takes over from the
// projection (0: the projection runs apart).
int fwd_fused_steps(const LayerGeom& g) {
    if (g.c_in > 64 || !(g.dtype == 0 ? fwd_fusable<float>(g.hidden) : fwd_fusable<bf16_t>(g.hidden))) return 0;
    return (g.c_in + 31) / 32;
}

size_t fwd_x_bytes(const LayerGeom& g) {
    return g.dtype == 0 ? (size_t)g.n_cells * (fwd_fused_steps(g) * 32 * 3 * 2 + 16) : 0;
}

// What a forward pass needs before its wavefront, in one launch: the rectangle
// id of every cell (-1 outside), the unit queue's counters at zero, zero
// output rows of the invalid cells, and the fp32 inputs of the rectangles'
// cells as the wavefront reads them: three bf16 pieces, channels padded with
// zeros to 32 CK, then 16 bytes whose first word says whether the cell is
// valid; a rectangle with an input beyond the largest bf16 in a valid cell is flagged. A workgroup takes 256 cells; it first lists the rectangles that meet
// them (rectangles are disjoint, so the list's order does not matter). Four
// launches before (id fill, painting, pieces, zeroing): two small images 678 ->
// 655 us through the three layers, word batch step 545 -> 528 us.
constexpr int LAYOUT_LIST = 512;
__global__ void __launch_bounds__(256)
k_forward_layout(int n, const RectD* __restrict__ rects, int canvas_w, int64_t n_cells, int32_t* rid,
                 const uint8_t* __restrict__ mask, unsigned* __restrict__ queue, uint2* __restrict__ y, int yrow_words,
                 int c, int cp, const float* __restrict__ x, bf16_t* __restrict__ xs, int* __restrict__ xinf) {
    __shared__ int list[LAYOUT_LIST];
    __shared__ RectD listed[LAYOUT_LIST];
    __shared__ int count;
    __shared__ int ids[256];
    const int tid = threadIdx.x;
    if (blockIdx.x == 0 && tid < 2) queue[tid] = 0u;
    for (int64_t c0 = (int64_t)blockIdx.x * 256; c0 < n_cells; c0 += (int64_t)gridDim.x * 256) {
        const int64_t cl = min(c0 + 255, n_cells - 1);
        const int ya = (int)(c0 / canvas_w), yb = (int)(cl / canvas_w);
        const int xa = ya == yb ? (int)(c0 - (int64_t)ya * canvas_w) : 0;
        const int xb = ya == yb ? (int)(cl - (int64_t)yb * canvas_w) : canvas_w - 1;
        __syncthreads();  // the previous block's ids and list are read
        if (tid == 0) count = 0;
        __syncthreads();
        for (int k = tid; k < n; k += 256) {  // n < 0: rid holds the ids already
            const RectD r = rects[k];
            if (r.y0 <= yb && r.y0 + r.h > ya && r.x0 <= xb && r.x0 + r.w > xa) {
                const int at = atomicAdd(&count, 1);
                if (at < LAYOUT_LIST) {
                    list[at] = k;
                    listed[at] = r;
                }
            }
        }
        __syncthreads();
        const int64_t p = c0 + tid;
        int id = -1;
        if (p < n_cells && n < 0) {
            id = rid[p];
        } else if (p < n_cells) {
            const int py = (int)(p / canvas_w), px = (int)(p - (int64_t)py * canvas_w);
            const bool whole = count <= LAYOUT_LIST;  // else the list is cut: look at every rectangle
            const int m = whole ? count : n;
            for (int i = 0; i < m; ++i) {
                const int k = whole ? list[i] : i;
                const RectD r = whole ? listed[i] : rects[k];
                if (py >= r.y0 && py < r.y0 + r.h && px >= r.x0 && px < r.x0 + r.w) id = k;
            }
            rid[p] = id;
        }
        const bool valid = id >= 0 && mask[p] != 0;
        ids[tid] = id < 0 ? -1 : valid;
        const int lane = tid & 63;
        for (uint64_t bm = __ballot(p < n_cells && !valid); bm; bm &= bm - 1) {
            uint2* row = y + (c0 + (tid & ~63) + __builtin_ctzll(bm)) * yrow_words;
            for (int k = lane; k < yrow_words; k += 64) row[k] = make_uint2(0u, 0u);
        }
        if (xs) {
            __syncthreads();
            const int per = cp / 8 + 1, row = 3 * cp + 8;
            for (int i = tid; i < 256 * per; i += 256) {
                const int cell = i / per, k = (i - cell * per) * 8;
                const int64_t pc = c0 + cell;
                if (pc >= n_cells || ids[cell] < 0) continue;
                if (k == cp) {
                    *reinterpret_cast<uint4*>(xs + pc * row + 3 * cp) = make_uint4(ids[cell], 0, 0, 0);
                    continue;
                }
                const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
                const floatx4 v0 = k < c ? St<float>::ld4(x + pc * c + k) : zero;
                const floatx4 v1 = k + 4 < c ? St<float>::ld4(x + pc * c + k + 4) : zero;
                const float v[8] = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
                float m = 0.0f;
#pragma unroll
                for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf(v[e]));
                if (m > BF16_LARGEST && ids[cell] > 0) atomicOr(&xinf[rid[pc]], 1);
                bf16x8 o[3];
                make_op<float>(v, o);
#pragma unroll
                for (int e = 0; e < 3; ++e) *reinterpret_cast<bf16x8*>(xs + pc * row + e * cp + k) = o[e];
            }
        }
    }
}

hipError_t launch_forward_layout(const LayerGeom& g, int n, const int32_t* d_rects, int32_t* d_rid,
                                 const uint8_t* d_mask, unsigned* d_queue, void* d_y, const void* d_x, void* d_xs,
                                 int* d_xinf, hipStream_t s) {
    const int cp = g.dtype == 0 ? 32 * fwd_fused_steps(g) : 0;
    const int yrow_words = 4 * g.hidden * (g.dtype == 1 ? 2 : 4) / 8;
    const int64_t blocks = std::min<int64_t>((g.n_cells + 255) / 256, 1 << 20);
    hipLaunchKernelGGL(k_forward_layout, dim3((unsigned)blocks), dim3(256), 0, s, n,
                       reinterpret_cast<const RectD*>(d_rects), g.canvas_w, g.n_cells, d_rid, d_mask, d_queue,
                       static_cast<uint2*>(d_y), yrow_words, g.c_in, cp, static_cast<const float*>(d_x),
                       static_cast<bf16_t*>(cp > 0 ? d_xs : nullptr), d_xinf);
    return hipGetLastError();
}

// Workgroups of a kernel that the device holds at once (256 CUs assumed when the
// query fails), two waves per SIMD at most: a third reads and writes more than
// the memory takes (word batch backward, fp32 H 16: 396 us with three, 355 with
// two; 128 images of 32 rows, bf16 H 32: 1314 and 1249).
static int resident_groups(const WaveKernel& k) {
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) {
        (void)hipGetLastError();
        cus = 256;
    }
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k.fn, k.threads, 0) != hipSuccess || per < 1) {
        (void)hipGetLastError();
        per = 1;
    }
    return cus * std::min(per, std::max(1, 512 / k.threads));
}

hipError_t launch_wavefront_fwd(const LayerGeom& g, int nt, int n_units, const int32_t* d_units,
                                const int32_t* d_rects, const uint8_t* d_mask, const FwdTensors& t, unsigned* d_queue,
                                hipStream_t s) {
    if (n_units == 0) return hipSuccess;
    WaveKernel k = fwd_kernel_of(g, nt, t.v != nullptr, false);
    if (!k.fn) return hipErrorInvalidValue;
    const int groups = resident_groups(k);
    if (g.dtype == 1 && g.hidden == 128 && n_units > groups) k = wide_fwd_kernel<true>(nt);
    FwdArgs a{d_units, d_rects, d_mask, t.u, t.v, t.wx, t.b, t.x, t.xf, t.xinf, g.c_in, t.z, t.c, t.y, g.canvas_w, 0,
              INT_MAX, n_units > groups ? d_queue : nullptr, n_units, nullptr};
    void* params[] = {&a};
    return hipLaunchKernel(k.fn, dim3(std::min(n_units, groups)), dim3(k.threads), params, 0, s);
}

// The backward kernel of a shape (bf16 H = 128 as in the forward).
static WaveKernel bwd_kernel_of(const LayerGeom& g, int nt, bool memory) {
    if (memory)
        return g.dtype != 0      ? WaveKernel{}
               : g.hidden == 16 ? bwd_kernel_mem_h16(nt)
               : g.hidden == 32 ? bwd_kernel_mem_h32(nt)
                                 : WaveKernel{};
    if (g.dtype == 0) {
        switch (g.hidden) {
            case 4: return bwd_kernel_f32_h4(nt);
            case 8: return bwd_kernel_f32_h8(nt);
            case 16: return bwd_kernel_f32_h16(nt);
            case 32: return bwd_kernel_f32_h32(nt);
            case 64: return bwd_kernel_f32_h64(nt);
            default: return {};
        }
    }
    switch (g.hidden) {
        case 32: return bwd_kernel_bf16_h32(nt);
        case 64: return bwd_kernel_bf16_h64(nt);
        case 128: return wide_bwd_kernel<true>(nt);
        default: return {};
    }
}

hipError_t launch_wavefront_bwd(const LayerGeom& g, int nt, int n_units, const int32_t* d_units,
                                const int32_t* d_rects, const uint8_t* d_mask, const BwdTensors& t, unsigned* d_queue,
                                hipStream_t s) {
    if (n_units == 0) return hipSuccess;
    WaveKernel k = bwd_kernel_of(g, nt, t.v != nullptr);
    if (!k.fn) return hipErrorInvalidValue;
    int groups = resident_groups(k);
    if (g.dtype == 1 && g.hidden == 128 && n_units <= 2 * groups) {  // one workgroup per CU is resident
        k = wide_bwd_kernel<false>(nt);
        groups = n_units;
    }
    const float* xf = g.dtype == 0 ? static_cast<const float*>(t.x) : nullptr;
    BwdArgs a{d_units, d_rects, d_mask, t.u, t.v, t.z, t.c, t.dy, t.wx, t.b, xf, g.c_in, t.y, g.canvas_w,
              n_units > groups ? d_queue : nullptr, n_units};
    void* params[] = {&a};
    return hipLaunchKernel(k.fn, dim3(std::min(n_units, groups)), dim3(k.threads), params, 0, s);
}

hipError_t build_wavefront_fwd_graph(const LayerGeom& g, int nt, int n_units, int max_steps, const int32_t* d_units,
                                     const int32_t* d_rects, const uint8_t* d_mask, const FwdTensors& t,
                                     const StepTensors* d_now, hipGraphExec_t* exec) {
    if (n_units <= 0 || max_steps <= 0) return hipErrorInvalidValue;
    const WaveKernel k = fwd_kernel_of(g, nt, false, true);
    if (!k.fn) return hipErrorInvalidValue;
    hipGraph_t graph;
    hipError_t e = hipGraphCreate(&graph, 0);
    if (e != hipSuccess) return e;
    hipGraphNode_t prev = nullptr;
    for (int st = 0; st < max_steps && e == hipSuccess; ++st) {
        FwdArgs a{d_units, d_rects, d_mask, t.u, t.v,        t.wx, t.b,    t.x,     t.xf, t.xinf, g.c_in,
                  t.z,     t.c,     t.y,    g.canvas_w, st, st + 1, nullptr, n_units, d_now};
        void* params[] = {&a};
        hipKernelNodeParams p{};
        p.func = const_cast<void*>(k.fn);
        p.gridDim = dim3(n_units);
        p.blockDim = dim3(k.threads);
        p.sharedMemBytes = 0;
        p.kernelParams = params;
        p.extra = nullptr;
        hipGraphNode_t node;
        e = hipGraphAddKernelNode(&node, graph, prev ? &prev : nullptr, prev ? 1 : 0, &p);
        prev = node;
    }
    if (e == hipSuccess) e = hipGraphInstantiate(exec, graph, nullptr, nullptr, 0);
    const hipError_t e2 = hipGraphDestroy(graph);
    return e != hipSuccess ? e : e2;
}

}  // namespace mdl
