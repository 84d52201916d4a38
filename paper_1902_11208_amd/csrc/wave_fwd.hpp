// Forward anti-diagonal wavefront of the four-direction 2D MDLSTM (Section III
// cell; Section IV-A: after input skewing every cell of an anti-diagonal
// depends only on the previous one; Section V: state from predecessors
// outside the cell's rectangle or with mask 0 is blocked).
//
// One workgroup runs one unit = (rectangle, scan direction) and walks its
// h + w - 1 local anti-diagonals; the cell of row y has its left predecessor
// on row y of the previous diagonal and its top predecessor on row y - 1.
//
// A wave owns 4 WQ hidden units of one or more 16-row tiles. All five gates
// of a hidden unit and cell end in one lane, so no pre-activation crosses
// lanes: lane 16q + n holds units 4 WQ w + WQ q + r, r < WQ, of row n. Per K
// step the wave runs WQ + 1 MFMA tiles: tile r < WQ has A rows (unit q, gate)
// for the four sigmoid gates of the lanes' unit r, the last tile has A rows
// (unit q, r) for the candidates of all of them (rows r >= WQ are zero). The
// reduction runs over [x | h_L | h_T]: the input part (bias, Wx x) of the
// next diagonal is computed behind the cell update of the current one, where
// it does not wait for anybody, so the projection needs no pass of its own.
// The A operands stay in registers for the whole unit.
//
// Between diagonals only h crosses waves, through LDS as ready operand rows
// [h_L | h_T] (each h is written twice: as its row's left and as the next
// row's top predecessor), double-buffered by diagonal parity: one barrier per
// diagonal. The top predecessor's cell state is the neighbouring lane's of
// the previous diagonal (a DPP move; rows 15 -> 16 through a rotation or LDS).
//
// fp32 operands are three bf16 pieces each (split.hpp).
//
// What bounds it: a diagonal's latency where units are few (MFMAs block the
// issue of their wave, so MFMA and cell update of a wave add up; those of the
// two waves of a SIMD overlap), memory traffic where they fill the chip.
// Measured, projection included, before (fp32 MFMA, candidate partials through
// LDS, two barriers, separate projection) and after:
//   fp32 H 32, one 31 x 777 line      1753 -> 1172 us (1.45 us a diagonal)
//   fp32 H 32, 64 lines of 32 rows    2270 -> 1175 us (3.63 GB, 3.1 TB/s)
//   fp32 H 16, 32 images of 32 rows    601 ->  388 us
//   fp32 H 16, 256 words               305 ->  174 us
//   bf16 H 64, 24 lines of 20-60 rows 14.2 ->  2.7 ms
#pragma once

#include <type_traits>

#include "kernels.hpp"
#include "wave.hpp"
#include "wave_plain.hpp"

namespace mdl {

template <int H, int NT, typename T, int CK, int WQ, int NG, bool MEM>
struct FwdK {
    static constexpr int P = Pieces<T>::N;
    static constexpr int UW = 4 * WQ, NWU = H / UW;     // hidden units per wave, waves per tile group
    static constexpr int TPG = NT / NG;                 // tiles per wave (group tg: tiles tg TPG ...)
    static constexpr int NTH = 64 * NWU * NG;
    static constexpr int KS = (2 * H + 31) / 32;        // K steps over [h_L | h_T]
    static constexpr int KP = 32 * KS + 8;              // operand row pitch: 16-byte reads of 16 rows hit distinct banks
    static constexpr int TILES = WQ + 1;
    // Registers per lane: up to 256, in which MFMA results need no moves from
    // accumulation registers, unless the operands alone take more.
    static constexpr int WPE = (TILES * (KS + CK) + (MEM ? WQ * KS : 0)) * P * 4 > 170 ? 1 : 2;
    // Inputs of a cell in 16-byte chunks: the x operands (fp32: pieces and a
    // validity chunk, as launch_forward_layout lays them out) or the pre-activations.
    static constexpr int QI = CK > 0 ? 4 * CK * P + (P == 3 ? 1 : 0) : 5 * H * (int)sizeof(T) / 16;
    static constexpr int PI = CK > 0 && P == 3 ? QI : QI + 1;  // LDS pitch, odd: rows in different banks
    // Outputs: the 5H activated gates, then the H outputs (storage type), then the H cell states (fp32).
    static constexpr int QZ = 5 * H * (int)sizeof(T) / 16, QY = H * (int)sizeof(T) / 16, QC = H / 4;
    static constexpr int QF = QZ + QY + QC;
    static constexpr int PF = QF + 1;
    static constexpr size_t HOP = (size_t)2 * (MEM ? 2 : 1) * P * (NT * 16 + 1) * KP * 2;
    static constexpr size_t IN1 = (size_t)NT * 16 * PI * 16, OUT1 = (size_t)NT * 16 * PF * 16;
    static constexpr size_t LIM = 156 * 1024;
    // Both pass through LDS where they fit: a lane's own values are pieces of
    // sixteen canvas rows per load or store, which the memory pipe takes one
    // lane per cycle (64 cycles an instruction; measured, 2.3 us a diagonal at
    // H = 32 and two tiles), whole rows in chunks go sixteen lanes per cycle.
    static constexpr bool STAGE_IN = NTH >= QI && HOP + 2 * IN1 <= LIM;
    static constexpr size_t BASE = HOP + (STAGE_IN ? 2 * IN1 : 0);
    // Output buffers: two by diagonal parity, or one and a second barrier.
    static constexpr int OBUF = NTH < QF ? 0 : BASE + 2 * OUT1 <= LIM ? 2 : (BASE + OUT1 <= LIM ? 1 : 0);
    static_assert(H % UW == 0 && NT % NG == 0 && NTH <= 1024, "wave split");
};

// TA: the group's tiles that hold rows of the rectangle.
// STEP: one diagonal per launch, [a.s0, a.s0 + 1), with the state of the one
// before read back from the outputs and cell states. Its loads are all on their
// way before the first wait, nothing is loaded ahead or left for a next diagonal
// (line batch, 621 launches: 7.6 -> 6.9 ms).
template <int H, int NT, typename T, int CK, int WQ, int NG, bool MEM, int TA, bool STEP>
__device__ __forceinline__ void fwd_unit(const FwdArgs& a, const int unit) {
    using K = FwdK<H, NT, T, CK, WQ, NG, MEM>;
    constexpr int P = K::P, NWU = K::NWU, TPG = K::TPG, KS = K::KS, KP = K::KP, TILES = K::TILES, NTH = K::NTH;
    constexpr bool STAGE_IN = K::STAGE_IN, STAGE_OUT = K::OBUF > 0;
    constexpr int OBUF = K::OBUF, PI = K::PI, QI = K::QI, PF = K::PF, QF = K::QF, QZ = K::QZ, QY = K::QY;
    constexpr int G = 5 * H, ROWS = NT * 16 + 1, CP = 32 * CK;
    constexpr bool FUSED = CK > 0;
    constexpr int TN = TA > 0 ? TA : 1;  // sizes of the tiles' registers
    using V = Vec<T, WQ>;
    auto& hop = lds_array<bf16_t[2][P][ROWS][KP], K, 0>();
    // with memory-state matrices, the same operand rows of the cell states
    auto& cop = lds_array<bf16_t[MEM ? 2 : 1][MEM ? P : 1][MEM ? ROWS : 1][KP], K, 1>();
    int& plain = lds_array<int, K, 2>();  // an infinite value was met
    auto& cedge = lds_array<float[2][NG][H], K, 3>();
    auto& ist = lds_array<u32x4[STAGE_IN ? 2 : 1][STAGE_IN ? NT * 16 * PI : 1], K, 4>();
    auto& ost = lds_array<u32x4[STAGE_OUT ? OBUF : 1][STAGE_OUT ? NT * 16 : 1][PF], K, 5>();
    auto& mst = lds_array<uint32_t[2][STAGE_IN && !(FUSED && P == 3) ? NTH : 1], K, 6>();

    int tid = threadIdx.x;
    // Opaque, or addresses that follow from it would be computed ahead of the
    // bodies and of the unit queue's loop and hold registers in all of them (fp32
    // H 32, 48 rows: 1150 -> 1075 us; not so with fp32 H 64 and four tiles, 4170
    // instead of 3480, whose loop leaves no registers for computing them again).
    if constexpr (!(H == 64 && NT == 4 && P == 3)) asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tg = NG == 1 ? 0 : wv / NWU, w = NG == 1 ? wv : wv % NWU;
    const int q = lane >> 4, n16 = lane & 15;
    const int u0 = K::UW * w + WQ * q;
    const int d = unit & 3;
    const RectD R = reinterpret_cast<const RectD*>(a.rects)[unit >> 2];
    const int steps = R.h + R.w - 1;
    const int sb = a.s0, se = min(a.s1, steps);
    if (sb >= se) return;
    // Whole units start at diagonal 0. Said here only where it takes 38 spilled
    // registers out of the loop (16 images of 64 rows 4836 -> 3515 us): elsewhere
    // it makes the loop slower (word batch 5%).
    if constexpr (!STEP && H == 64 && NT == 4 && P == 3) __builtin_assume(sb == 0);
    T* const Z = static_cast<T*>(a.z);
    T* const Y = static_cast<T*>(a.y);
    float* const Cs = a.c;

    for (int i = tid; i < (int)(sizeof(hop) / 16); i += NTH)
        reinterpret_cast<uint4*>(&hop[0][0][0][0])[i] = make_uint4(0, 0, 0, 0);
    if constexpr (MEM)
        for (int i = tid; i < (int)(sizeof(cop) / 16); i += NTH)
            reinterpret_cast<uint4*>(&cop[0][0][0][0])[i] = make_uint4(0, 0, 0, 0);
    if constexpr (NG > 1)
        for (int i = tid; i < 2 * NG * H; i += NTH) (&cedge[0][0][0])[i] = 0.0f;
    if (P == 3 && tid == 0) plain = FUSED ? a.xinf[unit >> 2] : 0;

    // values (hidden outputs, cell states) of row yy, the lane's units -> operand
    // rows of the next diagonal
    auto put = [&](auto& op, int buf, int yy, const float (&hv)[WQ]) {
        typename Vec<bf16_t, WQ>::R pc[P];
        if constexpr (P == 3) {
            uint32_t p0[3], p1[3];
            split2(hv[0], WQ > 1 ? hv[WQ > 1 ? 1 : 0] : 0.0f, p0);
            if constexpr (WQ == 4) split2(hv[2], hv[3], p1);
#pragma unroll
            for (int k = 0; k < P; ++k) {
                if constexpr (WQ == 4) pc[k] = u32x2{p0[k], p1[k]};
                else if constexpr (WQ == 2) pc[k] = p0[k];
                else pc[k] = (bf16_t)p0[k];
            }
        } else {
            pc[0] = Vec<bf16_t, WQ>::pack(hv);
        }
#pragma unroll
        for (int k = 0; k < P; ++k) {
            *reinterpret_cast<typename Vec<bf16_t, WQ>::R*>(&op[buf][k][yy][u0]) = pc[k];
            *reinterpret_cast<typename Vec<bf16_t, WQ>::R*>(&op[buf][k][yy + 1][H + u0]) = pc[k];
        }
    };

    float cprev[TN][WQ];  // cell states of the lane's rows on the previous diagonal
#pragma unroll
    for (int lt = 0; lt < TA; ++lt)
#pragma unroll
        for (int r = 0; r < WQ; ++r) cprev[lt][r] = 0.0f;
    // A operands, lane row n16 = 4 jj + e: tile r < WQ, gate e of unit
    // UW w + WQ jj + r; tile WQ, candidate of unit UW w + WQ jj + e.
    // Memory-state matrices: gates i, f_L, f_T of the sigmoid tiles (V rows).
    float wmax = 0.0f;  // largest magnitude of the wave's fp32 weights, NaN left out
    auto seen = [&](const float (&v)[8]) {
        if constexpr (P == 3) {
#pragma unroll
            for (int e = 0; e < 8; ++e) wmax = fmaxf(wmax, fabsf(v[e]));
        }
    };
    bf16x8 Ah[TILES][KS][P], Ax[TILES][FUSED ? CK : 1][P], Ac[MEM ? WQ : 1][MEM ? KS : 1][P];
    const T* const U = static_cast<const T*>(a.u) + (int64_t)d * G * 2 * H;
    const T* const Wx = static_cast<const T*>(a.wx) + (int64_t)d * G * a.c_in;
    const T* const Bd = static_cast<const T*>(a.b) + d * G;
    floatx4 bias[TILES];
    bool winf = false;
    auto load_weights = [&] {
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
            const int jj = n16 >> 2, e = n16 & 3;
            const bool ok = t < WQ || e < WQ;
            const int ul = K::UW * w + WQ * jj + (t < WQ ? t : (ok ? e : 0));
            const int row = (t < WQ ? e : 4) * H + ul;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const int k = 32 * ks + 8 * q;
                const T* p = U + (int64_t)row * 2 * H + k;
                const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
                const bool in = ok && k < 2 * H;
                const floatx4 v0 = in ? St<T>::ld4(p) : zero, v1 = in ? St<T>::ld4(p + 4) : zero;
                const float v[8] = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
                seen(v);
                make_op<T>(v, Ah[t][ks]);
            }
            if constexpr (MEM) {
                if (t < WQ) {
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        const int k = 32 * ks + 8 * q;
                        const T* p = static_cast<const T*>(a.v) + ((int64_t)d * 3 * H + (e < 3 ? e : 0) * H + ul) * 2 * H + k;
                        const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
                        const bool in = e < 3 && k < 2 * H;
                        const floatx4 v0 = in ? St<T>::ld4(p) : zero, v1 = in ? St<T>::ld4(p + 4) : zero;
                        const float v[8] = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
                        seen(v);
                        make_op<T>(v, Ac[t < WQ ? t : 0][ks]);
                    }
                }
            }
#pragma unroll
            for (int ks = 0; ks < CK; ++ks) {
                const int k = 32 * ks + 8 * q;
                const T* p = Wx + (int64_t)row * a.c_in + k;
                const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
                const floatx4 v0 = ok && k < a.c_in ? St<T>::ld4(p) : zero;
                const floatx4 v1 = ok && k + 4 < a.c_in ? St<T>::ld4(p + 4) : zero;
                const float v[8] = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
                seen(v);
                make_op<T>(v, Ax[t][ks]);
            }
        }
        if constexpr (FUSED) {
#pragma unroll
            for (int t = 0; t < TILES; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    bias[t][e] = t < WQ ? St<T>::ld1(Bd + e * H + u0 + t) : (e < WQ ? St<T>::ld1(Bd + 4 * H + u0 + e) : 0.0f);
        }
        __builtin_amdgcn_s_waitcnt(0);  // operands in registers before the step loop
        // taken here, or the weights would live until its use at the end
        winf = P == 3 && __any(wmax > BF16_LARGEST);
    };
    if constexpr (!STEP) load_weights();
    float cmax = 0.0f;  // largest cell state

    char* const sink = sink_ptr();
    const DiagMap M(R, d, a.canvas_w);
    const uint8_t* const mrow = a.mask + M.c0;
    const int xrow = P == 3 ? 8 * QI : a.c_in;  // 16-bit input values per cell
    const bf16_t* const xb = static_cast<const bf16_t*>(a.x) + M.c0 * xrow;
    T* const zb = Z + M.c0 * (4 * G) + d * G;
    T* const yb = Y + M.c0 * (4 * H) + d * H;
    float* const cb = Cs + M.c0 * (4 * H) + d * H;
    // Staged inputs: thread t moves chunk t % QI of rows t / QI, + RPI, ... of a
    // diagonal, loaded into registers four diagonals ahead and into LDS two
    // ahead (threads and rows past the last repeat a valid one: every lane
    // loads in every pass, so the number of loads in flight is the same on all
    // paths). Rows outside the diagonal read its nearest cell. Chunks of a
    // bf16 row past c_in read its first one and are zeroed.
    constexpr int RPI = NTH / QI < NT * 16 ? NTH / QI : NT * 16, NIT = (NT * 16 + RPI - 1) / RPI;
    constexpr bool MASKCHUNK = FUSED && P == 3;
    struct Set {
        u32x4 v[STAGE_IN ? NIT : 1];
        uint32_t mb;
        u32x4 x[TN][!STAGE_IN && FUSED ? CK * P : 1];
        typename V::R z[TN][!STAGE_IN && !FUSED ? 5 : 1];
        uint32_t m[TN];
    };
    constexpr int ZROW = 4 * G * (int)sizeof(T);
    const int irow = FUSED ? 2 * xrow : ZROW;
    const int it0 = tid % (RPI * QI), ic0 = it0 / QI, ir = it0 - ic0 * QI;
    const bool iok = !(FUSED && P == 1) || 8 * ir < a.c_in;
    const char* const ibase = (FUSED ? reinterpret_cast<const char*>(xb) : reinterpret_cast<const char*>(zb)) +
                              (iok ? 16 * ir : 0);
    auto load_tile = [&](int s, int lt, Set& in) {
        const int sc = min(s, steps - 1);
        const int ylo = max(0, sc - R.w + 1), yhi = min(R.h - 1, sc);
        const int yy = 16 * (tg * TPG + lt) + n16;
        const int idx = M.sx * sc + min(max(yy, ylo), yhi) * M.ky;
        in.m[lt] = mrow[idx];
        if constexpr (FUSED) {
            const bf16_t* xp = xb + (int64_t)idx * xrow + 8 * q;
#pragma unroll
            for (int ks = 0; ks < CK; ++ks)
#pragma unroll
                for (int k = 0; k < P; ++k) {
                    if constexpr (P == 3) {
                        in.x[lt][ks * P + k] = *reinterpret_cast<const u32x4*>(xp + k * CP + 32 * ks);
                    } else {
                        const bool in_row = 32 * ks + 8 * q < a.c_in;
                        const u32x4 v = *reinterpret_cast<const u32x4*>(xp + (in_row ? 32 * ks : -8 * q));
                        in.x[lt][ks] = in_row ? v : u32x4{0, 0, 0, 0};
                    }
                }
        } else {
            const T* zp = zb + u0 + (int64_t)idx * (4 * G);
#pragma unroll
            for (int t = 0; t < 5; ++t) in.z[lt][t] = ldw<T, WQ>(zp + t * H);
        }
    };
    auto load = [&](int s, Set& in) {
        if constexpr (STAGE_IN) {
            const int sc = min(s, steps - 1);
            const int ylo = max(0, sc - R.w + 1), yhi = min(R.h - 1, sc);
            const int sxs = M.sx * sc;
#pragma unroll
            for (int it = 0; it < NIT; ++it)
                in.v[it] = *reinterpret_cast<const u32x4*>(
                    ibase + (int64_t)(sxs + min(max(ic0 + it * RPI, ylo), yhi) * M.ky) * irow);
            if constexpr (!MASKCHUNK)
                in.mb = mrow[sxs + min(max(min(tid, NT * 16 - 1), ylo), yhi) * M.ky];
        } else {
#pragma unroll
            for (int lt = 0; lt < TA; ++lt) load_tile(s, lt, in);
        }
    };
    Set s0, s1;
    float hback[TN][WQ];
    auto behind = [&](int lt) {  // the lane's row of a tile has a cell on diagonal sb - 1
        const int yy = 16 * (tg * TPG + lt) + n16;
        return sb > 0 && yy < R.h && yy < sb && sb - 1 - yy < R.w;
    };
    if constexpr (STEP) {
        load(sb, s0);
#pragma unroll
        for (int lt = 0; lt < TA; ++lt)
            if (behind(lt)) {
                const int64_t p = M.at(M.base(sb - 1), 16 * (tg * TPG + lt) + n16) * (4 * H) + d * H + u0;
                const typename V::R hr = ldw<T, WQ>(Y + p);
                const typename Vec<float, WQ>::R cr = ldw<float, WQ>(Cs + p);
#pragma unroll
                for (int r = 0; r < WQ; ++r) {
                    hback[lt][r] = V::get(hr, r);
                    cprev[lt][r] = Vec<float, WQ>::get(cr, r);
                }
            }
        load_weights();
    }
    // registers -> LDS buffers of diagonal s
    auto stage_in = [&](int s, const Set& in) {
        if constexpr (STAGE_IN) {
#pragma unroll
            for (int it = 0; it < NIT; ++it)
                ist[s & 1][min(ic0 + it * RPI, NT * 16 - 1) * PI + ir] = iok ? in.v[it] : u32x4{0, 0, 0, 0};
            if constexpr (!MASKCHUNK) {
                // taken here, so that it waits for this set's loads and not,
                // moved past the next ones, for those
                uint32_t mb = in.mb;
                asm volatile("" : "+v"(mb));
                mst[s & 1][tid] = mb;
            }
        }
    };
    // A wave of one tile computes the input part of the next diagonal behind the
    // cell update; a wave of several tiles goes through them one after another
    // (from the bottom: a tile's top edge is the tile above it of the previous
    // diagonal), with the accumulators of one tile only.
    constexpr bool AHEAD = TPG == 1 && FUSED;
    constexpr int LEAD = AHEAD ? 2 : 1;
    // Pre-activations so far, leading products, products of the lower pieces.
    // fp32: an MFMA rounds its sum worse than an addition (measured 0.58 ulp
    // rms against 0.29), so both parts of the reduction start from zero, where
    // their sums are small, and meet the bias in additions. bf16: one sum.
    floatx4 zx[TILES], acc[TILES], low[TILES];
    uint32_t mk;
    // Diagonal s's pre-activations from its inputs alone (staged, or in `in`).
    auto start = [&](int s, int lt, const Set& in) {
        {
            const int yy = 16 * (tg * TPG + lt) + n16;
            const u32x4* row = &ist[s & 1][STAGE_IN ? yy * PI : 0];
            if constexpr (STAGE_IN) {
                mk = MASKCHUNK ? row[QI - 1][0] : mst[s & 1][yy];
            } else {
                mk = in.m[lt];  // taken here, as the staged mask byte
                asm volatile("" : "+v"(mk));
            }
#pragma unroll
            for (int t = 0; t < TILES; ++t) low[t] = floatx4{0.f, 0.f, 0.f, 0.f};
            if constexpr (FUSED) {
#pragma unroll
                for (int t = 0; t < TILES; ++t) acc[t] = P == 3 ? floatx4{0.f, 0.f, 0.f, 0.f} : bias[t];
#pragma unroll
                for (int ks = 0; ks < CK; ++ks) {
                    bf16x8 bx[P];
#pragma unroll
                    for (int k = 0; k < P; ++k) {
                        const u32x4 v = STAGE_IN ? row[4 * (CK * k + ks) + q] : in.x[lt][STAGE_IN ? 0 : ks * P + k];
                        __builtin_memcpy(&bx[k], &v, 16);
                    }
                    mma_tiles<P, TILES>(Ax, ks, bx, acc, low);
                }
                if constexpr (P == 3) {
#pragma unroll
                    for (int t = 0; t < TILES; ++t) {
                        zx[t] = acc[t];
                        acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
                    }
                }
            } else {
                typename V::R zv[5];
#pragma unroll
                for (int t = 0; t < 5; ++t)
                    zv[t] = STAGE_IN ? ldw<T, WQ>(reinterpret_cast<const T*>(row) + t * H + u0)
                                     : in.z[lt][STAGE_IN ? 0 : t];
#pragma unroll
                for (int r = 0; r < WQ; ++r) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) (P == 3 ? zx : acc)[r][e] = V::get(zv[e], r);
                    (P == 3 ? zx : acc)[WQ][r] = V::get(zv[4], r);
                }
                if constexpr (P == 3) {
#pragma unroll
                    for (int t = 0; t < TILES; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
                }
            }
        }
    };
    // Staged outputs of diagonal s written back: thread t stores chunk t % QF
    // of rows t / QF, + RPF, ... (threads and rows past the last, and rows
    // outside the diagonal, repeat a cell of it and write the same bytes
    // twice: every lane stores in every pass). Non-temporal: the next reader is
    // the backward or another layer (word batch 228 -> 187 us, line batch
    // 1300 -> 1284 us).
    constexpr int RPF = STAGE_OUT ? (NTH / QF < NT * 16 ? (NTH / QF > 0 ? NTH / QF : 1) : NT * 16) : 1;
    constexpr int NITF = (NT * 16 + RPF - 1) / RPF;
    static_assert(!STAGE_OUT || NTH >= QF, "a row per pass");
    const int ft0 = tid % (RPF * QF), fc0 = ft0 / QF, fr = ft0 - fc0 * QF;
    char* const fbase = fr < QZ        ? reinterpret_cast<char*>(zb) + 16 * fr
                        : fr < QZ + QY ? reinterpret_cast<char*>(yb) + 16 * (fr - QZ)
                                       : reinterpret_cast<char*>(cb) + 16 * (fr - QZ - QY);
    const int frow = fr < QZ ? ZROW : fr < QZ + QY ? 4 * H * (int)sizeof(T) : 16 * H;
    auto flush = [&](int s) {
        if constexpr (STAGE_OUT) {
            const int ylo = max(0, s - R.w + 1), yhi = min(R.h - 1, s);
            constexpr int GR = NITF < 4 ? NITF : 4;  // passes per LDS round trip (registers)
#pragma unroll
            for (int i0 = 0; i0 < NITF; i0 += GR) {
                u32x4 v[GR];
#pragma unroll
                for (int k = 0; k < GR; ++k)
                    if (i0 + k < NITF)
                        v[k] = ost[OBUF == 2 ? s & 1 : 0][min(max(fc0 + (i0 + k) * RPF, ylo), yhi)][fr];
#pragma unroll
                for (int k = 0; k < GR; ++k)
                    if (i0 + k < NITF)
                        __builtin_nontemporal_store(
                            v[k], reinterpret_cast<u32x4*>(
                                      fbase + (int64_t)(M.sx * s + min(max(fc0 + (i0 + k) * RPF, ylo), yhi) * M.ky) *
                                                  frow));
                if constexpr (NITF > GR) __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    // far: staged, the inputs of diagonal s + LEAD on their way to LDS (into the
    // buffer that diagonal s - 1's or s's input part has done with); unstaged,
    // with one tile per wave, the set to load those of s + 2 into, with several
    // the one set (this diagonal's, each tile replaced by the next one's).
    auto step = [&](int s, Set& far, const Set& nxt, auto with_flush) {
        const int cur = s & 1, prv = cur ^ 1;
        const int ylo = max(0, s - R.w + 1), yhi = min(R.h - 1, s);
        lds_barrier();  // h and edge states of diagonal s - 1 written
        auto contract = [&](int lt) {
            const int yy = 16 * (tg * TPG + lt) + n16;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                bf16x8 bh[P];
#pragma unroll
                for (int k = 0; k < P; ++k)
                    bh[k] = as_bf16x8(*reinterpret_cast<const uint4*>(&hop[prv][k][yy][32 * ks + 8 * q]));
                mma_tiles<P, TILES>(Ah, ks, bh, acc, low);
            }
            if constexpr (MEM) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    bf16x8 bc[P];
#pragma unroll
                    for (int k = 0; k < P; ++k)
                        bc[k] = as_bf16x8(*reinterpret_cast<const uint4*>(&cop[prv][k][yy][32 * ks + 8 * q]));
                    mma_tiles<P, WQ>(Ac, ks, bc, reinterpret_cast<floatx4(&)[WQ]>(acc),
                                     reinterpret_cast<floatx4(&)[WQ]>(low));
                }
            }
        };
        if constexpr (AHEAD && TA > 0) contract(0);
        if constexpr (decltype(with_flush)::value) flush(s - 1);
        if constexpr (!STEP) {
            stage_in(s + LEAD, far);
            if constexpr (STAGE_IN) load(s + LEAD + 2, far);
            else if constexpr (AHEAD) load(s + 2, far);
        }
        if constexpr (OBUF == 1) lds_barrier();  // the write-back's reads are done
#pragma unroll
        for (int lt = TA - 1; lt >= 0; --lt) {
            const int yy = 16 * (tg * TPG + lt) + n16;
            if constexpr (!AHEAD) {
                start(s, lt, far);
                if constexpr (!STAGE_IN && !STEP) load_tile(s + 1, lt, far);
                contract(lt);
            }
            float ct[WQ];  // cell states of the row above
#pragma unroll
            for (int r = 0; r < WQ; ++r) {
                float edge = 0.0f;
                if (lt > 0) edge = last_to_first(cprev[lt > 0 ? lt - 1 : 0][r]);
                else if (NG > 1 && tg > 0) edge = cedge[prv][tg > 0 ? tg - 1 : 0][u0 + r];
                ct[r] = row_above(cprev[lt][r], edge);
            }
            const bool in = yy >= ylo && yy <= yhi, live = in && mk != 0;
            auto sg = [](float z) { return cell_sigm<MEM>(z); };
            auto th = [](float z) { return cell_tanh<MEM>(z); };
            // The bias meets the lower products first: a leading sum lies on a grid
            // as coarse as the pre-activation's, where adding a bias rounds the same
            // way in every cell (mean error of the candidates 1.1e-8; 2.9e-9 this way).
            auto pre = [&](int t, int e) {
                if constexpr (P == 1) return acc[t][e];
                else if constexpr (FUSED) return ((low[t][e] + bias[t][e]) + zx[t][e]) + acc[t][e];
                else return (zx[t][e] + acc[t][e]) + low[t][e];
            };
            float gv[5][WQ], hv[WQ], cv[WQ];
#pragma unroll
            for (int r = 0; r < WQ; ++r) {
#pragma unroll
                for (int e = 0; e < 4; ++e) gv[e][r] = sg(pre(r, e));
                gv[4][r] = th(pre(WQ, r));
                const float cn = gv[0][r] * gv[4][r] + gv[1][r] * cprev[lt][r] + gv[2][r] * ct[r];
                const float hn = gv[3][r] * th(cn);
                cv[r] = live ? cn : 0.0f;
                hv[r] = live ? hn : 0.0f;
                cprev[lt][r] = cv[r];
                gv[0][r] = mk != 0 ? gv[0][r] : -1.0f;  // marks a masked cell for the backward
            }
            if constexpr (!STEP) put(hop, cur, yy, hv);
            if constexpr (MEM) {
#pragma unroll
                for (int r = 0; r < WQ; ++r) cmax = fmaxf(cmax, fabsf(cv[r]));
                put(cop, cur, yy, cv);
            }
            if constexpr (NG > 1) {
                if (lt == TPG - 1 && n16 == 15) {
#pragma unroll
                    for (int r = 0; r < WQ; ++r) cedge[cur][tg][u0 + r] = cv[r];
                }
            }
            if constexpr (STAGE_OUT) {
                u32x4* const row = &ost[OBUF == 2 ? cur : 0][yy][0];
#pragma unroll
                for (int t = 0; t < 5; ++t) stw<T, WQ>(reinterpret_cast<T*>(row) + t * H + u0, gv[t]);
                stw<T, WQ>(reinterpret_cast<T*>(row + QZ) + u0, hv);
                stw<float, WQ>(reinterpret_cast<float*>(row + QZ + QY) + u0, cv);
            } else {
                const int64_t idx = M.sx * s + yy * M.ky;
                T* const zp = in ? zb + u0 + idx * (4 * G) : reinterpret_cast<T*>(sink);
                T* const yp = in ? yb + u0 + idx * (4 * H) : reinterpret_cast<T*>(sink);
                float* const cp = in ? cb + u0 + idx * (4 * H) : reinterpret_cast<float*>(sink);
#pragma unroll
                for (int t = 0; t < 5; ++t) stw<T, WQ>(zp + t * H, gv[t]);
                stw<T, WQ>(yp, hv);
                stw<float, WQ>(cp, cv);
            }
            if constexpr (!AHEAD) __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (AHEAD && TA > 0 && !STEP) start(s + 1, 0, nxt);
    };

    auto met = [&] { return winf || (MEM && cmax > BF16_LARGEST); };
    constexpr bool ONE = !STAGE_IN && !AHEAD;
    if constexpr (STEP) {
        lds_barrier();  // every zero written before the read-back fills the same rows
#pragma unroll
        for (int lt = 0; lt < TA; ++lt) {
            if (behind(lt)) put(hop, (sb & 1) ^ 1, 16 * (tg * TPG + lt) + n16, hback[lt]);
            if constexpr (NG > 1) {
                if (lt == TPG - 1 && n16 == 15) {
#pragma unroll
                    for (int r = 0; r < WQ; ++r) cedge[(sb & 1) ^ 1][tg][u0 + r] = cprev[lt][r];
                }
            }
        }
        stage_in(sb, s0);
        if constexpr (STAGE_IN) lds_barrier();
        if constexpr (AHEAD && TA > 0) start(sb, 0, s0);
        step(sb, s0, s0, std::false_type{});
        if (P == 3 && met()) plain = 1;
        lds_barrier();
        if constexpr (STAGE_OUT) flush(sb);
        if constexpr (P == 3) {
            if (__builtin_amdgcn_readfirstlane(plain)) plain_fwd_unit<H, MEM>(kern_args<FwdArgs>(), unit, sb, se);
        }
        return;
    }
    load(sb, s0);
    if constexpr (!ONE) load(sb + 1, s1);
    if constexpr (STAGE_IN) {
        stage_in(sb, s0);
        if constexpr (LEAD == 2) stage_in(sb + 1, s1);
        load(sb + LEAD, s0);
        load(sb + LEAD + 1, s1);
        lds_barrier();
    }
    if constexpr (AHEAD && TA > 0) start(sb, 0, s0);
    if constexpr (STAGE_OUT) {
        // two steps ahead of the loop: it is entered with the memory operations
        // in flight that its own steps leave, so its waits are exact
        step(sb, s0, s1, std::false_type{});
        int s = sb + 1;
        if (s < se) {
            step(s, ONE ? s0 : s1, s0, std::true_type{});
            ++s;
        }
        while (s < se) {
            step(s, s0, s1, std::true_type{});
            if (++s >= se) break;
            step(s, ONE ? s0 : s1, s0, std::true_type{});
            ++s;
        }
        if (P == 3 && met()) plain = 1;
        lds_barrier();
        flush(se - 1);
    } else {
        // as many stores as a step has, into the sink, for the same reason
#pragma unroll
        for (int lt = 0; lt < TA; ++lt) {
            float zero[WQ];
#pragma unroll
            for (int r = 0; r < WQ; ++r) zero[r] = 0.0f;
#pragma unroll
            for (int t = 0; t < 5; ++t) stw<T, WQ>(reinterpret_cast<T*>(sink) + t * H, zero);
            stw<T, WQ>(reinterpret_cast<T*>(sink), zero);
            stw<float, WQ>(reinterpret_cast<float*>(sink), zero);
            asm volatile("" ::: "memory");
        }
        for (int s = sb;;) {
            step(s, s0, s1, std::false_type{});
            if (++s >= se) break;
            step(s, ONE ? s0 : s1, s0, std::false_type{});
            if (++s >= se) break;
        }
        if constexpr (P == 3) {
            if (met()) plain = 1;
            lds_barrier();
        }
    }
    if constexpr (P == 3) {
        if (__builtin_amdgcn_readfirstlane(plain)) plain_fwd_unit<H, MEM>(kern_args<FwdArgs>(), unit, sb, se);
    }
}

template <int H, int NT, typename T, int CK, int WQ, int NG, bool MEM, bool STEP>
__global__ void __launch_bounds__((FwdK<H, NT, T, CK, WQ, NG, MEM>::NTH))
__attribute__((amdgpu_waves_per_eu(FwdK<H, NT, T, CK, WQ, NG, MEM>::WPE))) k_fwd(FwdArgs args) {
    const FwdArgs a = STEP ? step_args(args) : args;
    using K = FwdK<H, NT, T, CK, WQ, NG, MEM>;
    auto run = [&](int unit) {
        if constexpr (NT == 1) {
            fwd_unit<H, NT, T, CK, WQ, NG, MEM, 1, STEP>(a, unit);
        } else {
            const int rows = reinterpret_cast<const RectD*>(a.rects)[unit >> 2].h;
            const int tg = NG == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) / K::NWU;
            with_tiles<K::TPG, NG == 1 ? 1 : 0>((rows + 15) / 16 - tg * K::TPG, [&](auto ta) {
                fwd_unit<H, NT, T, CK, WQ, NG, MEM, decltype(ta)::value, STEP>(a, unit);
            });
        }
    };
    if constexpr (STEP) run(a.units[blockIdx.x]);
    else for_units(a, run);
}

// Hidden sizes whose forward wavefront takes over the projection: where Wx's
// operands fit in registers beside U's. fp32 H = 64 has 240 registers of U in
// each of four waves already (with Wx it spills over a hundred). With 33-64
// channels some of the others spill too; forward with the projection inside
// against apart, us, 64 channels, 16 / 128 images of 16 t rows:
//   fp32 H 4,  t = 1    256 /  238 against  242 /  258
//              t = 4    470 /  857          511 /  829
//   fp32 H 16, t = 1    237 /  216          325 /  450
//              t = 4    655 /  986          863 / 1586
//   fp32 H 32, t = 1    554 /  429          491 /  758
//              t = 2    827 /  929          783 / 1405
//              t = 3   1338 / 1420         1372 / 2160
//              t = 4   2784 / 3706         2117 / 3871
//   memory H 16, t = 3 1118 / 1357          739 / 1226
//   memory H 32, t = 1  490 /  510          630 /  882
//                t = 4 2442 / 2971         2774 / 4317
// (fp32 H 8, the other heights of the memory layers and bf16: inside is faster.)
// Full batches gain from it all but everywhere; a few images of H 32 or of
// memory H 16 with 33-48 rows lose.
template <typename T>
constexpr bool fwd_fusable(int hidden) {
    return hidden <= (std::is_same<T, float>::value ? 32 : 64);
}

template <int H, int NT, typename T, int CK, int WQ, int NG, bool MEM>
WaveKernel fwd_kernel_ck(bool one_step) {
    constexpr int th = FwdK<H, NT, T, CK, WQ, NG, MEM>::NTH;
    if constexpr (!MEM) {
        if (one_step) return {reinterpret_cast<const void*>(&k_fwd<H, NT, T, CK, WQ, NG, MEM, true>), th};
    }
    return {reinterpret_cast<const void*>(&k_fwd<H, NT, T, CK, WQ, NG, MEM, false>), th};
}

template <int H, int NT, typename T, int WQ, int NG, bool MEM = false>
WaveKernel fwd_kernel(int ck, bool one_step = false) {
    if (ck == 0) return fwd_kernel_ck<H, NT, T, 0, WQ, NG, MEM>(one_step);
    if constexpr (fwd_fusable<T>(H)) {
        if (ck == 1) return fwd_kernel_ck<H, NT, T, 1, WQ, NG, MEM>(one_step);
        if (ck == 2) return fwd_kernel_ck<H, NT, T, 2, WQ, NG, MEM>(one_step);
    }
    return {};
}

// One translation unit per hidden size (k_wave_fwd_*.hip). one_step: the kernel
// of the per-diagonal schedule.
WaveKernel fwd_kernel_f32_h4(int nt, int ck, bool one_step);
WaveKernel fwd_kernel_f32_h8(int nt, int ck, bool one_step);
WaveKernel fwd_kernel_f32_h16(int nt, int ck, bool one_step);
WaveKernel fwd_kernel_f32_h32(int nt, int ck, bool one_step);
WaveKernel fwd_kernel_f32_h64(int nt, int ck, bool one_step);
WaveKernel fwd_kernel_bf16_h32(int nt, int ck, bool one_step);
WaveKernel fwd_kernel_bf16_h64(int nt, int ck, bool one_step);
WaveKernel fwd_kernel_mem_h16(int nt, int ck);
WaveKernel fwd_kernel_mem_h32(int nt, int ck);

}  // namespace mdl
