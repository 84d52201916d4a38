// Backward anti-diagonal wavefront, the reverse of wave_fwd.hpp's. With
// successors S (right, same row, next diagonal) and E (below, row + 1, next
// diagonal):
//   dh = dY + (U^T da_S)[0:H] + (U^T da_E)[H:2H]
//   dc = dh o (1 - tanh^2 c) + dc_S f_L(S) + dc_E f_T(E)
//   da = (dc g i(1-i), dc c_L f_L(1-f_L), dc c_T f_T(1-f_T), dh tanh(c) o(1-o), dc i (1-g^2))
//
// The lane mapping is the forward's: lane 16q + n of wave w owns units
// 4 WQ w + WQ q + r, r < WQ, of row n of each of its tiles. Per diagonal a wave
// updates its cells (phase A) and leaves da in LDS as operand rows; after a
// barrier it contracts them with the U^T rows of its own units, left and top
// predecessor part side by side in one MFMA tile (A rows (unit q, output),
// outputs: WQ left, WQ top; two tiles at WQ = 4), so the results land in the
// lanes that need them on the next diagonal: the left part on the same row, the
// top part and dc f_T one row up, a DPP move (rows 16 -> 15 through a rotation,
// or LDS between tile groups). The gates, upstream gradients and cell states
// come in, and the gate gradients leave, through LDS as whole rows in 16-byte
// chunks.
//
// fp32 operands are three bf16 pieces each (split.hpp).
//
// Measured before (scalar operand exchange, fp32 MFMA, partial sums of the
// products through LDS; bf16 H 64 with tall rectangles unstaged) and after:
//   fp32 H 32, 64 lines of 32 rows    1670 -> 1550 us (4.84 GB, 3.1 TB/s)
//   fp32 H 32, 32 images of 16 rows    163 ->  134 us
//   fp32 H 64, 64 images of 8 rows     292 ->  198 us
//   bf16 H 64, 24 lines of 20-60 rows 11.9 ->  2.9 ms
#pragma once

#include <type_traits>

#include "kernels.hpp"
#include "wave.hpp"
#include "wave_plain.hpp"

namespace mdl {

template <int H, int NT, typename T, int WQ, int NG, bool MEM>
struct BwdK {
    static constexpr int P = Pieces<T>::N;
    static constexpr int UW = 4 * WQ, NWU = H / UW;     // hidden units per wave, waves per tile group
    static constexpr int TPG = NT / NG;                 // tiles per wave (group tg: tiles tg TPG ...)
    static constexpr int NTH = 64 * NWU * NG;
    static constexpr int KS = (5 * H + 31) / 32;        // K steps over da
    static constexpr int KP = 32 * KS + 8;              // operand row pitch: 16-byte reads of 16 rows hit distinct banks
    // Outputs per lane: WQ left parts, WQ top parts; with memory-state matrices
    // as many again for the cell states.
    static constexpr int OUTS = (MEM ? 4 : 2) * WQ;
    static constexpr int OT = (OUTS + 3) / 4;           // output tiles per wave
    static constexpr int WPE = OT * KS * P * 4 > 170 || NTH > 512 ? 1 : 2;
    // Inputs of a cell in 16-byte chunks: 5H gates, H upstream gradients
    // (storage type), and H cell states (fp32) of the diagonal before; the
    // extra chunk of the pitch spreads rows over banks.
    static constexpr int QZ = 5 * H * (int)sizeof(T) / 16, QY = H * (int)sizeof(T) / 16, QC = H / 4;
    static constexpr int QF = QZ + QY + QC, PB = QF + 1, PZ = QZ + 1;
    static constexpr size_t IN1 = (size_t)NT * 16 * PB * 16;
    static constexpr size_t DA1 = (size_t)P * NT * 16 * KP * 2;
    static constexpr size_t DZ1 = P == 3 ? (size_t)NT * 16 * PZ * 16 : 0;  // one-piece operand rows are the dZ rows
    static constexpr size_t LIM = 158 * 1024;
    static constexpr bool STAGE = NTH >= QF && IN1 + DA1 + DZ1 <= LIM;
    // One barrier a diagonal where every buffer fits twice and one wave holds
    // all tiles; else single buffers and a second barrier.
    static constexpr bool DB = STAGE && NG == 1 && 2 * (IN1 + DA1 + DZ1) <= LIM;
    static constexpr int NB = DB ? 2 : 1;
    static constexpr bool FITS = STAGE || DA1 <= LIM;
    static_assert(H % UW == 0 && NT % NG == 0 && NTH <= 1024, "wave split");
    static_assert(!MEM || (NG == 1 && P == 3), "memory-state matrices: fp32, one tile group");
};

// TA: the group's tiles that hold rows of the rectangle.
template <int H, int NT, typename T, int WQ, int NG, bool MEM, int TA>
__device__ __forceinline__ void bwd_unit(const BwdArgs& a, const int unit) {
    using K = BwdK<H, NT, T, WQ, NG, MEM>;
    constexpr int P = K::P, NWU = K::NWU, TPG = K::TPG, KS = K::KS, KP = K::KP, OT = K::OT, NTH = K::NTH;
    constexpr int QZ = K::QZ, QY = K::QY, QF = K::QF, PB = K::PB, PZ = K::PZ, NB = K::NB;
    constexpr bool STAGE = K::STAGE, DB = K::DB;
    constexpr int G = 5 * H;
    using V = Vec<T, WQ>;
    auto& dap = lds_array<bf16_t[NB][P][NT * 16][KP], K, 0>();
    auto& dzs = lds_array<u32x4[NB][P == 3 && STAGE ? NT * 16 : 1][PZ], K, 1>();
    auto& ist = lds_array<u32x4[NB][STAGE ? NT * 16 * PB : 1], K, 2>();
    // between tile groups: the top parts and dc f_T of a group's first row
    int& plain = lds_array<int, K, 3>();  // a gate gradient without pieces was met
    static_assert(P == 1 || sizeof(dap) >= sizeof(float) * 4 * H * NT * 16, "scratch of plain_bwd_unit");
    auto& gedge = lds_array<float[NG][H], K, 4>();
    auto& dedge = lds_array<float[2][NG][H], K, 5>();

    int tid = threadIdx.x;
    // Opaque, or addresses that follow from it would be computed ahead of the
    // bodies and of the unit queue's loop and hold registers in all of them (fp32
    // H 64, 48 rows: 70 -> 13 spilled, 6.6 -> 5.6 ms).
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tg = NG == 1 ? 0 : wv / NWU, w = NG == 1 ? wv : wv % NWU;
    const int q = lane >> 4, n16 = lane & 15;
    const int u0 = K::UW * w + WQ * q;
    const int d = unit & 3;
    const RectD R = reinterpret_cast<const RectD*>(a.rects)[unit >> 2];
    const int steps = R.h + R.w - 1;
    T* const Z = static_cast<T*>(a.z);
    const T* const DY = static_cast<const T*>(a.dy);

    for (int i = tid; i < (int)(sizeof(dap) / 16); i += NTH)
        reinterpret_cast<uint4*>(&dap[0][0][0][0])[i] = make_uint4(0, 0, 0, 0);
    if (P == 3 && tid == 0) plain = 0;
    if constexpr (NG > 1) {
        for (int i = tid; i < NG * H; i += NTH) (&gedge[0][0])[i] = 0.0f;
        for (int i = tid; i < 2 * NG * H; i += NTH) (&dedge[0][0][0])[i] = 0.0f;
    }

    // Order of da along an operand row. Three pieces: (unit, sigmoid gate),
    // then the candidates: a lane writes its gates as one vector. One piece:
    // the canvas order, so that the rows leave as they are.
    auto u_row = [](int k) {  // row of U of operand value k
        if constexpr (P == 3) return k < 4 * H ? (k & 3) * H + (k >> 2) : k;
        else return k;
    };
    // A operands, lane row n16 = 4 jj + e of tile t: output o = 4t + e, the left
    // part (column) of unit UW w + WQ jj + o for o < WQ, then the top parts.
    float wmax = 0.0f;  // largest magnitude of the wave's fp32 weights, NaN left out
    bf16x8 A[OT][KS][P];
    const T* const U = static_cast<const T*>(a.u) + (int64_t)d * G * 2 * H;
#pragma unroll
    for (int t = 0; t < OT; ++t) {
        const int o = 4 * t + (n16 & 3), ub = K::UW * w + WQ * (n16 >> 2);
        const bool ok = o < K::OUTS, state = MEM && o >= 2 * WQ;
        const int ol = state ? o - 2 * WQ : o;
        // A piece MFMA's mean error is a little below zero (some 5e-11 of the sum's
        // size). With the top parts computed negated, those of a cell's two shares
        // cancel instead of adding up along the diagonals (gate gradients of the word
        // batch, summed per gate: 1.6e-7 off, 8.6e-8 this way, 8.5e-8 on the fp32 MFMA).
        const bool top = P == 3 && ol >= WQ;
        const int col = !ok ? 0 : ol < WQ ? ub + ol : H + ub + ol - WQ;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = 32 * ks + 8 * q + e;
                const int row = u_row(k < G ? k : 0);
                if (MEM && state)  // V has the rows of i, f_L, f_T
                    v[e] = ok && k < G && row < 3 * H
                               ? St<T>::ld1(static_cast<const T*>(a.v) + ((int64_t)d * 3 * H + row) * 2 * H + col)
                               : 0.0f;
                else
                    v[e] = ok && k < G ? St<T>::ld1(U + (int64_t)row * 2 * H + col) : 0.0f;
            }
            if constexpr (P == 3) {
#pragma unroll
                for (int e = 0; e < 8; ++e) wmax = fmaxf(wmax, fabsf(v[e]));
            }
            if (top) {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = -v[e];
            }
            make_op<T>(v, A[t][ks]);
        }
    }
    __builtin_amdgcn_s_waitcnt(0);  // operands in registers before the step loop

    const DiagMap M(R, d, a.canvas_w);
    T* const zb = Z + M.c0 * (4 * G) + d * G;
    const T* const dyb = DY + M.c0 * (4 * H) + d * H;
    const float* const cb = a.c + M.c0 * (4 * H) + d * H;
    constexpr int ZROW = 4 * G * (int)sizeof(T);

    // What the next diagonal (s - 1) takes over: the lane's own products (left
    // and top part), dc f_L, dc f_T, and the cell state of its own rows.
    float dmax = 0.0f;  // fp32: the largest gate gradient, NaN left out
    constexpr int TN = TA > 0 ? TA : 1;  // sizes of the tiles' registers
    float gl[TN][WQ], gt[TN][WQ], dcl[TN][WQ], dct[TN][WQ], co[TN][WQ];
#pragma unroll
    for (int lt = 0; lt < TA; ++lt) {
        const int yy = 16 * (tg * TPG + lt) + n16;
        const int yc = min(max(yy, max(0, steps - R.w)), R.h - 1);  // a row of the last diagonal
        const float* cp = cb + (int64_t)(M.sx * (steps - 1) + yc * M.ky) * (4 * H) + u0;
#pragma unroll
        for (int r = 0; r < WQ; ++r) {
            gl[lt][r] = gt[lt][r] = dcl[lt][r] = dct[lt][r] = 0.0f;
            co[lt][r] = cp[r];
        }
    }

    // Staged inputs: thread t moves chunk t % QF of rows t / QF, + RPI, ... of
    // diagonal s's record (its gates and upstream gradients, the cell states of
    // s - 1), into registers three or four diagonals ahead, into LDS one or two
    // ahead. Threads and rows past the last, and rows outside the diagonal,
    // repeat a valid one (every lane loads: the number of loads in flight is
    // the same on all paths).
    constexpr int RPI = STAGE ? (NTH / QF < NT * 16 ? NTH / QF : NT * 16) : 1;
    constexpr int NIT = (NT * 16 + RPI - 1) / RPI;
    struct Set {
        u32x4 v[STAGE ? NIT : 1];
        typename V::R g[STAGE ? 1 : TN][5], dy[STAGE ? 1 : TN];
        typename Vec<float, WQ>::R cl[STAGE ? 1 : TN], ct[STAGE ? 1 : TN];
    };
    const int it0 = tid % (RPI * QF), ic0 = it0 / QF, ir = it0 - ic0 * QF;
    const int back = ir >= QZ + QY ? 1 : 0;
    const char* const ibase = ir < QZ        ? reinterpret_cast<const char*>(zb) + 16 * ir
                              : ir < QZ + QY ? reinterpret_cast<const char*>(dyb) + 16 * (ir - QZ)
                                             : reinterpret_cast<const char*>(cb) + 16 * (ir - QZ - QY);
    const int irow = ir < QZ ? ZROW : ir < QZ + QY ? 4 * H * (int)sizeof(T) : 16 * H;
    auto load = [&](int s, Set& in) {
        if constexpr (STAGE) {
            const int sc = max(s - back, 0);
            const int ylo = max(0, sc - R.w + 1), yhi = min(R.h - 1, sc);
            const int sxs = M.sx * sc;
#pragma unroll
            for (int it = 0; it < NIT; ++it)
                in.v[it] = *reinterpret_cast<const u32x4*>(
                    ibase + (int64_t)(sxs + min(max(ic0 + it * RPI, ylo), yhi) * M.ky) * irow);
        }
    };
    // unstaged: the lane's own inputs of one tile (a missing top predecessor
    // reads the cell itself; the left one's state is also that of the row's own
    // cell on the next diagonal, so it is the row's even where the row is not
    // in diagonal s)
    auto load_tile = [&](int s, int lt, Set& in) {
        if constexpr (!STAGE) {
            const int sc = max(s, 0);
            const int ylo = max(0, sc - R.w + 1), yhi = min(R.h - 1, sc);
            const int yc = min(max(16 * (tg * TPG + lt) + n16, ylo), yhi);
            const int idx = M.sx * sc + yc * M.ky;
            const int sl = max(s - 1, 0);
            const int il = M.sx * sl + min(max(16 * (tg * TPG + lt) + n16, max(0, sl - R.w + 1)), min(R.h - 1, sl)) * M.ky;
            const int iu = yc > 0 ? idx - M.sx - M.ky : idx;
#pragma unroll
            for (int t = 0; t < 5; ++t) in.g[lt][t] = ldw<T, WQ>(zb + (int64_t)idx * (4 * G) + t * H + u0);
            in.dy[lt] = ldw<T, WQ>(dyb + (int64_t)idx * (4 * H) + u0);
            in.cl[lt] = ldw<float, WQ>(cb + (int64_t)il * (4 * H) + u0);
            in.ct[lt] = ldw<float, WQ>(cb + (int64_t)iu * (4 * H) + u0);
        }
    };
    auto stage_in = [&](int s, const Set& in) {
        if constexpr (STAGE) {
#pragma unroll
            for (int it = 0; it < NIT; ++it)
                ist[DB ? s & 1 : 0][min(ic0 + it * RPI, NT * 16 - 1) * PB + ir] = in.v[it];
        }
    };
    // Staged gate gradients of diagonal s to the workspace (as the forward's
    // write-back, but cached: the gradient kernel that reads them comes next;
    // non-temporal stores took 233 us on the word batch, these 217).
    constexpr int RPF = STAGE ? (NTH / QZ < NT * 16 ? NTH / QZ : NT * 16) : 1;
    constexpr int NITF = (NT * 16 + RPF - 1) / RPF;
    const int ft0 = tid % (RPF * QZ), fc0 = ft0 / QZ, fr = ft0 - fc0 * QZ;
    char* const fbase = reinterpret_cast<char*>(zb) + 16 * fr;
    auto flush = [&](int s) {
        if constexpr (STAGE) {
            const int ylo = max(0, s - R.w + 1), yhi = min(R.h - 1, s);
            constexpr int GR = NITF < 4 ? NITF : 4;  // passes per LDS round trip (registers)
#pragma unroll
            for (int i0 = 0; i0 < NITF; i0 += GR) {
                u32x4 v[GR];
#pragma unroll
                for (int k = 0; k < GR; ++k)
                    if (i0 + k < NITF) {
                        const int cell = min(max(fc0 + (i0 + k) * RPF, ylo), yhi);
                        if constexpr (P == 3) v[k] = dzs[DB ? s & 1 : 0][cell][fr];
                        else v[k] = reinterpret_cast<const u32x4*>(&dap[DB ? s & 1 : 0][0][cell][0])[fr];
                    }
#pragma unroll
                for (int k = 0; k < GR; ++k)
                    if (i0 + k < NITF) {
                        const int cell = min(max(fc0 + (i0 + k) * RPF, ylo), yhi);
                        *reinterpret_cast<u32x4*>(fbase + (int64_t)(M.sx * s + cell * M.ky) * ZROW) = v[k];
                    }
            }
        }
    };
    char* const sink = sink_ptr();

    // Phase A of tile lt: da of the lane's units. `far` holds the unstaged inputs.
    auto cells = [&](int s, int lt, const Set& in, const float (&gtv)[WQ], const float (&dtv)[WQ]) {
        const int ylo = max(0, s - R.w + 1), yhi = min(R.h - 1, s);
        const int yy = 16 * (tg * TPG + lt) + n16;
        const u32x4* row = &ist[DB ? s & 1 : 0][STAGE ? yy * PB : 0];
        const bool inr = yy >= ylo && yy <= yhi;
        typename V::R gr[5], dyr;
        typename Vec<float, WQ>::R clr, ctr;
        if constexpr (STAGE) {
#pragma unroll
            for (int t = 0; t < 5; ++t) gr[t] = ldw<T, WQ>(reinterpret_cast<const T*>(row) + t * H + u0);
            dyr = ldw<T, WQ>(reinterpret_cast<const T*>(row + QZ) + u0);
            clr = ldw<float, WQ>(reinterpret_cast<const float*>(row + QZ + QY) + u0);
            const u32x4* up = yy > 0 ? row - PB : row;
            ctr = ldw<float, WQ>(reinterpret_cast<const float*>(up + QZ + QY) + u0);
        } else {
#pragma unroll
            for (int t = 0; t < 5; ++t) gr[t] = in.g[lt][t];
            dyr = in.dy[lt];
            clr = in.cl[lt];
            ctr = in.ct[lt];
        }
        const bool hasl = s - yy > 0, hast = yy > 0;
        float da[5][WQ];
#pragma unroll
        for (int r = 0; r < WQ; ++r) {
            const float gi = V::get(gr[0], r), gfl = V::get(gr[1], r), gft = V::get(gr[2], r), go = V::get(gr[3], r),
                        gg = V::get(gr[4], r);
            const bool live = inr && !(gi < 0.0f);  // a NaN stays
            const float cl = Vec<float, WQ>::get(clr, r), cu = Vec<float, WQ>::get(ctr, r);
            const float cL = hasl ? cl : 0.0f, cT = hast ? cu : 0.0f;
            const float dh = V::get(dyr, r) + gl[lt][r] + gtv[r];
            const float tc = MEM ? tanhf(co[lt][r]) : tanh_fast(co[lt][r]);
            const float dc = dcl[lt][r] + dtv[r] + dh * go * (1.0f - tc * tc);
            co[lt][r] = cl;
            da[0][r] = live ? dc * gg * gi * (1.0f - gi) : 0.0f;
            da[1][r] = live ? dc * cL * gfl * (1.0f - gfl) : 0.0f;
            da[2][r] = live ? dc * cT * gft * (1.0f - gft) : 0.0f;
            da[3][r] = live ? dh * tc * go * (1.0f - go) : 0.0f;
            da[4][r] = live ? dc * gi * (1.0f - gg * gg) : 0.0f;
            if constexpr (P == 3) {
#pragma unroll
                for (int t = 0; t < 5; ++t) dmax = fmaxf(dmax, fabsf(da[t][r]));
            }
            dcl[lt][r] = live ? dc * gfl : 0.0f;
            dct[lt][r] = live ? dc * gft : 0.0f;
        }
        const int b = DB ? s & 1 : 0;
        if constexpr (P == 3) {
#pragma unroll
            for (int r = 0; r < WQ; ++r) {
                uint32_t lo[3], hi[3];
                split2(da[0][r], da[1][r], lo);
                split2(da[2][r], da[3][r], hi);
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    *reinterpret_cast<u32x2*>(&dap[b][k][yy][4 * (u0 + r)]) = u32x2{lo[k], hi[k]};
            }
            uint32_t p0[3], p1[3];
            split2(da[4][0], WQ > 1 ? da[4][WQ > 1 ? 1 : 0] : 0.0f, p0);
            if constexpr (WQ == 4) split2(da[4][2], da[4][3], p1);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                bf16_t* p = &dap[b][k][yy][4 * H + u0];
                if constexpr (WQ == 4) *reinterpret_cast<u32x2*>(p) = u32x2{p0[k], p1[k]};
                else if constexpr (WQ == 2) *reinterpret_cast<uint32_t*>(p) = p0[k];
                else *p = (bf16_t)p0[k];
            }
            if constexpr (STAGE) {
#pragma unroll
                for (int t = 0; t < 5; ++t)
                    stw<float, WQ>(reinterpret_cast<float*>(&dzs[b][yy][0]) + t * H + u0, da[t]);
            }
        } else {
#pragma unroll
            for (int t = 0; t < 5; ++t) stw<T, WQ>(&dap[b][0][yy][t * H + u0], da[t]);
        }
        if constexpr (!STAGE) {
            T* const zp = inr ? zb + (int64_t)(M.sx * s + yy * M.ky) * (4 * G) + u0 : reinterpret_cast<T*>(sink);
#pragma unroll
            for (int t = 0; t < 5; ++t) stw<T, WQ>(zp + t * H, da[t]);
        }
    };
    auto step = [&](int s, Set& far) {
        // From the top: a tile's bottom edge is the first row of the tile
        // below it, of the previous diagonal.
#pragma unroll
        for (int lt = 0; lt < TA; ++lt) {
            float gtv[WQ], dtv[WQ];
#pragma unroll
            for (int r = 0; r < WQ; ++r) {
                float eg = 0.0f, ed = 0.0f;
                if (lt + 1 < TA) {
                    eg = first_to_last(gt[lt + 1 < TA ? lt + 1 : 0][r]);
                    ed = first_to_last(dct[lt + 1 < TA ? lt + 1 : 0][r]);
                } else if (NG > 1 && TA == TPG && tg + 1 < NG) {
                    eg = gedge[tg + 1 < NG ? tg + 1 : 0][u0 + r];
                    ed = dedge[(s & 1) ^ 1][tg + 1 < NG ? tg + 1 : 0][u0 + r];
                }
                gtv[r] = row_below(gt[lt][r], eg);
                dtv[r] = row_below(dct[lt][r], ed);
            }
            cells(s, lt, far, gtv, dtv);
            if constexpr (!STAGE) load_tile(s - 1, lt, far);
            if constexpr (NG > 1) {
                if (lt == 0 && n16 == 0) {
#pragma unroll
                    for (int r = 0; r < WQ; ++r) dedge[s & 1][tg][u0 + r] = dct[0][r];
                }
            }
        }
        lds_barrier();  // da of the diagonal written
#pragma unroll
        for (int lt = 0; lt < TA; ++lt) {
            const int yy = 16 * (tg * TPG + lt) + n16;
            floatx4 acc[OT], low[OT];
#pragma unroll
            for (int t = 0; t < OT; ++t) acc[t] = low[t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                bf16x8 b[P];
#pragma unroll
                for (int k = 0; k < P; ++k)
                    b[k] = as_bf16x8(*reinterpret_cast<const uint4*>(&dap[DB ? s & 1 : 0][k][yy][32 * ks + 8 * q]));
                mma_tiles<P, OT>(A, ks, b, acc, low);
            }
#pragma unroll
            for (int o = 0; o < K::OUTS; ++o) {
                const float v = P == 3 ? acc[o >> 2][o & 3] + low[o >> 2][o & 3] : acc[o >> 2][o & 3];
                if (o < WQ) gl[lt][o % WQ] = v;
                else if (o < 2 * WQ) gt[lt][o % WQ] = P == 3 ? -v : v;
                else if (o < 3 * WQ) dcl[lt][o % WQ] += v;  // the states' share of dc
                else dct[lt][o % WQ] += P == 3 ? -v : v;
            }
            if constexpr (NG > 1) {
                if (lt == 0 && n16 == 0) {
#pragma unroll
                    for (int r = 0; r < WQ; ++r) gedge[tg][u0 + r] = gt[0][r];
                }
            }
        }
        flush(s);
        stage_in(s - NB, far);
        if constexpr (STAGE) load(s - NB - 2, far);
        if constexpr (!DB) lds_barrier();
    };

    Set s0, s1;
    if constexpr (STAGE) {
        load(steps - 1, s0);
        stage_in(steps - 1, s0);
        if constexpr (DB) {
            load(steps - 2, s1);
            stage_in(steps - 2, s1);
        }
        load(steps - 1 - NB, s0);
        load(steps - 2 - NB, s1);
    } else {
#pragma unroll
        for (int lt = 0; lt < TA; ++lt) load_tile(steps - 1, lt, s0);
    }
    lds_barrier();
    if (P == 3 && wmax > BF16_LARGEST) plain = 1;
    // two steps ahead of the loop: it is entered with the memory operations in
    // flight that its own steps leave, so its waits are exact
    int s = steps - 1;
    step(s, s0);
    if (--s >= 0) {
        step(s, STAGE ? s1 : s0);
        --s;
    }
    while (s >= 0) {
        step(s, s0);
        if (--s < 0) break;
        step(s, STAGE ? s1 : s0);
        --s;
    }
    if constexpr (P == 3) {
        if (dmax > BF16_LARGEST) plain = 1;
        lds_barrier();
        if (__builtin_amdgcn_readfirstlane(plain))
            plain_bwd_unit<H, MEM>(kern_args<BwdArgs>(), unit, reinterpret_cast<float*>(&dap[0][0][0][0]), NT * 16);
    }
}

template <int H, int NT, typename T, int WQ, int NG, bool MEM>
__global__ void __launch_bounds__((BwdK<H, NT, T, WQ, NG, MEM>::NTH))
__attribute__((amdgpu_waves_per_eu(BwdK<H, NT, T, WQ, NG, MEM>::WPE))) k_bwd(BwdArgs a) {
    using K = BwdK<H, NT, T, WQ, NG, MEM>;
    if constexpr (NT == 1) {
        for_units(a, [&](int unit) { bwd_unit<H, NT, T, WQ, NG, MEM, 1>(a, unit); });
    } else {
        for_units(a, [&](int unit) {
            const int rows = reinterpret_cast<const RectD*>(a.rects)[unit >> 2].h;
            const int tg = NG == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) / K::NWU;
            with_tiles<K::TPG, NG == 1 ? 1 : 0>((rows + 15) / 16 - tg * K::TPG, [&](auto ta) {
                bwd_unit<H, NT, T, WQ, NG, MEM, decltype(ta)::value>(a, unit);
            });
        });
    }
}

template <int H, int NT, typename T, int WQ, int NG, bool MEM = false>
WaveKernel bwd_kernel() {
    static_assert(BwdK<H, NT, T, WQ, NG, MEM>::FITS, "LDS");
    return {reinterpret_cast<const void*>(&k_bwd<H, NT, T, WQ, NG, MEM>), BwdK<H, NT, T, WQ, NG, MEM>::NTH};
}

// One translation unit per hidden size (k_wave_bwd_*.hip).
WaveKernel bwd_kernel_f32_h4(int nt);
WaveKernel bwd_kernel_f32_h8(int nt);
WaveKernel bwd_kernel_f32_h16(int nt);
WaveKernel bwd_kernel_f32_h32(int nt);
WaveKernel bwd_kernel_f32_h64(int nt);
WaveKernel bwd_kernel_bf16_h32(int nt);
WaveKernel bwd_kernel_bf16_h64(int nt);
WaveKernel bwd_kernel_mem_h16(int nt);
WaveKernel bwd_kernel_mem_h32(int nt);

}  // namespace mdl
