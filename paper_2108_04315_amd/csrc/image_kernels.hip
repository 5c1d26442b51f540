// image_kernels.hip -- gfx950 image kernels of the MISR SCG hot path, for one
// scale factor S (compiled once per S with -DMISR_SCALE=S).
//
// Work decomposition: every kernel walks a work list of (view, tile) items;
// a tile is TH x TW owned HR pixels.  A 512-thread workgroup stages the tile's
// window (owned pixels plus EXT = max(L-1, 2) on each side) into LDS once and
// runs every frame's separable band passes from there:
//
//   forward  A_k x  : pass 1 along rows    (HR rows -> LR columns, L taps, stride S)
//                     pass 2 along columns (HR rows -> LR rows,    L taps, stride S)
//   adjoint A_k^T r : pass 3 along columns (LR rows -> HR rows, ceil(L/S) taps)
//                     pass 4 along rows    (LR cols -> HR cols)
//
// A_k = C_y,k (x) C_x,k holds exactly because the warp, the PSF and the
// binning of the observation model (Sec. 3.1, Eq. sisr) are all separable,
// zero padding included, so each 2-D operator becomes two 1-D banded ones.
// Each wave runs whole strips of an operator (pass 1 and 2 of its own LR
// columns, pass 3 and 4 of its own HR columns), so that its passes follow each
// other in its own LDS without a workgroup barrier; only the residual crosses
// waves (one barrier per frame).  The weights of all rows and columns away
// from the image edge are the same L numbers per frame and axis: a frame's
// 2 L weights sit in scalar registers.  What bounds the passes is the latency
// of their chain (LDS round trips, barriers, scalar loads) and VALU issue: one
// barrier instead of four per frame and no per-row weight loads took the
// standalone adjoint of 9 frames of 1024^2 at x3 from 157 to 98 us, k_trial
// from 64.6 to 56.6 us at 2048^2 x2 (4 frames) and from 779 to 569 us at
// 6144^2 x3 (9 frames).
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "device_common.h"
#include "pass_end.h"

#ifndef MISR_SCALE
#error "compile with -DMISR_SCALE=<s>"
#endif

namespace misr {

constexpr int kNTI = 512;          // threads per workgroup of the image kernels
constexpr int kNWI = kNTI / 64;    // waves per workgroup

// Tile shapes: variant 0 is the widest tile for which one 64-lane wave spans
// every tile dimension a pass maps to lanes and two workgroups fit a CU's LDS
// in both the trial and the update pass; variant 1 is about half as wide;
// variant 2 is a trial-kernel shape as wide as the trial pass's LDS alone
// allows (the update pass stages two windows), paired with variant 0's
// update shape; kNarrow is the narrow tile that variant 0's kernels run for
// small images.
constexpr int ceil_div(int a, int b) { return (a + b - 1) / b; }
constexpr int odd(int v) { return (v % 2) ? v : v + 1; }

// A wave's strip of a forward over NI x NJ LR pixels: pass 1 gives every
// wave CJ neighbouring LR columns (lanes on HR rows), pass 2 lays the strip's
// CI-row blocks x CJ columns over the lanes.
template <int S, int L, int NI, int NJ>
struct Strip {
    static constexpr int CJ = ceil_div(NJ, kNWI);
    static constexpr int calc_ci() {
        int ci = 1;
        while (ceil_div(NI, ci) * CJ > 64) ++ci;
        return ci;
    }
    static constexpr int CI = calc_ci();
    static constexpr int NIB = ceil_div(NI, CI);
    static constexpr int HS = 65;   // column stride of the wave's pass-1 output
    static constexpr int rows = S * (NIB * CI - 1) + L;
    static constexpr int LDS = (CJ - 1) * HS + (rows > 64 ? rows : 64);
};

template <int S, int L, int TV>
struct Tile {
    static constexpr int EXT = (L - 1 > 2) ? L - 1 : 2;   // window margin (HR px)
    static constexpr int NTAP = (L + S - 1) / S;         // adjoint taps per output
    static constexpr int calc_th() {
        int best = S;
        for (int th = S; th + 2 <= 64; th += S)
            if (S * ((th + L - 2) / S) + L <= 64) best = th;
        return best;
    }
    static constexpr int TH = calc_th();
    static constexpr int NIM = (TH + L - 2) / S + 1;     // LR rows touching the tile
    static constexpr int NRM = S * (NIM - 1) + L;        // HR rows those read
    // LDS floats by which the tile's width is chosen: a window, one LR row
    // set in pass-1 and residual form, and the owned p (trial pass), or two
    // windows (update pass, unless the shape is the trial kernel's own)
    static constexpr int shape_floats(int tw) {
        const int wcp = odd(tw + 2 * EXT);
        const int njp = odd((tw + L - 2) / S + 1);
        const int xs = (TH + 2 * EXT) * wcp + S * 4 + 8;
        const int hx = NRM * njp + S * 4 * njp;
        const int hr = hx + NIM * njp;
        const int gs = TH * (tw + 1);
        const int trial = xs + (hr > gs ? hr : gs) + TH * tw;
        const int upd = 2 * xs + hx + NIM * njp;
        return (TV == 2 || trial > upd) ? trial : upd;
    }
    static constexpr int calc_tw() {
        int best = kNWI * S;
        for (int tw = kNWI * S; tw <= 1024; tw += kNWI * S)
            if ((tw + L - 2) / S + 1 <= 64 && shape_floats(tw) * 4 <= 79 * 1024) best = tw;
        // variant 1: about half as wide (more workgroups for small images);
        // the narrow tile: two columns per wave and phase at scale 2, else as
        // variant 1
        const int half = best / 2 / (kNWI * S) * (kNWI * S);
        if (TV == 1 || TV == kNarrow) best = half > kNWI * S ? half : kNWI * S;
        if (TV == kNarrow && S == 2) best = 2 * kNWI * S;
        return best;
    }
    static constexpr int TW = calc_tw();
    static constexpr int WR = TH + 2 * EXT, WC = TW + 2 * EXT, WCP = odd(WC);
    static constexpr int NJM = (TW + L - 2) / S + 1;     // LR columns touching the tile
    static constexpr int CV = TW / kNWI;                 // pass 4 / prior columns per wave
    using FT = Strip<S, L, NIM, NJM>;                    // the trial's forward
    using FU = Strip<S, L, TH / S, TW / S>;              // forward of the owned LR pixels
    // adjoint strip: the CV columns of a wave gather from at most NJG LR
    // columns; pass 3 lays those x NUB blocks of CU rows over the lanes
    static constexpr int NJG = (S - 1 + CV - 1) / S + NTAP;
    static constexpr int CU = ceil_div(ceil_div(TH, 64 / NJG), S) * S;
    static constexpr int NUB = ceil_div(TH, CU);
    static constexpr int TS = odd(NUB * CU);             // column stride of pass 3's output
    static constexpr int XS = WR * WCP + S * kNWI * FT::CJ + 8;
    static constexpr int PWT = FT::LDS > NJG * TS ? FT::LDS : NJG * TS;   // per wave, trial
    static constexpr int RP = kNWI * FT::CJ + 1;         // row stride of the residual
    static constexpr int RSR = FT::NIB * FT::CI > NIM ? FT::NIB * FT::CI : NIM;
    static constexpr int RSS = RSR * RP;                 // one residual buffer of two
    static constexpr int RSX = ((NUB * CU - TH) / S + 2) * RP;   // rows the padded blocks read
    static constexpr int GP = TW + 1;                    // row stride of the LDS gradient
    static constexpr int BANDS = kNWI * PWT + 2 * RSS + RSX;
    static constexpr int PO = XS + (BANDS > TH * GP ? BANDS : TH * GP);
    // the owned p stays in LDS where two workgroups per CU still fit, else
    // the output re-reads it
    static constexpr bool POL = (PO + TH * TW) * 4 <= 79 * 1024;
    static constexpr int SMEM = PO + (POL ? TH * TW : 0);
    static constexpr int SMEM_U = 2 * XS + kNWI * FU::LDS;          // update pass
    static constexpr int SMEM_F = XS + kNWI * FU::LDS;              // standalone forward
    static constexpr int SMEM_A = XS + kNWI * PWT + 2 * RSS + RSX;  // standalone adjoint
    static_assert(NRM <= 64 && TH + 2 <= 64 && NJM <= 64 && NJG <= 64, "a wave spans a dimension");
    static_assert(CV % S == 0 && CU % S == 0, "phase-aligned groups");
    static_assert(TH * GP <= XS, "the standalone adjoint's output tile");
    static_assert(SMEM * 4 <= 81408 && (TV == 2 || SMEM_U * 4 <= 81408), "two workgroups per CU");
};

// Orders a wave's LDS writes before its own lanes' later reads: DS operations
// of one wave complete in order, so only the compiler has to keep them so.
FI void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One frame's band weights along one axis.  Every LR row whose taps are not
// cut by the image edge has the same L weights, c (scalar registers for a
// whole frame); rows outside [lo, hi) (a few at either edge) take theirs from
// the table, whose row -1 and row n are zero.
template <int L>
struct AxisW {
    float c[L];
    int lo, hi, n;
    const AS4 float *tab;
    // some LR row of [i, i + m) has weights of its own (uniform)
    FI bool special(int i, int m) const {
        return max(i, 0) < min(i + m, lo) || max(i, hi) < min(i + m, n);
    }
    FI const AS4 float *row(int i) const { return tab + min(max(i, -1), n) * L; }
};
template <int L>
FI AxisW<L> axis_y(const AS4 OpDev &op, int k) {
    AxisW<L> a;
#pragma unroll
    for (int l = 0; l < L; ++l) a.c[l] = op.cwy[k][l];
    a.lo = op.loy[k];
    a.hi = op.hiy[k];
    a.n = op.H / op.s;
    a.tab = cst(op.wy) + (i64)k * op.fsy * L;
    return a;
}
template <int L>
FI AxisW<L> axis_x(const AS4 OpDev &op, int k) {
    AxisW<L> a;
#pragma unroll
    for (int l = 0; l < L; ++l) a.c[l] = op.cwx[k][l];
    a.lo = op.lox[k];
    a.hi = op.hix[k];
    a.n = op.W / op.s;
    a.tab = cst(op.wx) + (i64)k * op.fsx * L;
    return a;
}

// A wave's strip of the forward: the NI LR rows from i0 at the CJ LR columns
// from j0 + CJ wv.  win: the window at the first tap of LR pixel (i0, j0).
//   pass 1 (lanes on HR rows): hx[c][r] = sum_l wx[j][l] win[r][S (CJ wv + c) + l]
//   pass 2 (lanes on CI-row blocks x columns): sum_l wy[i][l] hx[c][S i + l]
// Both passes of a strip belong to one wave, so nothing but that wave's own
// LDS order separates them (no workgroup barrier), and every frame's weights
// are the same scalars for all rows and columns away from the image edge.
// out(i, c, v[CI]): the results of LR rows i.. of the strip's column c.
template <int S, int L, class G, class F>
FI void fwd_strip(const float *win, int wcp, float *hx, const AxisW<L> &ay, const AxisW<L> &ax,
                  int i0, int j0, int lane, int wv, F out) {
    constexpr int CJ = G::CJ, CI = G::CI, NX = S * (CJ - 1) + L, NH = S * (CI - 1) + L;
    const int jw = j0 + CJ * wv;
    {
        const float *src = win + lane * wcp + S * CJ * wv;
        float xv[NX];
#pragma unroll
        for (int t = 0; t < NX; ++t) xv[t] = src[t];
        if (!ax.special(jw, CJ)) {
#pragma unroll
            for (int c = 0; c < CJ; ++c) {
                float a = 0.f;
#pragma unroll
                for (int l = 0; l < L; ++l) a = fmaf(ax.c[l], xv[S * c + l], a);
                hx[c * G::HS + lane] = a;
            }
        } else {
#pragma unroll
            for (int c = 0; c < CJ; ++c) {
                const AS4 float *wb = ax.row(jw + c);
                float a = 0.f;
#pragma unroll
                for (int l = 0; l < L; ++l) a = fmaf(wb[l], xv[S * c + l], a);
                hx[c * G::HS + lane] = a;
            }
        }
    }
    wave_lds_order();
    const int ib = lane / CJ, cj = lane - ib * CJ;
    if (ib < G::NIB) {
        const float *src = hx + cj * G::HS + S * CI * ib;
        float hv[NH], av[CI];
#pragma unroll
        for (int t = 0; t < NH; ++t) hv[t] = src[t];
        if (!ay.special(i0, G::NIB * CI)) {
#pragma unroll
            for (int c = 0; c < CI; ++c) {
                float a = 0.f;
#pragma unroll
                for (int l = 0; l < L; ++l) a = fmaf(ay.c[l], hv[S * c + l], a);
                av[c] = a;
            }
        } else {
#pragma unroll
            for (int c = 0; c < CI; ++c) {
                const AS1 float *wb = (const AS1 float *)ay.row(i0 + ib * CI + c);
                float a = 0.f;
#pragma unroll
                for (int l = 0; l < L; ++l) a = fmaf(wb[l], hv[S * c + l], a);
                av[c] = a;
            }
        }
        out(ib * CI, cj, av);
    }
    wave_lds_order();
}

// A wave's strip of the adjoint, pass 3: tt[j][u] = sum_i wy[i][U - S i - offy]
// rs[i][j] for the NJG LR columns its CV HR columns gather from (lanes on
// columns x blocks of CU rows).  PH = (U0 - offy) mod S fixes every tap
// offset at compile time.  rs holds the tile's LR rows and columns from
// (iF, jF) on, zero outside the image; LR columns shared by neighbouring
// waves are computed by each of them.
template <int S, int L, int TV, int PH>
FI void pass3_ph(const float *rs, float *tt, int U0, int offy, int iF, int jrel,
                 const AxisW<L> &ay, int lane) {
    using T = Tile<S, L, TV>;
    constexpr int CU = T::CU, NTAP = T::NTAP;
    constexpr int NIG = (PH + CU - 1) / S + NTAP;
    const int ub = lane / T::NJG, cj = lane - ub * T::NJG;
    if (ub >= T::NUB) return;
    const int ib = (U0 - offy - PH) / S - (NTAP - 1) + ub * (CU / S);   // (an exact division)
    const float *src = rs + (ib - iF) * T::RP + jrel + cj;
    float rv[NIG];
    // LR row t contributes to row c of the block through tap PH + c + S (NTAP - 1 - t)
#pragma unroll
    for (int t = 0; t < NIG; ++t)
        rv[t] = (PH + S * (NTAP - 1 - t) < L) ? src[t * T::RP] : 0.f;
    float *dst = tt + cj * T::TS + ub * CU;
    if (!ay.special(iF - 1, T::RSR + (T::NUB * CU - T::TH) / S + 2)) {
#pragma unroll
        for (int c = 0; c < CU; ++c) {
            const int dq = (PH + c) / S, ph = (PH + c) % S;
            float a = 0.f;
#pragma unroll
            for (int m = 0; m < NTAP; ++m)
                if (ph + S * m < L) a = fmaf(ay.c[ph + S * m], rv[dq - m + NTAP - 1], a);
            dst[c] = a;
        }
    } else if constexpr (S > 1) {
        // tap by tap (by rows, as below, a tiled 4096^2 solve at scale 2 took
        // 28.3 ms instead of 28.05, the adjoint of 9 frames of 1024^2 at scale 3
        // 62.7 us instead of 62.3)
#pragma unroll
        for (int c = 0; c < CU; ++c) {
            const int dq = (PH + c) / S, ph = (PH + c) % S;
            float a = 0.f;
#pragma unroll
            for (int m = 0; m < NTAP; ++m)
                if (ph + S * m < L) {
                    const AS1 float *wb = (const AS1 float *)ay.row(ib + dq - m + NTAP - 1);
                    a = fmaf(wb[ph + S * m], rv[dq - m + NTAP - 1], a);
                }
            dst[c] = a;
        }
    } else {
        // row by row from the last, the order of the sums above: a row's taps
        // are neighbours in the table, and four rows' loads are in flight
        // together.  (Tap by tap, the loads of band 16 spilled 90 registers of the
        // trial kernel: cost and gradient of 16 frames of 33 x 20 took 134 us, now
        // 106.)
        constexpr int G = 4;
        float a[CU];
#pragma unroll
        for (int c = 0; c < CU; ++c) a[c] = 0.f;
#pragma unroll
        for (int t1 = NIG - 1; t1 >= 0; t1 -= G) {
            float wv[G][CU];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int t = t1 - g;
                if (t < 0) break;
                const AS1 float *wb = (const AS1 float *)ay.row(ib + t);
#pragma unroll
                for (int c = 0; c < CU; ++c) {
                    const int l = PH + c + S * (NTAP - 1 - t);
                    wv[g][c] = l >= 0 && l < L ? wb[l] : 0.f;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int t = t1 - g;
                if (t < 0) break;
#pragma unroll
                for (int c = 0; c < CU; ++c) {
                    const int l = PH + c + S * (NTAP - 1 - t);
                    if (l >= 0 && l < L) a[c] = fmaf(wv[g][c], rv[t], a[c]);
                }
            }
        }
#pragma unroll
        for (int c = 0; c < CU; ++c) dst[c] = a[c];
    }
}

// Pass 4: g[u][v] += sum_j wx[j][V - S j - offx] tt[j][u] for the wave's CV
// columns; lanes take rows (u = lane - 2).  jb: the LR column of tt's first.
template <int S, int L, int TV, int PH>
FI void pass4_ph(const float *tt, float (&gacc)[Tile<S, L, TV>::CV], int jb, const AxisW<L> &ax,
                 int lane) {
    using T = Tile<S, L, TV>;
    constexpr int CV = T::CV, NTAP = T::NTAP;
    constexpr int NJG = (PH + CV - 1) / S + NTAP;
    const int ur = min(max(lane - 2, 0), T::TH - 1);
    float tv[NJG];
#pragma unroll
    for (int t = 0; t < NJG; ++t) tv[t] = tt[t * T::TS + ur];
    if (!ax.special(jb, NJG)) {
#pragma unroll
        for (int c = 0; c < CV; ++c) {
            const int dq = (PH + c) / S, ph = (PH + c) % S;
            float a = 0.f;
#pragma unroll
            for (int m = 0; m < NTAP; ++m)
                if (ph + S * m < L) a = fmaf(ax.c[ph + S * m], tv[dq - m + NTAP - 1], a);
            gacc[c] += a;
        }
    } else {
#pragma unroll
        for (int c = 0; c < CV; ++c) {
            const int dq = (PH + c) / S, ph = (PH + c) % S;
            float a = 0.f;
#pragma unroll
            for (int m = 0; m < NTAP; ++m)
                if (ph + S * m < L)
                    a = fmaf(ax.row(jb + dq - m + NTAP - 1)[ph + S * m], tv[dq - m + NTAP - 1], a);
            gacc[c] += a;
        }
    }
}

// Runs f with the phase ph in [0, S) as a compile-time constant (uniform).
template <int S, class F>
FI void by_phase(int ph, F f) {
    if (ph == 0) f(std::integral_constant<int, 0>{});
    if constexpr (S > 1) if (ph == 1) f(std::integral_constant<int, 1>{});
    if constexpr (S > 2) if (ph == 2) f(std::integral_constant<int, 2>{});
    if constexpr (S > 3) if (ph == 3) f(std::integral_constant<int, 3>{});
}

// One frame's adjoint of the residual rs (rows and columns from (iF, jF)) into
// the wave's CV columns; tt: the wave's own LDS.
template <int S, int L, int TV>
FI void adj_strip(const float *rs, float *tt, float (&gacc)[Tile<S, L, TV>::CV], int U0, int V0,
                  int offy, int offx, int iF, int jF, const AxisW<L> &ay, const AxisW<L> &ax,
                  int lane, int wv) {
    using T = Tile<S, L, TV>;
    const int jb = fdiv(V0 + wv * T::CV - offx, S) - (T::NTAP - 1);
    by_phase<S>(pmod(U0 - offy, S), [&](auto ph) {
        pass3_ph<S, L, TV, decltype(ph)::value>(rs, tt, U0, offy, iF, jb - jF, ay, lane);
    });
    wave_lds_order();
    by_phase<S>(pmod(V0 - offx, S), [&](auto ph) {
        pass4_ph<S, L, TV, decltype(ph)::value>(tt, gacc, jb, ax, lane);
    });
    wave_lds_order();
}

// The 8 BTV offsets d = (dx, dy) in [0, 2]^2 minus the origin (Eq. prior, w = 3).
__device__ constexpr int kDX[8] = {1, 2, 0, 1, 2, 0, 1, 2};
__device__ constexpr int kDY[8] = {0, 0, 1, 1, 1, 2, 2, 2};

// BTV prior on the window, swept left to right over the wave's CV columns
// with lanes on rows (u = lane - 2, two rows of halo).  Each pair (i, i+d)
// is evaluated once, by the lane of i; the pixel i+d takes the share back
// from the same lane's history (same row, dx columns earlier) or, for rows
// below, from the lane dy above through DPP lane shifts of the per-dy sums.
// The 3-column window and the 2-step history rotate through three register
// slots, so the loop is unrolled by three and nothing is moved.  Steps 0
// and 1 (columns cv0-2, cv0-1) only fill the history.  The gradient
// accumulates into gs (LDS, row stride GP).
//
// Rounding of a pixel's sums: the shares gamma_d psi(z_d) = g z are rounded
// products, except that in interior tiles (CHECK = false) a share that enters
// a single sum of its wave's strip is fused into it: the shares from the two
// columns before the strip (first column), and the shares whose partner lies
// past the strip (last one or two columns).  The narrow tile rounds as the
// wide one does, so that results do not depend on which of them a pixel falls
// into: cw0 is the strip's first column within the strips of variant 0.  (But
// for a strip of scale 1 across two wide tiles of which the edge cuts one: all
// of it rounds as at the edge.)
template <int S, int L, int TV, bool EPS0, bool CHECK>
FI void btv_sweep(const float *xs, float *gs, const float (&gam)[8], float eps, int U0, int V0,
                  int H, int W, int th_own, int tw_own, int cw0, double &e_reg) {
#pragma clang fp contract(off)
    using T = Tile<S, L, TV>;
    constexpr bool NAR = TV == kNarrow;
    constexpr int CV = T::CV, NSTEP = CV + 2;
    // the strips whose edges fix the rounding: CVW columns, the last FL fused
    constexpr int CVW = NAR ? Tile<S, L, 0>::CV : CV, FL = (CVW + 2) % 3;
    const int lane = threadIdx.x & 63, wv = uni(threadIdx.x >> 6);
    const int u = lane - 2;
    const int cv0 = wv * CV;
    const int U = U0 + u;
    const int ur = min(u, T::TH - 1);
    const float e2 = eps * eps;
    const bool row_tile = u >= 0 && u < T::TH;
    const bool own_row = u >= 0 && u < (CHECK ? th_own : T::TH);
    // pair validity per row offset (both pixels inside the image)
    bool rok[3];
#pragma unroll
    for (int dy = 0; dy < 3; ++dy) rok[dy] = !CHECK || (U >= 0 && U + dy < H);
    const float *base = xs + (T::EXT + ur) * T::WCP + T::EXT + cv0 - 2;
    float *grow = gs + max(u, 0) * T::GP + cv0 - 2;
    float win[3][3];    // win[dy][slot]: window column c (from cv0 - 2) sits in slot (c + 1) % 3
    float hist[3][8];   // hist[slot][d]: the step's lambda gamma_d psi(z_d), slot t % 3
    float hz[3][8], hg[3][8];   // its factors
#pragma unroll
    for (int dy = 0; dy < 3; ++dy) {
        win[dy][1] = base[dy * T::WCP + 0];
        win[dy][2] = base[dy * T::WCP + 1];
    }
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int d = 0; d < 8; ++d) hist[q][d] = 0.f;
    float gam_sum = 0.f;
#pragma unroll
    for (int d = 0; d < 8; ++d) gam_sum += gam[d];
    double eacc = 0.0;
    // step t handles column cv0 + t - 2 and loads window column t + 2 (slot
    // t % 3); FIRST: fused shares from the columns before, LAST: shares with
    // dx >= LAST fused into the pixel's own sum
    auto step = [&](auto slot_c, auto out_c, int t, auto kind) {
#pragma clang fp contract(off)
        constexpr int Q = decltype(slot_c)::value;
        constexpr bool OUT = decltype(out_c)::value;
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) win[dy][Q] = base[dy * T::WCP + t + 2];
        const int v = cv0 + t - 2, V = V0 + v;
        bool cok[3];
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) cok[dx] = !CHECK || (V >= 0 && V + dx < W);
        const float x0 = win[0][(Q + 1) % 3];
        // the prior's cost of the column; for interior tiles (every pair
        // valid) the sum of gamma_d B_d, B_d = |(z_d, eps)|, less eps times
        // the sum of the gamma_d, which shares gamma_d / B_d with the gradient
        float eb = 0.f;
#pragma unroll
        for (int d = 0; d < 8; ++d) {
            const int dx = kDX[d], dy = kDY[d];
            const float z = x0 - win[dy][(Q + 1 + dx) % 3];
            if (EPS0) {
                const float ps = (z > 0.f) ? 1.f : ((z < 0.f) ? -1.f : 0.f);
                const bool valid = rok[dy] && cok[dx];
                hist[Q][d] = valid ? gam[d] * ps : 0.f;
                eb = fmaf(valid ? gam[d] : 0.f, fabsf(z), eb);
            } else if (CHECK) {
                const bool valid = rok[dy] && cok[dx];
                const float dd = fmaf(z, z, e2);
                const float r = rsq(dd);
                hist[Q][d] = valid ? gam[d] * (z * r) : 0.f;
                eb = fmaf(valid ? gam[d] : 0.f, fmaf(dd, r, -eps), eb);
            } else {
                const float dd = fmaf(z, z, e2);
                const float gr = gam[d] * rsq(dd);
                hist[Q][d] = gr * z;
                hz[Q][d] = z;
                hg[Q][d] = gr;
                eb = fmaf(gr, dd, eb);
            }
        }
        if (!EPS0 && !CHECK) eb = fmaf(-eps, gam_sum, eb);
        if (OUT) {
            // shares of the pairs (i - d, i): from dx steps back, dy lanes up
            float own = 0.f, back[3] = {0.f, 0.f, 0.f};
            auto sums = [&](auto first_c, auto last_c) {
#pragma clang fp contract(off)
                constexpr bool FIRST = decltype(first_c)::value && !CHECK && !EPS0;
                constexpr int LAST = CHECK || EPS0 ? 3 : decltype(last_c)::value;
#pragma unroll
                for (int d = 0; d < 8; ++d) {
                    const int dx = kDX[d], dy = kDY[d];
                    own = dx >= LAST ? fmaf(hz[Q][d], hg[Q][d], own) : own + hist[Q][d];
                    const int P = (Q + 3 - dx) % 3;
                    back[dy] = FIRST && dx > 0 ? fmaf(hz[P][d], hg[P][d], back[dy])
                                               : back[dy] + hist[P][d];
                }
            };
            kind(sums);
            const float up = wave_shr1(back[1] + wave_shr1(back[2]));
            const float gsum = own - back[0] - up;
            if (row_tile) grow[t] += gsum;
            if (own_row && (!CHECK || v < tw_own)) eacc += (double)eb;
        }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;
    using F = std::false_type;
    using Tr = std::true_type;
    auto mid = [](auto sums) { sums(F{}, I3{}); };
    step(I0{}, F{}, 0, mid);
    step(I1{}, F{}, 1, mid);
    if constexpr (NAR) {
        // strips that start and end with variant 0's, or anywhere in them
        constexpr bool ALIGNED = CVW % CV == 0;
        auto at = [&](auto c_c) {
            constexpr int c = decltype(c_c)::value;
            step(std::integral_constant<int, (c + 2) % 3>{}, Tr{}, c + 2, [&](auto sums) {
                const int cw = cw0 + c >= CVW ? cw0 + c - CVW : cw0 + c;   // uniform
                constexpr bool HEAD = !ALIGNED || c == 0, TAIL = !ALIGNED || c >= CV - 2;
                if (HEAD && cw == 0)
                    sums(Tr{}, I3{});
                else if (TAIL && FL == 2 && cw == CVW - 2)
                    sums(F{}, I2{});
                else if (TAIL && FL >= 1 && cw == CVW - 1)
                    sums(F{}, I1{});
                else
                    sums(F{}, I3{});
            });
        };
        [&]<int... c>(std::integer_sequence<int, c...>) {
            (at(std::integral_constant<int, c>{}), ...);
        }(std::make_integer_sequence<int, CV>{});
    } else {
        step(I2{}, Tr{}, 2, [](auto sums) { sums(Tr{}, I3{}); });
#pragma unroll 1
        for (int t = 3; t + 2 < NSTEP; t += 3) {
            step(I0{}, Tr{}, t, mid);
            step(I1{}, Tr{}, t + 1, mid);
            step(I2{}, Tr{}, t + 2, mid);
        }
        // steps after the last full group of three
        if constexpr (FL == 1) step(I0{}, Tr{}, NSTEP - 1, [](auto sums) { sums(F{}, I1{}); });
        if constexpr (FL == 2) {
            step(I0{}, Tr{}, NSTEP - 2, [](auto sums) { sums(F{}, I2{}); });
            step(I1{}, Tr{}, NSTEP - 1, [](auto sums) { sums(F{}, I1{}); });
        }
    }
    e_reg += eacc;
}

// Curvature of the prior along p (Moller's step 2 without forming x + sk p):
// sum over owned pairs of gamma q^2 Q(z, sk q), z, q the pair differences of
// x and p; [ru0,ru1) x [rv0,rv1) is the owned part of the tile.  With eps > 0
// every pair first takes the first-order series of psi_quot, Q(z, h) =
// eps^2 / B^3 (1 - 3/2 h z / B^2), B = |(z, eps)|: in u = q / B the term is
// gamma eps^2 u^2 / B times (1 - 3/2 sk u z / B).  The next term of the series
// is at most 2 (h / B)^2 relative, so for |h| / B = sk |u| < kCurvTau = 1e-4
// the truncation stays below FP32 rounding; a pixel with a pair beyond that
// sums its pairs again, those beyond by psi_quot (its series; the closed form
// runs only where a pair needs it), so the common case takes one branch per
// pixel.
//
// VALU issue bounds the sweep (about 13 operations and a reciprocal root per
// pair).  A step takes NC neighbouring columns of NRB rows RS apart, NC NRB =
// 64, so that every lane owns a pixel (48 x 96 tile: 72 steps of 64 pixels;
// lanes on the 48 rows of one column took 96), and a pixel needs nothing from
// its neighbours but the LDS windows.  Images whose flat parts send half of
// the pixels beyond the series (128^2) recomputed the whole pixel with both
// branches of psi_quot before.  k_upcurv: 49.9 ->
// 45.1 us at 2048^2, 25.0 -> 21.1 us at 128^2 (six tiles, one per CU).
template <int S, int L, int TV, bool CHECK, bool EPS0>
FI void curv_sweep(const float *xs, const float *ps, const float (&gam)[8], float eps, float sk,
                   int U0, int V0, int H, int W, int ru0, int ru1, int rv0, int rv1,
                   double &dreg) {
    using T = Tile<S, L, TV>;
    constexpr int NC = T::TW % 32 == 0 ? 32 : (T::TW % 16 == 0 ? 16 : 8), NRB = 64 / NC;
    constexpr int RS = ceil_div(T::TH, NRB), NST = T::TW / NC * RS, SPW = ceil_div(NST, kNWI);
    static_assert(T::TW % NC == 0, "whole column groups");
    const int lane = threadIdx.x & 63, wv = uni(threadIdx.x >> 6);
    const int cl = lane % NC, ul = lane / NC * RS;
    const float e2 = eps * eps;
    float gq[8];   // gamma_d eps^2
#pragma unroll
    for (int d = 0; d < 8; ++d) gq[d] = gam[d] * e2;
    constexpr float kCurvTau = 1e-4f;
    const float c15 = -1.5f * sk;
    const float umax_ok = kCurvTau / sk;   // sk |u| < tau  <=>  |u| < tau / sk
    double acc = 0.0;
    const int s1 = min((wv + 1) * SPW, NST);
    for (int st = wv * SPW; st < s1; ++st) {
        const int g = st / RS, r = st - g * RS;   // column group, row within each block
        const int u = ul + r, v = g * NC + cl;
        const int off = (T::EXT + (NRB * RS > T::TH ? min(u, T::TH - 1) : u)) * T::WCP + T::EXT + v;
        float wx[3][3], wp[3][3];
#pragma unroll
        for (int dy = 0; dy < 3; ++dy)
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) {
                wx[dy][dx] = xs[off + dy * T::WCP + dx];
                wp[dy][dx] = ps[off + dy * T::WCP + dx];
            }
        // pair validity (both pixels inside the image)
        const int U = U0 + u, V = V0 + v;
        bool ok[8];
#pragma unroll
        for (int d = 0; d < 8; ++d) ok[d] = !CHECK || (U + kDY[d] < H && V + kDX[d] < W);
        float a = 0.f;
        if (EPS0) {
#pragma unroll
            for (int d = 0; d < 8; ++d) {
                const float z = wx[0][0] - wx[kDY[d]][kDX[d]];
                const float qd = wp[0][0] - wp[kDY[d]][kDX[d]];
                const float tq = gam[d] * qd * qd * psi_quot(z, sk * qd, eps, e2);
                a += ok[d] ? tq : 0.f;
            }
        } else {
            float z[8], qd[8], rB[8], uu[8], tq[8], umax = 0.f;
#pragma unroll
            for (int d = 0; d < 8; ++d) {
                z[d] = wx[0][0] - wx[kDY[d]][kDX[d]];
                qd[d] = wp[0][0] - wp[kDY[d]][kDX[d]];
                rB[d] = rsq(fmaf(z[d], z[d], e2));
                uu[d] = qd[d] * rB[d];
                const float poly = fmaf(c15, uu[d] * (z[d] * rB[d]), 1.f);
                tq[d] = (uu[d] * uu[d]) * rB[d] * poly;
                umax = fmaxf(umax, fabsf(uu[d]));
                a = fmaf(ok[d] ? gq[d] : 0.f, tq[d], a);
            }
            if (!(umax < umax_ok)) {
                a = 0.f;
#pragma unroll
                for (int d = 0; d < 8; ++d) {
                    const float h = sk * qd[d];
                    const bool far = !(fabsf(uu[d]) < umax_ok);
                    float q = psi_series(z[d], h, rB[d], e2);
                    if (far && !(fabsf(h * rB[d]) < 1e-3f)) q = psi_closed(z[d], h, rB[d], e2);
                    const float tf = far ? gam[d] * qd[d] * qd[d] * q : gq[d] * tq[d];
                    a += ok[d] ? tf : 0.f;
                }
            }
        }
        const bool own = CHECK ? (u >= ru0 && u < ru1 && v >= rv0 && v < rv1)
                               : (NRB * RS == T::TH || u < T::TH);
        acc += own ? (double)a : 0.0;
    }
    dreg += acc;
}

// --------------------------------------------------------------- the tiles
// Window staging by rows: wave wv takes window rows wv, wv + kNWI, ... (so
// every row quantity is wave-uniform and sits in scalar registers) and lane
// takes columns lane + 64 c.  Loads are issued unconditionally from clamped
// coordinates; elements outside the view are stored as zero.
template <class T>
struct WinMap {
    static constexpr int NR = (T::WR + kNWI - 1) / kNWI;   // rows per wave
    static constexpr int NC = (T::WC + 63) / 64;           // columns per lane
};
struct WinCol {
    int vb, vc;   // view column, clamped into the view
    bool in;      // inside the window and the view
};
template <class T>
FI WinCol win_col(int lane, int c, int v0, int Wb) {
    WinCol w;
    const int col = lane + 64 * c;
    w.vb = v0 - T::EXT + col;
    w.vc = min(max(w.vb, 0), Wb - 1);
    w.in = col < T::WC && w.vb >= 0 && w.vb < Wb;
    return w;
}

struct TileOrigin {
    int u0, v0, u1, v1, U0, V0;
};

template <int S, int L, int TV>
FI TileOrigin tile_origin(const AS4 Proj &P, int ty, int tx) {
    using T = Tile<S, L, TV>;
    TileOrigin o;
    o.u0 = P.oy0 + ty * T::TH;
    o.v0 = P.ox0 + tx * T::TW;
    o.u1 = min(o.u0 + T::TH, P.oy1);
    o.v1 = min(o.v0 + T::TW, P.ox1);
    o.U0 = P.gy0 + o.u0;
    o.V0 = P.gx0 + o.v0;
    return o;
}

// Fused cost + gradient at x_t = x + alpha p (mode 1) or at x (mode 0):
// every frame's forward, residual, data cost and adjoint, then the BTV cost
// and gradient; writes g_t = grad J(x_t) to g[cur^1] for the owned pixels and
// the partial sums {E_data, E_reg, |g_t|^2, g_t.g_k, g_t.p}.
template <int S, int L, int TV, class ST, class SY>
FI void tile_trial(const AS4 Proj &P, const AS4 ScgState &st, int ty, int tx, int mode,
                   float *sm, double *red, double *part) {
    using T = Tile<S, L, TV>;
    using raw = typename ST::raw;
    using rawy = typename SY::raw;
    const AS4 OpDev &op = *cst(P.op);
    int tid = threadIdx.x;
    // per-tile index arithmetic is recomputed rather than kept live across the
    // work-list loop (where it would be spilled)
    asm volatile("" : "+v"(tid));
    const TileOrigin o = tile_origin<S, L, TV>(P, ty, tx);
    const int H = op.H, W = op.W, h = H / S, w = W / S, K = op.K;
    float *xs = sm;
    float *bands = xs + T::XS;                  // each wave's pass-1 / pass-3 output
    float *rs = bands + kNWI * T::PWT;          // the residual, two buffers
    float *po = sm + T::PO;                     // p at the owned pixels, for g_t . p

    const int xc = st.xc;
    const AS1 raw *xb = glb((const raw *)P.x[xc]);
    const AS1 float *pb = glb(P.p[xc]);
    const float af = (mode == 1) ? st.alpha_f : 0.f;
    const int Hb = P.Hb, Wb = P.Wb, ld = P.ld;
    const bool sr = st.wt.x_rounding == 1;
    const unsigned seed = st.rseed;
    const AS4 OpDev &opg = op;
    const i64 Wg = opg.W;
    // window of x_t into LDS: every load first (clamped, unconditional), then
    // the arithmetic, so that the loads are in flight together.  Global loads
    // are issued at raised wave priority (here, for g_k and for the frames):
    // the other workgroup on the CU is usually in a compute phase, and its
    // waves would otherwise delay the issue of the loads (measured: k_trial
    // 65.4 -> 64.0 us at 2048^2)
    using WM = WinMap<T>;
    const int lane0 = tid & 63, wv0 = uni(tid >> 6);
    WinCol wc[WM::NC];
#pragma unroll
    for (int c = 0; c < WM::NC; ++c) wc[c] = win_col<T>(lane0, c, o.v0, Wb);
    if (mode == 1) {
        float xr[WM::NR][WM::NC], pr[WM::NR][WM::NC];
        __builtin_amdgcn_s_setprio(2);
#pragma unroll
        for (int r = 0; r < WM::NR; ++r) {
            const int ub = o.u0 - T::EXT + wv0 + kNWI * r;
            const i64 rb = (i64)min(max(ub, 0), Hb - 1) * ld;
#pragma unroll
            for (int c = 0; c < WM::NC; ++c) {
                xr[r][c] = ST::ld(xb + rb, wc[c].vc);
                pr[r][c] = pb[rb + wc[c].vc];
            }
        }
        __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int r = 0; r < WM::NR; ++r) {
            const int row = wv0 + kNWI * r, ub = o.u0 - T::EXT + row;
            if (row < T::WR) {
                const bool rin = ub >= 0 && ub < Hb;
                const int ou = row - T::EXT;
#pragma unroll
                for (int c = 0; c < WM::NC; ++c) {
                    const int col = lane0 + 64 * c, ov = col - T::EXT;
                    const float v = fmaf(af, pr[r][c], xr[r][c]);
                    const float vr =
                        sr ? ST::rnd_sr(v, pixel_hash((i64)(P.gy0 + ub) * Wg + P.gx0 + wc[c].vb,
                                                      seed))
                           : ST::rnd(v);
                    if (col < T::WC) xs[row * T::WCP + col] = (rin && wc[c].in) ? vr : 0.f;
                    if (T::POL && ou >= 0 && ou < T::TH && ov >= 0 && ov < T::TW)
                        po[ou * T::TW + ov] = pr[r][c];
                }
            }
        }
    } else {
        float xr[WM::NR][WM::NC];
#pragma unroll
        for (int r = 0; r < WM::NR; ++r) {
            const int ub = o.u0 - T::EXT + wv0 + kNWI * r;
            const i64 rb = (i64)min(max(ub, 0), Hb - 1) * ld;
#pragma unroll
            for (int c = 0; c < WM::NC; ++c) xr[r][c] = ST::ld(xb + rb, wc[c].vc);
        }
#pragma unroll
        for (int r = 0; r < WM::NR; ++r) {
            const int row = wv0 + kNWI * r, ub = o.u0 - T::EXT + row;
            if (row < T::WR) {
                const bool rin = ub >= 0 && ub < Hb;
#pragma unroll
                for (int c = 0; c < WM::NC; ++c) {
                    const int col = lane0 + 64 * c;
                    if (col < T::WC) xs[row * T::WCP + col] = (rin && wc[c].in) ? xr[r][c] : 0.f;
                }
            }
        }
    }
    float gacc[T::CV];
#pragma unroll
    for (int c = 0; c < T::CV; ++c) gacc[c] = 0.f;
    double e_data = 0.0;
    const int data_p = st.wt.data_p;
    const float epsd = st.wt.eps_data, e2d = epsd * epsd;
    const AS1 rawy *yb = glb((const rawy *)P.y);
    const float yscale = st.wt.y_scale;
    using FT = typename T::FT;
    constexpr int CI = FT::CI, CJ = FT::CJ;
    const int ibl = lane0 / CJ, cjl = lane0 - ibl * CJ;
    // the frame values of pass 2, one frame ahead: each lane loads those of
    // its own rows and column (clamped into the frame)
    rawy yn[CI];
    auto load_y = [&](int k) {
        const int i = cdiv(o.U0 - L + 1 - op.offy[k], S) + ibl * CI;
        const int j = cdiv(o.V0 - L + 1 - op.offx[k], S) + wv0 * CJ + cjl;
        const AS1 rawy *yk = yb + (i64)k * h * w + min(max(j, 0), w - 1);
        __builtin_amdgcn_s_setprio(2);
#pragma unroll
        for (int c = 0; c < CI; ++c) yn[c] = yk[(i64)min(max(i + c, 0), h - 1) * w];
        __builtin_amdgcn_s_setprio(0);
    };
    load_y(0);
    __syncthreads();

    // One barrier per frame: the residual of frame k is published before the
    // adjoint strips read it, and frame k + 1 writes the other buffer.
    float *band = bands + wv0 * T::PWT;
    for (int k = 0; k < K; ++k) {
        const int offy = op.offy[k], offx = op.offx[k];
        const AxisW<L> ay = axis_y<L>(op, k), ax = axis_x<L>(op, k);
        // LR rows and columns touching the tile (NIM x NJM from (iF, jF));
        // those outside the frame hold a zero residual
        const int iF = cdiv(o.U0 - L + 1 - offy, S), jF = cdiv(o.V0 - L + 1 - offx, S);
        float *rsk = rs + (k & 1) * T::RSS;
        const float *win =
            xs + (S * iF + offy - o.U0 + T::EXT) * T::WCP + S * jF + offx - o.V0 + T::EXT;
        fwd_strip<S, L, FT>(win, T::WCP, band, ay, ax, iF, jF, lane0, wv0,
                            [&](int i0, int cj, const float (&av)[CI]) {
            const int j = wv0 * CJ + cj, gj = jF + j;
            const bool in_j = gj >= 0 && gj < w;
            const bool own_j = (S * gj >= o.V0) && (S * gj < P.gx0 + o.v1);
#pragma unroll
            for (int c = 0; c < CI; ++c) {
                const int gi = iF + i0 + c;
                const float r = fmaf(-SY::cv(yn[c]), yscale, av[c]);
                const bool own = own_j && (S * gi >= o.U0) && (S * gi < P.gy0 + o.u1);
                float rv;
                if (data_p == 2) {
                    const double ro = own ? (double)r : 0.0;
                    e_data += ro * ro;
                    rv = 2.f * r;
                } else {
                    float ph, ps;
                    phi_psi(r, epsd, e2d, ph, ps);
                    e_data += own ? (double)ph : 0.0;
                    rv = ps;
                }
                rsk[(i0 + c) * T::RP + j] = (in_j && gi >= 0 && gi < h) ? rv : 0.f;
            }
        });
        if (k + 1 < K) load_y(k + 1);
        __syncthreads();
        adj_strip<S, L, TV>(rsk, band, gacc, o.U0, o.V0, offy, offx, iF, jF, ay, ax, lane0, wv0);
    }
    __syncthreads();

    // data-term gradient to LDS (lanes hold rows), then the prior adds in place
    float *gs = bands;
    {
        const int u = lane0 - 2;
        if (u >= 0 && u < T::TH)
#pragma unroll
            for (int c = 0; c < T::CV; ++c) gs[u * T::GP + wv0 * T::CV + c] = gacc[c];
    }
    // the output pass's loads of g_k are issued here, so that they are in
    // flight during the prior's sweep (p at the owned pixels is in LDS)
    const int cur = st.cur;
    AS1 float *gout = glbw(P.g[cur ^ 1]);
    const AS1 float *gk = glb(P.g[cur]);
    const AS1 float *pk = glb(P.p[xc]);
    AS1 float *pz = glbw(P.p[xc]);
    // owned pixels by rows as in the staging: wave wv0 takes tile rows
    // wv0 + kNWI r, lane takes columns lane0 + 64 c
    constexpr int ONR = (T::TH + kNWI - 1) / kNWI, ONC = (T::TW + 63) / 64;
    int ocol[ONC];     // clamped view column
    bool cown[ONC];    // column owned
#pragma unroll
    for (int c = 0; c < ONC; ++c) {
        const int col = lane0 + 64 * c;
        cown[c] = col < T::TW && o.v0 + col < o.v1;
        ocol[c] = min(o.v0 + col, o.v1 - 1);
    }
    // g_k at the owned pixels; the wide tile issues these loads before the
    // prior's sweep so that they are in flight during it, the narrow tile
    // (whose sweep leaves no registers to carry them) after it
    constexpr bool PRE = TV == 0 || TV == kNarrow;
    float gkv[ONR][ONC];
    auto load_gk = [&]() {
        __builtin_amdgcn_s_setprio(2);
#pragma unroll
        for (int r = 0; r < ONR; ++r) {
            const i64 rb = (i64)min(o.u0 + wv0 + kNWI * r, o.u1 - 1) * ld;
#pragma unroll
            for (int c = 0; c < ONC; ++c) gkv[r][c] = gk[rb + ocol[c]];
        }
        __builtin_amdgcn_s_setprio(0);
    };
    if (PRE && mode == 1) load_gk();
    float gam[8];
#pragma unroll
    for (int d = 0; d < 8; ++d) gam[d] = st.wt.gam[kDY[d] * 3 + kDX[d]];
    const float eps = st.wt.eps;
    double e_reg = 0.0;
    // interior tiles: every pair of the sweep lies inside the image, tile owned
    // whole.  A narrow tile's wave goes by the wide tile that its columns lie in:
    // where the widths do not divide (56 and 24 columns, 80 and 32), a narrow
    // tile lies across two wide ones, of which the second may be cut by the edge;
    // at scale 1 so may a wave's columns, which then go by both.
    constexpr int TWW = TV == kNarrow ? Tile<S, L, 0>::TW : T::TW;
    const int vrel = o.v0 - P.ox0, vin = vrel % TWW;
    auto inner_cols = [&](int v) {   // the (wide) tile that holds column v (from ox0)
        const int a = v - v % TWW;
        return P.gx0 + P.ox0 + a >= 2 && P.gx0 + P.ox0 + a + TWW + 2 <= W &&
               P.ox0 + a + TWW <= P.ox1;
    };
    const int vw = TV == kNarrow ? vrel + wv0 * T::CV : vrel;
    const bool inner = o.U0 >= 2 && o.U0 + T::TH + 2 <= H && o.u1 - o.u0 == T::TH &&
                       inner_cols(vw) &&
                       (TWW % T::CV == 0 || inner_cols(vw + T::CV - 1));   // (by wave)
    const int tho = o.u1 - o.u0, two = o.v1 - o.v0;
    const int cw0 = (vin + wv0 * T::CV) % (TWW / kNWI);
    if (eps == 0.f)
        btv_sweep<S, L, TV, true, true>(xs, gs, gam, eps, o.U0, o.V0, H, W, tho, two, cw0, e_reg);
    else if (inner)
        btv_sweep<S, L, TV, false, false>(xs, gs, gam, eps, o.U0, o.V0, H, W, tho, two, cw0,
                                          e_reg);
    else
        btv_sweep<S, L, TV, false, true>(xs, gs, gam, eps, o.U0, o.V0, H, W, tho, two, cw0,
                                         e_reg);
    __syncthreads();
    // owned gradient out, with its inner products (g_k is widened to double
    // only here: widened at its load, it would be carried across the sweep
    // in twice the registers)
    double gg = 0.0, ggk = 0.0, gp = 0.0;
    if (!PRE && mode == 1) load_gk();
    if (mode == 1)
#pragma unroll
        for (int r = 0; r < ONR; ++r)
#pragma unroll
            for (int c = 0; c < ONC; ++c) asm volatile("" : "+v"(gkv[r][c]));
#pragma unroll
    for (int r = 0; r < ONR; ++r) {
        const int row = wv0 + kNWI * r;
        if (row >= T::TH || o.u0 + row >= o.u1) continue;   // wave-uniform
        const i64 rb = (i64)(o.u0 + row) * ld;
#pragma unroll
        for (int c = 0; c < ONC; ++c) {
            if (!cown[c]) continue;
            const int col = lane0 + 64 * c;
            const float gv = gs[row * T::GP + col];
            gout[rb + ocol[c]] = gv;
            gg += (double)gv * (double)gv;
            // start direction buffer for the init pass (none when the caller
            // evaluates the cost and gradient alone without one)
            if (mode == 0 && pz) pz[rb + ocol[c]] = 0.f;
            if (mode == 1) {
                ggk += (double)gv * (double)gkv[r][c];
                gp += (double)gv * (double)(T::POL ? po[row * T::TW + col] : pk[rb + ocol[c]]);
            }
        }
    }
    double v[5] = {e_data, e_reg, gg, ggk, gp};
    pass_end<5, kNTI>(v, part, red, P, mode);
}

// Data part of the curvature over the owned LR pixels (all edges are
// multiples of S): L2 (DP = 2), 2 |A_k p|^2, exact since the term is
// quadratic; L1 (DP = 1, Charbonnier), the sum of (A_k p)^2 Q(r, sk A_k p) with
// r = A_k x - y_k and Q the quotient the prior's pairs use.  Each wave runs
// its own strip of every frame with no barrier; [iA, iB) x [jA, jB) are the
// owned LR pixels.
template <int S, int L, int TV, class SY, int DP>
FI double upd_data_part(const AS4 Proj &P, const AS4 ScgState &st, const TileOrigin &o,
                        const float *xs, const float *ps, float *band, int iA, int iB, int jA,
                        int jB, int lane, int wv) {
    using T = Tile<S, L, TV>;
    using FU = typename T::FU;
    using rawy = typename SY::raw;
    const AS4 OpDev &op = *cst(P.op);
    const int h = op.H / S, w = op.W / S, K = op.K;
    const float skd = st.sigk_f, epsd = st.wt.eps_data, e2d = epsd * epsd;
    const AS1 rawy *yb = glb((const rawy *)P.y);
    const int i0t = o.U0 / S, j0t = o.V0 / S;
    double ap2 = 0.0;
    for (int k = 0; k < K; ++k) {
        const int woff = (op.offy[k] + T::EXT) * T::WCP + op.offx[k] + T::EXT;
        const AxisW<L> ay = axis_y<L>(op, k), ax = axis_x<L>(op, k);
        float xa[FU::CI];
        if (DP == 1)
            fwd_strip<S, L, FU>(xs + woff, T::WCP, band, ay, ax, i0t, j0t, lane, wv,
                                [&](int, int, const float (&av)[FU::CI]) {
#pragma unroll
                for (int c = 0; c < FU::CI; ++c) xa[c] = av[c];
            });
        const AS1 rawy *yk = yb + (i64)k * h * w;
        fwd_strip<S, L, FU>(ps + woff, T::WCP, band, ay, ax, i0t, j0t, lane, wv,
                            [&](int i0, int cj, const float (&av)[FU::CI]) {
            const int gj = j0t + wv * FU::CJ + cj;
#pragma unroll
            for (int c = 0; c < FU::CI; ++c) {
                const int gi = i0t + i0 + c;
                const bool own = gj >= jA && gj < jB && gi >= iA && gi < iB;
                if (DP == 2) {
                    const double a = own ? (double)av[c] : 0.0;
                    ap2 += a * a;
                } else if (own) {
                    const float r = fmaf(-SY::ld(yk, (i64)gi * w + gj), st.wt.y_scale, xa[c]);
                    ap2 += (double)(av[c] * av[c] * psi_quot(r, skd * av[c], epsd, e2d));
                }
            }
        });
    }
    return DP == 2 ? 2.0 * ap2 : ap2;
}

// Accepted step: x <- x + alpha p, p <- -g_t + beta p (into the other buffer
// of each pair), then Moller's curvature at the new (x, p) without forming
// x + sigma_k p: data part 2 sum_k |A_k p|^2 for the L2 term (exact: it is
// quadratic) or sum_k (A_k p)^2 Q(A_k x - y_k, sigma_k A_k p) for the L1
// (Charbonnier) term, prior part lambda sum gamma q^2 Q(z, sigma_k q).
// Partial sums {data part, prior part, |p|^2, p.r}.
template <int S, int L, int TV, class ST, class SY>
FI void tile_upcurv(const AS4 Proj &P, const AS4 ScgState &st, int ty, int tx, float *sm,
                    double *red, double *part) {
    static_assert(TV != 2, "the trial kernel's own tile shape");
    using T = Tile<S, L, TV>;
    using raw = typename ST::raw;
    const AS4 OpDev &op = *cst(P.op);
    int tid = threadIdx.x;
    // per-tile index arithmetic is recomputed rather than kept live across the
    // work-list loop (where it would be spilled)
    asm volatile("" : "+v"(tid));
    // update tiles cover the update rectangle (owned plus halo); reductions
    // count only their intersection with the owned rectangle [ou0,ou1) x [ov0,ov1)
    TileOrigin o;
    o.u0 = P.uy0 + ty * T::TH;
    o.v0 = P.ux0 + tx * T::TW;
    o.u1 = min(o.u0 + T::TH, P.uy1);
    o.v1 = min(o.v0 + T::TW, P.ux1);
    o.U0 = P.gy0 + o.u0;
    o.V0 = P.gx0 + o.v0;
    const int ou0 = max(o.u0, P.oy0), ou1 = min(o.u1, P.oy1);
    const int ov0 = max(o.v0, P.ox0), ov1 = min(o.v1, P.ox1);
    const int H = op.H, W = op.W;
    float *xs = sm;
    float *ps = xs + T::XS;
    float *bands = ps + T::XS;  // each wave's pass-1 output

    const int src = st.upd_src, dst = src ^ 1;
    const AS1 raw *xb = glb((const raw *)P.x[src]);
    const AS1 float *pb = glb(P.p[src]);
    const AS1 float *gt = glb(P.g[st.cur]);
    AS1 raw *xo = glbw((raw *)P.x[dst]);
    AS1 float *po = glbw(P.p[dst]);
    const float af = st.alpha_f, bf = st.beta_f;
    const int Hb = P.Hb, Wb = P.Wb, ld = P.ld;
    const bool sr = st.wt.x_rounding == 1;
    const unsigned seed = st.rseed;
    const i64 Wg = W;
    double pp = 0.0, pr = 0.0;
    {
        // every load first (clamped, unconditional, at raised wave priority
        // as in the trial pass), then the update
        using WM = WinMap<T>;
        const int lane0 = tid & 63, wv0 = uni(tid >> 6);
        WinCol wc[WM::NC];
#pragma unroll
        for (int c = 0; c < WM::NC; ++c) wc[c] = win_col<T>(lane0, c, o.v0, Wb);
        float xr[WM::NR][WM::NC], pr0[WM::NR][WM::NC], gr[WM::NR][WM::NC];
        __builtin_amdgcn_s_setprio(2);
#pragma unroll
        for (int r = 0; r < WM::NR; ++r) {
            const int ub = o.u0 - T::EXT + wv0 + kNWI * r;
            const i64 rb = (i64)min(max(ub, 0), Hb - 1) * ld;
#pragma unroll
            for (int c = 0; c < WM::NC; ++c) {
                xr[r][c] = ST::ld(xb + rb, wc[c].vc);
                pr0[r][c] = pb[rb + wc[c].vc];
                gr[r][c] = gt[rb + wc[c].vc];
            }
        }
        __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int r = 0; r < WM::NR; ++r) {
            const int row = wv0 + kNWI * r, ub = o.u0 - T::EXT + row;
            if (row < T::WR) {
                const bool rin = ub >= 0 && ub < Hb;
                const bool urow = rin && ub >= o.u0 && ub < o.u1;   // updated rows
                const bool orow = ub >= ou0 && ub < ou1;            // owned rows
                const i64 rb = (i64)ub * ld;                        // in the view when urow
#pragma unroll
                for (int c = 0; c < WM::NC; ++c) {
                    const int col = lane0 + 64 * c, vb = wc[c].vb;
                    const bool in = rin && wc[c].in;
                    const float v = fmaf(af, pr0[r][c], xr[r][c]);
                    float xv = sr ? ST::rnd_sr(v, pixel_hash((i64)(P.gy0 + ub) * Wg + P.gx0 + vb,
                                                             seed))
                                  : ST::rnd(v);
                    float pv = fmaf(bf, pr0[r][c], -gr[r][c]);
                    xv = in ? xv : 0.f;
                    pv = in ? pv : 0.f;
                    if (urow && wc[c].in && vb >= o.v0 && vb < o.v1) {
                        ST::st(xo, rb + vb, xv);
                        po[rb + vb] = pv;
                        if (orow && vb >= ov0 && vb < ov1) {
                            pp += (double)pv * (double)pv;
                            pr -= (double)pv * (double)gr[r][c];
                        }
                    }
                    if (col < T::WC) {
                        xs[row * T::WCP + col] = xv;
                        ps[row * T::WCP + col] = pv;
                    }
                }
            }
        }
    }
    __syncthreads();
    // data part over the owned LR pixels (all edges are multiples of S): L2,
    // 2 |A_k p|^2 (exact, the term is quadratic); L1 (Charbonnier), the sum of
    // (A_k p)^2 Q(r, sk A_k p) with r = A_k x - y_k, the same quotient as the
    // prior's pairs
    double ap2 = 0.0;
    const int lane = tid & 63, wv = uni(tid >> 6);
    const int iA = (P.gy0 + ou0) / S, iB = (P.gy0 + ou1) / S;
    const int jA = (P.gx0 + ov0) / S, jB = (P.gx0 + ov1) / S;
    float *band = bands + wv * T::FU::LDS;
    if (iA < iB && jA < jB) {
        if (st.wt.data_p == 2)
            ap2 = upd_data_part<S, L, TV, SY, 2>(P, st, o, xs, ps, band, iA, iB, jA, jB, lane, wv);
        else
            ap2 = upd_data_part<S, L, TV, SY, 1>(P, st, o, xs, ps, band, iA, iB, jA, jB, lane, wv);
    }
    // prior part over the owned pairs (i, i+d)
    const float eps = st.wt.eps, sk = st.sigk_f;
    float gam[8];
#pragma unroll
    for (int d = 0; d < 8; ++d) gam[d] = st.wt.gam[kDY[d] * 3 + kDX[d]];
    double dreg = 0.0;
    const int ru0 = ou0 - o.u0, ru1 = ou1 - o.u0, rv0 = ov0 - o.v0, rv1 = ov1 - o.v0;
    const bool inner = o.U0 + T::TH + 2 <= H && o.V0 + T::TW + 2 <= W && ru0 == 0 &&
                       ru1 == T::TH && rv0 == 0 && rv1 == T::TW;
    if (eps == 0.f)
        curv_sweep<S, L, TV, true, true>(xs, ps, gam, eps, sk, o.U0, o.V0, H, W, ru0, ru1, rv0, rv1,
                                     dreg);
    else if (inner)
        curv_sweep<S, L, TV, false, false>(xs, ps, gam, eps, sk, o.U0, o.V0, H, W, ru0, ru1, rv0,
                                       rv1, dreg);
    else
        curv_sweep<S, L, TV, true, false>(xs, ps, gam, eps, sk, o.U0, o.V0, H, W, ru0, ru1, rv0,
                                      rv1, dreg);
    double v[4] = {ap2, dreg, pp, pr};
    pass_end<4, kNTI>(v, part, red, P, 2);
}

// y[k] = A_k x on the owned LR pixels of one tile.
template <int S, int L, int TV, class ST>
FI void tile_forward(const AS4 Proj &P, int ty, int tx, const void *xin, void *yout, float *sm) {
    using T = Tile<S, L, TV>;
    using raw = typename ST::raw;
    const AS4 OpDev &op = *cst(P.op);
    int tid = threadIdx.x;
    // per-tile index arithmetic is recomputed rather than kept live across the
    // work-list loop (where it would be spilled)
    asm volatile("" : "+v"(tid));
    const TileOrigin o = tile_origin<S, L, TV>(P, ty, tx);
    const int h = op.H / S, w = op.W / S, K = op.K;
    float *xs = sm;
    const AS1 raw *xb = glb((const raw *)xin);
    const int Hb = P.Hb, Wb = P.Wb, ld = P.ld;
    const int lane = tid & 63, wv = uni(tid >> 6);
    {
        // every load first, as in the trial pass (one at a time behind its
        // bounds check, 2000^2 LR at s = 2 took 59.4 us; this takes 45.6)
        using WM = WinMap<T>;
        WinCol wc[WM::NC];
#pragma unroll
        for (int c = 0; c < WM::NC; ++c) wc[c] = win_col<T>(lane, c, o.v0, Wb);
        float xr[WM::NR][WM::NC];
#pragma unroll
        for (int r = 0; r < WM::NR; ++r) {
            const int ub = o.u0 - T::EXT + wv + kNWI * r;
            const i64 rb = (i64)min(max(ub, 0), Hb - 1) * ld;
#pragma unroll
            for (int c = 0; c < WM::NC; ++c) xr[r][c] = ST::cv(*at32(xb + rb, wc[c].vc));
        }
#pragma unroll
        for (int r = 0; r < WM::NR; ++r) {
            const int row = wv + kNWI * r, ub = o.u0 - T::EXT + row;
            const bool rin = ub >= 0 && ub < Hb;
            if (row < T::WR)
#pragma unroll
                for (int c = 0; c < WM::NC; ++c) {
                    const int col = lane + 64 * c;
                    if (col < T::WC) xs[row * T::WCP + col] = rin && wc[c].in ? xr[r][c] : 0.f;
                }
        }
    }
    __syncthreads();
    const int NIo = (o.u1 - o.u0) / S, NJo = (o.v1 - o.v0) / S;
    const int iA = o.U0 / S, jA = o.V0 / S;
    using FU = typename T::FU;
    float *band = xs + T::XS + wv * FU::LDS;
    AS1 raw *yo = glbw((raw *)yout);
    for (int k = 0; k < K; ++k) {
        const AxisW<L> ay = axis_y<L>(op, k), ax = axis_x<L>(op, k);
        const float *win = xs + (op.offy[k] + T::EXT) * T::WCP + op.offx[k] + T::EXT;
        fwd_strip<S, L, FU>(win, T::WCP, band, ay, ax, iA, jA, lane, wv,
                            [&](int i0, int cj, const float (&av)[FU::CI]) {
            const int j = wv * FU::CJ + cj;
            const i64 at = ((i64)k * h + iA + i0) * w + jA + j;
#pragma unroll
            for (int c = 0; c < FU::CI; ++c)
                if (j < NJo && i0 + c < NIo) ST::st(yo, at + (i64)c * w, av[c]);
        });
    }
}

// x = sum_k A_k^T r_k on the owned HR pixels of one tile.
template <int S, int L, int TV, class ST>
FI void tile_adjoint(const AS4 Proj &P, int ty, int tx, const void *r, float *xout, float *sm) {
    using T = Tile<S, L, TV>;
    using raw = typename ST::raw;
    const AS4 OpDev &op = *cst(P.op);
    int tid = threadIdx.x;
    // per-tile index arithmetic is recomputed rather than kept live across the
    // work-list loop (where it would be spilled)
    asm volatile("" : "+v"(tid));
    const TileOrigin o = tile_origin<S, L, TV>(P, ty, tx);
    const int h = op.H / S, w = op.W / S, K = op.K;
    float *gs = sm;
    const int lane = tid & 63, wv = uni(tid >> 6);
    float *band = gs + T::XS + wv * T::PWT;
    float *rs = gs + T::XS + kNWI * T::PWT;
    const AS1 raw *rb = glb((const raw *)r);
    float gacc[T::CV];
#pragma unroll
    for (int c = 0; c < T::CV; ++c) gacc[c] = 0.f;
    // the LR rows and columns touching the tile, NIM x NJM from (iF, jF), one
    // frame ahead in registers; zero outside the frame
    constexpr int NQ = ceil_div(T::NIM * T::NJM, kNTI);
    float rn[NQ];
    auto load_r = [&](int k) {
        const int iF = cdiv(o.U0 - L + 1 - op.offy[k], S);
        const int jF = cdiv(o.V0 - L + 1 - op.offx[k], S);
#pragma unroll
        for (int e = 0; e < NQ; ++e) {
            const int q = tid + e * kNTI, ii = q / T::NJM, jj = q - ii * T::NJM;
            const int gi = iF + ii, gj = jF + jj;
            const bool in = gi >= 0 && gi < h && gj >= 0 && gj < w;
            const float v = ST::ld(rb, ((i64)k * h + min(max(gi, 0), h - 1)) * w +
                                           min(max(gj, 0), w - 1));
            rn[e] = in ? v : 0.f;
        }
    };
    load_r(0);
    for (int k = 0; k < K; ++k) {
        const int offy = op.offy[k], offx = op.offx[k];
        const AxisW<L> ay = axis_y<L>(op, k), ax = axis_x<L>(op, k);
        const int iF = cdiv(o.U0 - L + 1 - offy, S), jF = cdiv(o.V0 - L + 1 - offx, S);
        float *rsk = rs + (k & 1) * T::RSS;
#pragma unroll
        for (int e = 0; e < NQ; ++e) {
            const int q = tid + e * kNTI, ii = q / T::NJM, jj = q - ii * T::NJM;
            if (ii < T::NIM) rsk[ii * T::RP + jj] = rn[e];
        }
        if (k + 1 < K) load_r(k + 1);
        __syncthreads();
        adj_strip<S, L, TV>(rsk, band, gacc, o.U0, o.V0, offy, offx, iF, jF, ay, ax, lane, wv);
    }
    {
        const int u = lane - 2;
        if (u >= 0 && u < T::TH)
#pragma unroll
            for (int c = 0; c < T::CV; ++c) gs[u * T::GP + wv * T::CV + c] = gacc[c];
    }
    __syncthreads();
    AS1 float *xo = glbw(xout);
    const int ld = P.ld;
    for (int q = tid; q < T::TH * T::TW; q += kNTI) {
        const int uu = q / T::TW, vv = q - uu * T::TW;
        if (o.u0 + uu >= o.u1 || o.v0 + vv >= o.v1) continue;
        xo[(i64)(o.u0 + uu) * ld + o.v0 + vv] = gs[uu * T::GP + vv];
    }
}

// -------------------------------------------------------------- the kernels
// The item count is read from device memory so that one captured launch can
// serve a changing list; the trial and update kernels are launched with one
// workgroup per item, the standalone operators walk the list with a grid
// stride.
//
// Workgroups are dispatched to the 8 XCDs round-robin in blockIdx order, and
// each XCD has its own L2.  With one workgroup per item, workgroup b takes
// item xcd_item(b, n): XCD b % 8 gets one contiguous run of the list (a band
// of neighbouring tiles), so the halos neighbouring tiles share are re-read
// from that XCD's L2 rather than fetched again.
//
// A tile is a chain of dependent phases (windows in, a barrier per frame, the
// sweeps, the reduction): a 48 x 96 tile alone on a CU takes 22 us at scale 2
// whatever the image, so an image of few tiles leaves most CUs idle for as
// long.  Items of small images (Item::nar) are narrow tiles of the same
// height: 48 x 32 takes 15 us (trial) and 11-13 us (update; 48 x 96: 20-27).
// The same kernels run them, so that a batch of small and large images stays
// one launch per pass.
FI int xcd_item(int b, int n) {
    const int q = n >> 3, r = n & 7, x = b & 7, j = b >> 3;
    return x * q + min(x, r) + j;
}
template <int S, int L, int TV, class ST, class SY>
__global__ void __launch_bounds__(kNTI, 4) k_trial(const Proj *projs, const Item *items,
                                                const int *n_items, double *partials,
                                                int mode) {
    __shared__ float sm[Tile<S, L, TV>::SMEM];
    __shared__ double red[kNV * kNWI];
    // one workgroup per item (the launch grid is the item count): no loop, so
    // nothing is hoisted out of one and kept live through the tile
    const int n = *cst(n_items);
    const int b = blockIdx.x;
    if (b >= n) return;
    const int it = (int)gridDim.x == n ? xcd_item(b, n) : b;
    const AS4 Item &itm = cst(items)[it];
    const AS4 Proj &P = cst(projs)[itm.proj];
    const AS4 ScgState &st = *cst(P.st);
    if (mode == 1 && !st.active) return;
    double *part = partials + (i64)it * kNV;
    if (TV == 0 && itm.nar)
        tile_trial<S, L, TV == 0 ? kNarrow : TV, ST, SY>(P, st, itm.ty, itm.tx, mode, sm,
                                                                red, part);
    else
        tile_trial<S, L, TV, ST, SY>(P, st, itm.ty, itm.tx, mode, sm, red, part);
}

template <int S, int L, int TV, class ST, class SY>
__global__ void __launch_bounds__(kNTI, 4) k_upcurv(const Proj *projs, const Item *items,
                                                 const int *n_items, double *partials) {
    __shared__ float sm[Tile<S, L, TV>::SMEM_U];
    __shared__ double red[kNV * kNWI];
    const int n = *cst(n_items);
    const int b = blockIdx.x;
    if (b >= n) return;
    const int it = (int)gridDim.x == n ? xcd_item(b, n) : b;
    const AS4 Item &itm = cst(items)[it];
    const AS4 Proj &P = cst(projs)[itm.proj];
    const AS4 ScgState &st = *cst(P.st);
    if (!st.do_update) return;
    double *part = partials + (i64)it * kNV;
    if (TV == 0 && itm.nar)
        tile_upcurv<S, L, TV == 0 ? kNarrow : TV, ST, SY>(P, st, itm.ty, itm.tx, sm, red,
                                                                 part);
    else
        tile_upcurv<S, L, TV, ST, SY>(P, st, itm.ty, itm.tx, sm, red, part);
}

template <int S, int L, int TV, class ST>
__global__ void __launch_bounds__(kNTI) k_forward(const Proj *projs, const Item *items, int n,
                                                  const void *xin, void *yout) {
    __shared__ float sm[Tile<S, L, TV>::SMEM_F];
    for (int it = blockIdx.x; it < n; it += gridDim.x) {
        const AS4 Item &itm = cst(items)[it];
        const AS4 Proj &P = cst(projs)[itm.proj];
        if (TV == 0 && itm.nar)
            tile_forward<S, L, TV == 0 ? kNarrow : TV, ST>(P, itm.ty, itm.tx, xin, yout, sm);
        else
            tile_forward<S, L, TV, ST>(P, itm.ty, itm.tx, xin, yout, sm);
        __syncthreads();
    }
}

template <int S, int L, int TV, class ST>
__global__ void __launch_bounds__(kNTI) k_adjoint(const Proj *projs, const Item *items, int n,
                                                  const void *r, float *xout) {
    __shared__ float sm[Tile<S, L, TV>::SMEM_A];
    for (int it = blockIdx.x; it < n; it += gridDim.x) {
        const AS4 Item &itm = cst(items)[it];
        const AS4 Proj &P = cst(projs)[itm.proj];
        if (TV == 0 && itm.nar)
            tile_adjoint<S, L, TV == 0 ? kNarrow : TV, ST>(P, itm.ty, itm.tx, r, xout, sm);
        else
            tile_adjoint<S, L, TV, ST>(P, itm.ty, itm.tx, r, xout, sm);
        __syncthreads();
    }
}

// --------------------------------------------------- launchers for this S
// Band lengths instantiated per scale (the operator's L is rounded up).
#if MISR_SCALE == 1
#define MISR_LIST(X) X(4) X(8) X(16)
#elif MISR_SCALE == 2
#define MISR_LIST(X) X(6) X(8) X(9) X(12) X(16)
#elif MISR_SCALE == 3
#define MISR_LIST(X) X(6) X(9) X(10) X(12) X(16)
#elif MISR_SCALE == 4
#define MISR_LIST(X) X(12) X(16)
#endif

#define MISR_CAT2(a, b) a##b
#define MISR_CAT(a, b) MISR_CAT2(a, b)
#define MISR_FN(name) MISR_CAT(name, MISR_SCALE)

// Kernel keys: key = Lp | (tile variant << 8); variant 0 is the widest tile
// that fits, variant 1 about half as wide (chosen per operator by the tile
// autotuner).
// the update pass and the operators: variant 2 runs variant 0's shape
#define MISR_VARIANT(key, BODY) \
    if (((key) >> 8) == 1) {    \
        constexpr int tv = 1;   \
        BODY                    \
    } else {                    \
        constexpr int tv = 0;   \
        BODY                    \
    }
// the trial pass: every variant is its own shape
#define MISR_VARIANT_TRIAL(key, BODY) \
    if (((key) >> 8) == 0) {          \
        constexpr int tv = 0;         \
        BODY                          \
    } else if (((key) >> 8) == 1) {   \
        constexpr int tv = 1;         \
        BODY                          \
    } else {                          \
        constexpr int tv = 2;         \
        BODY                          \
    }

// Tile shapes of a kernel key (band length | variant << 8, or | kNarrow << 8
// for the narrow tile of variant 0's kernels): the update
// pass's (and the operators'), then the trial pass's.  Variant 2 pairs the
// trial kernel's own wider shape with variant 0's update shape; it exists
// only where that shape is wider.
template <int L>
constexpr bool wide_trial() {
    return Tile<MISR_SCALE, L, 2>::TW > Tile<MISR_SCALE, L, 0>::TW;
}

int MISR_FN(tile_dims_s)(int key, int *th, int *tw) {
    const int v = key >> 8, Lp = key & 255;
#define X(l)                                                        \
    if (Lp == l) {                                                  \
        if (v == kNarrow) {                                         \
            using TN = Tile<MISR_SCALE, l, kNarrow>;            \
            using T0 = Tile<MISR_SCALE, l, 0>;                      \
            static_assert(TN::SMEM <= T0::SMEM && TN::SMEM_U <= T0::SMEM_U && \
                          TN::SMEM_F <= T0::SMEM_F && TN::SMEM_A <= T0::SMEM_A, \
                          "narrow tiles run in variant 0's kernels"); \
            *th = TN::TH;                                           \
            *tw = TN::TW;                                           \
            return 1;                                               \
        }                                                           \
        if (v == 1) {                                               \
            *th = Tile<MISR_SCALE, l, 1>::TH;                       \
            *tw = Tile<MISR_SCALE, l, 1>::TW;                       \
            return 1;                                               \
        }                                                           \
        if (v == 0 || (v == 2 && wide_trial<l>())) {                \
            *th = Tile<MISR_SCALE, l, 0>::TH;                       \
            *tw = Tile<MISR_SCALE, l, 0>::TW;                       \
            return 1;                                               \
        }                                                           \
        return 0;                                                   \
    }
    MISR_LIST(X)
#undef X
    return 0;
}

int MISR_FN(tile_dims_trial_s)(int key, int *th, int *tw) {
    if (!MISR_FN(tile_dims_s)(key, th, tw)) return 0;
    const int Lp = key & 255;
#define X(l)                                         \
    if (Lp == l && (key >> 8) == 2) {                \
        *th = Tile<MISR_SCALE, l, 2>::TH;            \
        *tw = Tile<MISR_SCALE, l, 2>::TW;            \
    }
    MISR_LIST(X)
#undef X
    return 1;
}

// code = st_code(x storage, y storage): the frames share the iterate's
// storage, or the iterate is FP32 over 16-bit frames.
#define MISR_CODES(LAUNCH, l)                         \
    if (code == st_code(ST_F32, ST_F32))              \
        LAUNCH(l, StF32, StF32);                      \
    else if (code == st_code(ST_F16, ST_F16))         \
        LAUNCH(l, StF16, StF16);                      \
    else if (code == st_code(ST_BF16, ST_BF16))       \
        LAUNCH(l, StBF16, StBF16);                    \
    else if (code == st_code(ST_F32, ST_F16))         \
        LAUNCH(l, StF32, StF16);                      \
    else if (code == st_code(ST_F32, ST_BF16))        \
        LAUNCH(l, StF32, StBF16);                     \
    else if (code == st_code(ST_F32, ST_U16))         \
        LAUNCH(l, StF32, StU16);                      \
    else                                              \
        return hipErrorInvalidValue;

hipError_t MISR_FN(launch_trial_s)(int key, int code, int grid, hipStream_t s, const Proj *projs,
                                   const Item *items, const int *n_items, double *partials,
                                   int mode) {
    if ((key >> 8) > 2) return hipErrorInvalidValue;
    const int Lp = key & 255;
#define LAUNCH(l, SX, SY)                                                                    \
    hipLaunchKernelGGL((k_trial<MISR_SCALE, l, tv, SX, SY>), dim3(grid), dim3(kNTI), 0, s, \
                       projs, items, n_items, partials, mode)
#define X(l)                                        \
    if (Lp == l) {                                  \
        MISR_VARIANT_TRIAL(key, MISR_CODES(LAUNCH, l))    \
        return hipGetLastError();                   \
    }
    MISR_LIST(X)
#undef X
#undef LAUNCH
    return hipErrorInvalidValue;
}

hipError_t MISR_FN(launch_upcurv_s)(int key, int code, int grid, hipStream_t s, const Proj *projs,
                                    const Item *items, const int *n_items,
                                    double *partials) {
    if ((key >> 8) > 2) return hipErrorInvalidValue;
    const int Lp = key & 255;
#define LAUNCH(l, SX, SY)                                                                     \
    hipLaunchKernelGGL((k_upcurv<MISR_SCALE, l, tv, SX, SY>), dim3(grid), dim3(kNTI), 0, s, \
                       projs, items, n_items, partials)
#define X(l)                                        \
    if (Lp == l) {                                  \
        MISR_VARIANT(key, MISR_CODES(LAUNCH, l))    \
        return hipGetLastError();                   \
    }
    MISR_LIST(X)
#undef X
#undef LAUNCH
    return hipErrorInvalidValue;
}

#define MISR_STYPES(LAUNCH, l)          \
    if (stype == ST_F32)                \
        LAUNCH(l, StF32);               \
    else if (stype == ST_F16)           \
        LAUNCH(l, StF16);               \
    else                                \
        LAUNCH(l, StBF16);

hipError_t MISR_FN(launch_forward_s)(int key, int stype, int grid, hipStream_t s, const Proj *projs,
                                     const Item *items, int n, const void *x, void *y) {
    if ((key >> 8) > 2) return hipErrorInvalidValue;
    const int Lp = key & 255;
#define LAUNCH(l, ST)                                                                            \
    hipLaunchKernelGGL((k_forward<MISR_SCALE, l, tv, ST>), dim3(grid), dim3(kNTI), 0, s, projs, \
                       items, n, x, y)
#define X(l)                                         \
    if (Lp == l) {                                   \
        MISR_VARIANT(key, MISR_STYPES(LAUNCH, l))    \
        return hipGetLastError();                    \
    }
    MISR_LIST(X)
#undef X
#undef LAUNCH
    return hipErrorInvalidValue;
}

hipError_t MISR_FN(launch_adjoint_s)(int key, int stype, int grid, hipStream_t s, const Proj *projs,
                                     const Item *items, int n, const void *r, float *x) {
    if ((key >> 8) > 2) return hipErrorInvalidValue;
    const int Lp = key & 255;
#define LAUNCH(l, ST)                                                                            \
    hipLaunchKernelGGL((k_adjoint<MISR_SCALE, l, tv, ST>), dim3(grid), dim3(kNTI), 0, s, projs, \
                       items, n, r, x)
#define X(l)                                         \
    if (Lp == l) {                                   \
        MISR_VARIANT(key, MISR_STYPES(LAUNCH, l))    \
        return hipGetLastError();                    \
    }
    MISR_LIST(X)
#undef X
#undef LAUNCH
    return hipErrorInvalidValue;
}

}  // namespace misr
