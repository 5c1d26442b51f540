// general_kernels.hip -- the SCG hot path for general operators: per-frame
// affine warps M_k and non-separable PSFs B_k (A_k = D B_k M_k of Eq. sisr
// with general factors), where A_k is not a Kronecker product of two banded
// 1-D operators and the band kernels do not apply.
//
// Matrix-free form (OpDev::mf): A_k is applied from its factors.  Forward,
// per LR tile: the warped image z = M_k v on the HR window the tile's outputs
// read is built in LDS (bilinear samples of v, zero off the grid), then each
// LR pixel takes its Q x Q window of z times the frame's blur-and-bin kernel
// C_k (B_k's P x P PSF convolved with D's s x s box, over s^2).  Adjoint, per
// HR tile: per frame the residual window is staged in LDS, the
// back-projection w = B_k^T D^T r_k is formed on the HR window the tile's
// pixels gather from (the preimage of the tile under the warp), and each
// pixel sums w over the positions whose warped coordinates lie within one
// pixel of it, times the bilinear (tent) weights: the transpose of the
// forward's sampling, gathered rather than scattered, so each output is a
// fixed-order sum.  Per pass and HR pixel this reads x, p (and the frames)
// once instead of the sparse matrices' entries.
//
// Stored form (warps whose windows exceed the LDS, or on request):
// A = [A_0; ...; A_{K-1}] is held as an ELL matrix over the K h w LR rows and
// its transpose over the H W HR rows (built once per operator on the host,
// entry q of row r at [q * rows + r], so a wave reads each entry slot of 64
// consecutive rows in one coalesced access).  One thread per row, kGenRows
// rows per work item.
//
// The launches of a pass share one item list, and each takes the items of its
// role (item.tx).  The trial evaluates the LR rows (forward at x + alpha p,
// residual, data cost) and the HR rows (adjoint of the residual, BTV prior,
// gradient and inner products); the update pass the HR rows (x, p update,
// prior curvature) and the LR rows (data curvature along the new p).  Stored
// form: two launches each, as the second reads what the first wrote.
// Matrix-free: one each, since A x and A p are kept (the residual at
// x + alpha p is formed as its window is staged) and the LR tiles form the
// new p = beta p - g as they sample it.  The kernels are compiled per scale;
// a batch launches once per form and scale.  Views are FP32 and untiled.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_common.h"

namespace misr {

// The 8 BTV offsets d = (dx, dy) in [0, 2]^2 minus the origin (Eq. prior).
__device__ constexpr int kGX[8] = {1, 2, 0, 1, 2, 0, 1, 2};
__device__ constexpr int kGY[8] = {0, 0, 1, 1, 1, 2, 2, 2};

typedef float f32x4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------ matrix-free

// (M_k v)(u, v) from the warped coordinate (r, c) of HR pixel (u, v): the
// bilinear sample of v; zero off the grid, corners off the grid weigh
// nothing.  The corners are read at clamped positions, unconditionally, so
// that a thread keeps the loads of several samples in flight (behind a branch
// per corner they waited for each other), and count as zero off the grid.
struct MfSample {
    int at[4];
    bool ok[4];
    float fa, fb;
};
FI MfSample mf_corners(int H, int W, int u, int v, double r, double c) {
    MfSample s;
    const double r0 = floor(r), c0 = floor(c);
    s.fa = (float)(r - r0);
    s.fb = (float)(c - c0);
    // clamped before the conversion: a corner beyond the grid weighs nothing
    const int ir = (int)fmin(fmax(r0, -2.0), (double)H + 1.0);
    const int ic = (int)fmin(fmax(c0, -2.0), (double)W + 1.0);
    const bool in = u >= 0 && u < H && v >= 0 && v < W;
    const bool r0k = in && ir >= 0 && ir < H, r1k = in && ir + 1 >= 0 && ir + 1 < H;
    const bool c0k = ic >= 0 && ic < W, c1k = ic + 1 >= 0 && ic + 1 < W;
    const int ra = min(max(ir, 0), H - 1) * W, rb = min(max(ir + 1, 0), H - 1) * W;
    const int ca = min(max(ic, 0), W - 1), cb = min(max(ic + 1, 0), W - 1);
    s.at[0] = ra + ca;
    s.at[1] = ra + cb;
    s.at[2] = rb + ca;
    s.at[3] = rb + cb;
    s.ok[0] = r0k && c0k;
    s.ok[1] = r0k && c1k;
    s.ok[2] = r1k && c0k;
    s.ok[3] = r1k && c1k;
    return s;
}
FI float mf_bilinear(const MfSample &s, const float (&v)[4]) {
    float acc = 0.f;
    acc = fmaf((1.f - s.fa) * (1.f - s.fb), s.ok[0] ? v[0] : 0.f, acc);
    acc = fmaf((1.f - s.fa) * s.fb, s.ok[1] ? v[1] : 0.f, acc);
    acc = fmaf(s.fa * (1.f - s.fb), s.ok[2] ? v[2] : 0.f, acc);
    return fmaf(s.fa * s.fb, s.ok[3] ? v[3] : 0.f, acc);
}

// Tile q of LR item t: an item takes kMfLRG consecutive tiles of one frame
// (frames in turn, tiles row-major); frame, tile row and column, or false
// past the frame's last tile.
FI bool mf_lr_tile(const AS4 OpDev &op, int t, int q, int &k, int &ti, int &tj) {
    const int h = op.H / op.s, w = op.W / op.s, TI = mf_ti(op.s);
    const int nti = (h + TI - 1) / TI, ntj = (w + kMfTJ - 1) / kMfTJ;
    const int ng = (nti * ntj + kMfLRG - 1) / kMfLRG;
    k = t / ng;
    const int c = (t - k * ng) * kMfLRG + q;
    if (c >= nti * ntj) return false;
    ti = c / ntj;
    tj = c - ti * ntj;
    return true;
}

// e / d for 0 <= e < 2^21, d >= 1, through the float reciprocal inv = 1 / d:
// (e + 1/2) / d lies at least 1/(2 d) from an integer, well above the
// product's rounding error, so the truncation is exact.
FI int mf_div(int e, float inv) { return (int)(((float)e + 0.5f) * inv); }

// The two LR pixels' Q x Q windows times the kernel ck: window row a is row a
// of the first pixel and row a - S of the second.  PSFs of up to 7 taps are
// unrolled whole, larger ones by rows, so that a row's weights and window reads
// are in flight together (with Q a variable and four columns at a time, the
// forward of 2 frames of 330 x 410 at s = 3 with 15-tap PSFs took 48 us, now 24).
template <int S, int Q>
FI void mf_conv(const float *zb, int ZC, const AS4 float *ck, float (&acc)[kMfCPT]) {
    if constexpr (Q <= S + 6) {
#pragma unroll
        for (int a = 0; a < Q + S; ++a)
#pragma unroll
            for (int b = 0; b < Q; ++b) {
                const float z = zb[a * ZC + b];
                if (a < Q) acc[0] = fmaf(ck[a * Q + b], z, acc[0]);
                if (a >= S) acc[1] = fmaf(ck[(a - S) * Q + b], z, acc[1]);
            }
    } else {
#pragma unroll 1
        for (int a = 0; a < Q + S; ++a) {
            float z[Q];
#pragma unroll
            for (int b = 0; b < Q; ++b) z[b] = zb[a * ZC + b];
            if (a < Q) {
#pragma unroll
                for (int b = 0; b < Q; ++b) acc[0] = fmaf(ck[a * Q + b], z[b], acc[0]);
            }
            if (a >= S) {
#pragma unroll
                for (int b = 0; b < Q; ++b) acc[1] = fmaf(ck[(a - S) * Q + b], z[b], acc[1]);
            }
        }
    }
}

// (A_k v) at this thread's LR pixels of LR tile (ti, tj) of frame k: rows
// i + c, c < kMfCPT, of column j, into out[c] (pixels past the frame are
// computed and not used: the caller checks i + c < h, j < w).  zs: the
// warped window, free again on return.  vec(base, c): element base + c of v.
//
// The window's samples bound the forward (two FP64 coordinates, four corner
// loads each): kMfSU of them per thread are in flight together.  Two rows of
// a column share S fewer than Q of the window rows they read.
// With both, k_mf_upd on a 1024^2 image (s = 2, 4 frames, Q = 8) takes 36 us
// for what took two launches of 25 + 20; the taps, read from memory by every
// lane of a wave alike, were half of that chain before mf_conv had Q known.
constexpr int kMfSU = 4;
template <int S, class V>
FI void mf_forward(const AS4 OpDev &op, int k, int ti, int tj, V vec, float *zs, int &i, int &j,
                   float (&out)[kMfCPT]) {
    constexpr int TI = mf_ti(S);
    static_assert(kMfCPT == 2 && TI * kMfTJ == kMfCPT * kGenRows, "two rows per thread");
    const int H = op.H, W = op.W, Q = op.Q, R = (op.P - 1) / 2;
    const int i0 = ti * TI, j0 = tj * kMfTJ;
    const int ZR = S * (TI - 1) + Q, ZC = S * (kMfTJ - 1) + Q;
    const int u0 = S * i0 - R, v0 = S * j0 - R;
    const double m0 = op.gm[k][0], m1 = op.gm[k][1], m2 = op.gm[k][2];
    const double m3 = op.gm[k][3], m4 = op.gm[k][4], m5 = op.gm[k][5];
    const float izc = 1.f / (float)ZC;
    const int nz = ZR * ZC;
    // the window's extent under the warp (affine: at its corners); where the
    // window and every corner of its samples lie on the grid, the samples need
    // no bounds, and their addresses are 32-bit offsets from the first where
    // the rows they span hold few enough elements (an enlarging warp of a very
    // wide image spans more)
    double rmin = 1e300, rmax = -1e300, cmin = 1e300, cmax = -1e300;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const double u = (q & 1) ? u0 + ZR - 1 : u0, v = (q & 2) ? v0 + ZC - 1 : v0;
        const double r = fma(m0, u, fma(m1, v, m2)), c = fma(m3, u, fma(m4, v, m5));
        rmin = fmin(rmin, r);
        rmax = fmax(rmax, r);
        cmin = fmin(cmin, c);
        cmax = fmax(cmax, c);
    }
    constexpr double kTol = 1e-6;   // (above the corners' own rounding)
    if (u0 >= 0 && v0 >= 0 && u0 + ZR <= H && v0 + ZC <= W && rmin >= kTol && cmin >= kTol &&
        rmax <= H - 1 - kTol && cmax <= W - 1 - kTol &&
        (rmax - rmin + 3.0) * W < kAt32Elems) {
        const int rb = uni((int)rmin), cb = uni((int)cmin);
        const i64 base = (i64)rb * W + cb;
        for (int e0 = threadIdx.x; e0 < nz; e0 += kMfSU * kGenRows) {
            float fa[kMfSU], fb[kMfSU], val[kMfSU][4];
#pragma unroll
            for (int n = 0; n < kMfSU; ++n) {
                const int e = min(e0 + n * kGenRows, nz - 1);
                const int a = mf_div(e, izc), b = e - a * ZC;
                const double u = u0 + a, v = v0 + b;
                const double r = fma(m0, u, fma(m1, v, m2)), c = fma(m3, u, fma(m4, v, m5));
                const double r0 = floor(r), c0 = floor(c);
                fa[n] = (float)(r - r0);
                fb[n] = (float)(c - c0);
                const unsigned at = (unsigned)(((int)r0 - rb) * W + (int)c0 - cb);
                val[n][0] = vec(base, at);
                val[n][1] = vec(base, at + 1);
                val[n][2] = vec(base, at + W);
                val[n][3] = vec(base, at + W + 1);
            }
#pragma unroll
            for (int n = 0; n < kMfSU; ++n) {
                float acc = 0.f;
                acc = fmaf((1.f - fa[n]) * (1.f - fb[n]), val[n][0], acc);
                acc = fmaf((1.f - fa[n]) * fb[n], val[n][1], acc);
                acc = fmaf(fa[n] * (1.f - fb[n]), val[n][2], acc);
                acc = fmaf(fa[n] * fb[n], val[n][3], acc);
                if (e0 + n * kGenRows < nz) zs[e0 + n * kGenRows] = acc;
            }
        }
    } else {
        for (int e0 = threadIdx.x; e0 < nz; e0 += kMfSU * kGenRows) {
            MfSample s[kMfSU];
            float val[kMfSU][4];
#pragma unroll
            for (int n = 0; n < kMfSU; ++n) {
                const int e = min(e0 + n * kGenRows, nz - 1);
                const int a = mf_div(e, izc), b = e - a * ZC;
                const double u = u0 + a, v = v0 + b;
                s[n] = mf_corners(H, W, u0 + a, v0 + b, fma(m0, u, fma(m1, v, m2)),
                                  fma(m3, u, fma(m4, v, m5)));
#pragma unroll
                for (int q = 0; q < 4; ++q) val[n][q] = vec(s[n].at[q], 0u);
            }
#pragma unroll
            for (int n = 0; n < kMfSU; ++n)
                if (e0 + n * kGenRows < nz) zs[e0 + n * kGenRows] = mf_bilinear(s[n], val[n]);
        }
    }
    __syncthreads();
    const int il = kMfCPT * (threadIdx.x / kMfTJ), jl = threadIdx.x % kMfTJ;
    const AS4 float *ck = cst(op.gker) + (i64)k * Q * Q;
    const float *zb = zs + S * il * ZC + S * jl;
    float acc[kMfCPT] = {0.f, 0.f};
    if (Q == S + 6)
        mf_conv<S, S + 6>(zb, ZC, ck, acc);
    else if (Q == S + 4)
        mf_conv<S, S + 4>(zb, ZC, ck, acc);
    else
        switch (op.P) {   // uniform; odd, at most 15 (misr_geometry_check)
        case 1: mf_conv<S, S>(zb, ZC, ck, acc); break;
        case 3: mf_conv<S, S + 2>(zb, ZC, ck, acc); break;
        case 9: mf_conv<S, S + 8>(zb, ZC, ck, acc); break;
        case 11: mf_conv<S, S + 10>(zb, ZC, ck, acc); break;
        case 13: mf_conv<S, S + 12>(zb, ZC, ck, acc); break;
        default: mf_conv<S, S + 14>(zb, ZC, ck, acc); break;
        }
    __syncthreads();
    i = i0 + il;
    j = j0 + jl;
#pragma unroll
    for (int c = 0; c < kMfCPT; ++c) out[c] = acc[c];
}

// Clamped conversion of a window bound (the operator's windows are small,
// the clamp only keeps the conversion defined).
FI int mf_int(double v) { return (int)fmin(fmax(v, -1073741824.0), 1073741824.0); }

constexpr int kMfRR = 4;   // rows of a residual window per wave, loaded a frame ahead
struct MfGeo {
    int i[4];     // the back-projection window: ua, va, ub, vb
    float f[4];   // tile-relative origins: preimage (u, v), warped (r, c)
};
FI float readlane_f(float v, int k) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k));
}

// acc[t] += sum_k (A_k^T r_k)(pixel) for this thread's four pixels of HR
// tile (tu, tv) (rows tu kMfTU + threadIdx.x / 64 + 4 t, column
// tv kMfTV + threadIdx.x % 64); res.value(res.load(row, j)) gives r_k (LR
// row `row` of all frames' rows, times w).  lds: kMfWin floats
// plus kMfQP^2, free again on return.
//
// Per frame: the back-projection window [ua, ub] x [va, vb] holds every
// candidate position of every pixel of the tile (a pixel's candidates start
// at floor(u(p) - eu) + 1, ncu of them), so the gathers need no bounds
// checks; positions off the grid hold 0.  Position (u, v) takes the residual
// of LR pixels i = floor((u + R) / s) - t, t < NT = ceil(Q / s), with kernel
// row (u + R) mod s + s t (rows from Q on are zero in the padded copy), so
// every position runs the same NT x NT taps.
template <int S, class Rf>
FI void mf_adjoint(const AS4 OpDev &op, int tu, int tv, Rf res, float *lds, float (&acc)[4]) {
    const int H = op.H, W = op.W, Q = op.Q, R = (op.P - 1) / 2;
    const int h = H / S, w = W / S;
    const int NT = (Q + S - 1) / S;
    const int U0 = tu * kMfTU, V0 = tv * kMfTV;
    const int U1 = min(U0 + kMfTU, H) - 1, V1 = min(V0 + kMfTV, W) - 1;
    const int row = uni(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const bool full = U0 + kMfTU <= H && V0 + kMfTV <= W;   // (uniform)
    float *cpl = lds + kMfWin;
    // every frame's geometry at once, one frame per lane (in FP64 and the same
    // for the whole tile: computed frame by frame, by all lanes alike, it was
    // a serial chain at the head of each)
    MfGeo gl;
    {
        const int k = min(lane, op.K - 1);
        const double g0 = op.gi[k][0], g1 = op.gi[k][1], g2 = op.gi[k][2];
        const double g3 = op.gi[k][3], g4 = op.gi[k][4], g5 = op.gi[k][5];
        const double m0 = op.gm[k][0], m1 = op.gm[k][1], m2 = op.gm[k][2];
        const double m3 = op.gm[k][3], m4 = op.gm[k][4], m5 = op.gm[k][5];
        const double eu = op.eu[k], ev = op.ev[k];
        double umin = 1e300, umax = -1e300, vmin = 1e300, vmax = -1e300;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double pr = (q & 1) ? U1 : U0, pc = (q & 2) ? V1 : V0;
            const double uc = fma(g0, pr, fma(g1, pc, g2)), vc = fma(g3, pr, fma(g4, pc, g5));
            umin = fmin(umin, uc);
            umax = fmax(umax, uc);
            vmin = fmin(vmin, vc);
            vmax = fmax(vmax, vc);
        }
        const int ua = mf_int(floor(umin - eu)) + 1, va = mf_int(floor(vmin - ev)) + 1;
        gl.i[0] = ua;
        gl.i[1] = va;
        gl.i[2] = min(mf_int(floor(umax + eu)) + 1, ua + op.ru[k] - 1);
        gl.i[3] = min(mf_int(floor(vmax + ev)) + 1, va + op.rv[k] - 1);
        // tile-relative coordinates in FP32 (magnitudes of the tile's extent):
        // the preimage of the tile's corner pixel (U0, V0) less the window's
        // origin, and the warped coordinate of the window's origin less the
        // corner pixel, both from FP64 once per tile.  A rounding that moves a
        // pixel's first candidate by one position changes only candidates at
        // the edge of its support, whose tent weights are zero to rounding.
        gl.f[0] = (float)(fma(g0, (double)U0, fma(g1, (double)V0, g2)) - ua);
        gl.f[1] = (float)(fma(g3, (double)U0, fma(g4, (double)V0, g5)) - va);
        gl.f[2] = (float)(fma(m0, (double)ua, fma(m1, (double)va, m2)) - U0);
        gl.f[3] = (float)(fma(m3, (double)ua, fma(m4, (double)va, m5)) - V0);
    }
    // frame k's window: the LR pixels (i0, j0).. of NI x NJ; whether the tile
    // gathers from nothing on the grid (uniform)
    struct Win {
        int ua, va, ub, vb, i0, j0, NI, NJ;
        bool none, rows;
    };
    auto window = [&](int k) {
        Win n;
        n.ua = __builtin_amdgcn_readlane(gl.i[0], k);
        n.va = __builtin_amdgcn_readlane(gl.i[1], k);
        n.ub = __builtin_amdgcn_readlane(gl.i[2], k);
        n.vb = __builtin_amdgcn_readlane(gl.i[3], k);
        n.none = n.ub < 0 || n.ua > H - 1 || n.vb < 0 || n.va > W - 1;
        n.i0 = fdiv(n.ua + R, S) - NT + 1;
        n.j0 = fdiv(n.va + R, S) - NT + 1;
        n.NI = fdiv(n.ub + R, S) - n.i0 + 1;
        n.NJ = fdiv(n.vb + R, S) - n.j0 + 1;
        n.rows = n.NI <= 4 * kMfRR && n.NJ <= 64;
        return n;
    };
    // A residual window of up to 16 rows and 64 columns (scales from 2, warps
    // near the identity) is loaded by rows, one wave each, a frame ahead: its
    // loads pass under the frame before.
    typename Rf::Raw raw[kMfRR];
    auto load = [&](int k, const Win &n) {
        if (n.none || !n.rows) return;
        const int jc = min(max(n.j0 + lane, 0), w - 1);
#pragma unroll
        for (int q = 0; q < kMfRR; ++q) {
            const int i = min(max(n.i0 + min(row + 4 * q, n.NI - 1), 0), h - 1);
            raw[q] = res.load(((i64)k * h + i) * w, jc);
        }
    };
    // taps an LR pixel, per axis, of the product by cells below; 0: positions
    // one by one, at scale 1 (where a cell is a position and the taps are many),
    // for one tap, more than 5, and 5 at scale 4 (16 phases of 25 taps are four
    // loads of taps for about 100 cells a tile: adjoint of 4 frames of 330 x 410
    // with 15-tap PSFs 75.7 us by cells, 66.5 by positions)
    const int ntc = S > 1 && NT >= 2 && NT <= (S == 4 ? 4 : 5) ? NT : 0;
    Win nw = window(0);
    load(0, nw);
    for (int k = 0; k < op.K; ++k) {
        const Win n = nw;
        if (k + 1 < op.K) nw = window(k + 1);
        auto ahead = [&]() {
            if (k + 1 < op.K) load(k + 1, nw);
        };
        if (n.none) {
            ahead();
            continue;
        }
        const int ua = n.ua, va = n.va, ub = n.ub, vb = n.vb;
        const int RU = ub - ua + 1, RV = vb - va + 1;
        const int i0 = n.i0, j0 = n.j0, NI = n.NI, NJ = n.NJ;
        float *rsm = lds, *wt = lds + NI * NJ;
        const float inj = 1.f / (float)NJ;
        // the back-projection window: whole cells where cells() forms it and
        // those fit the LDS (no bounds per position but the grid's), else
        // [ua, ub] x [va, vb]; its origin and row stride
        const int uc = S * (i0 + NT - 1) - R, vc = S * (j0 + NT - 1) - R;
        const int RUC = S * (NI - NT + 1), RVC = S * (NJ - NT + 1);
        const bool whole = ntc > 0 && NI * NJ + RUC * RVC <= kMfWin;
        const int uw = whole ? uc : ua, vw = whole ? vc : va, RW = whole ? RVC : RV;
        if (n.rows) {
            const bool in_j = j0 + lane >= 0 && j0 + lane < w;
#pragma unroll
            for (int q = 0; q < kMfRR; ++q) {
                const int a = row + 4 * q;
                if (a < NI && lane < NJ)
                    rsm[a * NJ + lane] =
                        in_j && i0 + a >= 0 && i0 + a < h ? res.value(raw[q]) : 0.f;
            }
        } else {
            for (int e = threadIdx.x; e < NI * NJ; e += kGenRows) {
                const int a = mf_div(e, inj), i = i0 + a, j = j0 + e - a * NJ;
                rsm[e] = (i >= 0 && i < h && j >= 0 && j < w)
                             ? res.value(res.load(((i64)k * h + i) * w, j))
                             : 0.f;
            }
        }
        // The S x S positions of a cell (one LR pixel's block) take the same
        // NT x NT residuals, each position (phase) with its own taps: a
        // product of phases x taps with taps x cells, on the matrix cores in
        // blocks of 4 phases x 64 cells with one tap per instruction (FP32
        // fused multiply-adds in the taps' order, as one thread would sum
        // them).  A lane holds its cell's residuals and, of the taps, those of
        // phase lane % 4 of each block.
        auto cells = [&](auto nt) {
            constexpr int NTC = decltype(nt)::value, NP = S * S, G = (NP + 3) / 4;
            const AS1 float *cp = glb(op.gkp) + (i64)k * NP * NTC * NTC;
            const int m = threadIdx.x & 3;
            // blocks of phases taken together: as many as hold their taps in
            // 32 registers
            constexpr int GC = mf_cmax(1, 32 / (NTC * NTC));
            const int ncu = NI - NTC + 1, ncv = NJ - NTC + 1, nc = ncu * ncv;
            const int uo = S * (i0 + NTC - 1) - R, vo = S * (j0 + NTC - 1) - R;
            const float inv = 1.f / (float)ncv;
#pragma unroll
            for (int g0 = 0; g0 < G; g0 += GC) {
                float tap[GC][NTC * NTC];
#pragma unroll
                for (int g = 0; g < GC; ++g)
#pragma unroll
                    for (int q = 0; q < NTC * NTC; ++q)
                        tap[g][q] = cp[min(4 * (g0 + g) + m, NP - 1) * NTC * NTC + q];
                if (g0 == 0) {
                    ahead();
                    __syncthreads();
                }
                for (int e0 = 0; e0 < nc; e0 += kGenRows) {   // (uniform: every lane takes part)
                    const int e = min(e0 + (int)threadIdx.x, nc - 1);
                    const int cu = mf_div(e, inv), cv = e - cu * ncv;
                    const float *rr = rsm + (cu + NTC - 1) * NJ + cv + NTC - 1;
                    float rw[NTC * NTC];
#pragma unroll
                    for (int t = 0; t < NTC; ++t)
#pragma unroll
                        for (int t2 = 0; t2 < NTC; ++t2) rw[t * NTC + t2] = rr[-t * NJ - t2];
                    const int u0c = uo + S * cu, v0c = vo + S * cv;
                    float *wc = wt + (u0c - uw) * RW + v0c - vw;
                    // rows and columns of the cell inside the window and on the grid
                    bool inu[S], inv_[S], onu[S], onv[S];
#pragma unroll
                    for (int a = 0; a < S; ++a) {
                        inu[a] = whole || (u0c + a >= ua && u0c + a <= ub);
                        inv_[a] = whole || (v0c + a >= va && v0c + a <= vb);
                        onu[a] = u0c + a >= 0 && u0c + a < H;
                        onv[a] = v0c + a >= 0 && v0c + a < W;
                    }
#pragma unroll
                    for (int g = 0; g < GC; ++g) {
                        if (g0 + g >= G) break;
                        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int q = 0; q < NTC * NTC; ++q)
                            sum = __builtin_amdgcn_mfma_f32_4x4x1f32(tap[g][q], rw[q], sum, 0, 0, 0);
#pragma unroll
                        for (int n = 0; n < 4; ++n) {
                            const int ph = 4 * (g0 + g) + n, a = ph / S, b = ph % S;
                            if (ph >= NP) break;
                            const float val = onu[a] && onv[b] ? sum[n] : 0.f;
                            if (inu[a] && inv_[b]) wc[a * RW + b] = val;
                        }
                    }
                }
            }
        };
        // positions one by one, over [ua, ub] x [va, vb]; the taps' count is
        // known to the compiler where it is small (0: NT).  The phases' taps lie
        // an odd number of words apart: neighbouring positions are of different
        // phases, and an even square put them in the same bank.
        auto positions = [&](auto nt) {
            constexpr int NTC = decltype(nt)::value, UT = S == 1 ? 6 : 1;
            int n1 = NTC > 0 ? NTC : NT;
            if (NTC == 0) asm volatile("" : "+s"(n1));   // (nothing of this is kept across frames)
            const int n2 = n1 * n1, pst = n2 | 1, nk = S * S * n2;
            const float irv = 1.f / (float)RV;
            const AS1 float *cp = glb(op.gkp) + (i64)k * nk;
            if (S == 1 || pst == n2) {
                for (int e = threadIdx.x; e < nk; e += kGenRows) cpl[e] = cp[e];
            } else {
                const float in2 = 1.f / (float)n2;
                for (int e = threadIdx.x; e < nk; e += kGenRows)
                    cpl[e + mf_div(e, in2)] = cp[e];
            }
            ahead();
            __syncthreads();
            for (int e = threadIdx.x; e < RU * RV; e += kGenRows) {
                const int a = mf_div(e, irv);
                const int u = ua + a, v = va + e - a * RV;
                float sum = 0.f;
                if (u >= 0 && u < H && v >= 0 && v < W) {
                    const int qu = fdiv(u + R, S), qv = fdiv(v + R, S);
                    const float *cr = cpl + ((u + R - S * qu) * S + (v + R - S * qv)) * pst;
                    const float *rr = rsm + (qu - i0) * NJ + (qv - j0);
#pragma unroll UT
                    for (int t = 0; t < n1; ++t)
#pragma unroll 6
                        for (int t2 = 0; t2 < n1; ++t2)
                            sum = fmaf(cr[t * n1 + t2], rr[-t * NJ - t2], sum);
                }
                wt[e] = sum;
            }
        };
        switch (ntc) {   // uniform
        case 2: cells(std::integral_constant<int, 2>{}); break;
        case 3: cells(std::integral_constant<int, 3>{}); break;
        case 4: cells(std::integral_constant<int, 4>{}); break;
        case 5:
            if constexpr (S < 4) cells(std::integral_constant<int, 5>{});
            break;
        default:
            if (S == 1 && NT == 3)
                positions(std::integral_constant<int, 3>{});
            else if ((S == 1 || S == 4) && NT == 5)
                positions(std::integral_constant<int, 5>{});
            else
                positions(std::integral_constant<int, 0>{});
            break;
        }
        __syncthreads();
        const float m0f = (float)op.gm[k][0], m1f = (float)op.gm[k][1];
        const float m3f = (float)op.gm[k][3], m4f = (float)op.gm[k][4];
        const float g0f = (float)op.gi[k][0], g1f = (float)op.gi[k][1];
        const float g3f = (float)op.gi[k][3], g4f = (float)op.gi[k][4];
        const float euf = (float)op.eu[k], evf = (float)op.ev[k];
        const int ncu = op.ncu[k], ncv = op.ncv[k];
        const bool c33 = ncu == 3 && ncv == 3;   // the near-identity warps (uniform)
        const float ub0 = readlane_f(gl.f[0], k), vb0 = readlane_f(gl.f[1], k);
        const float rb0 = readlane_f(gl.f[2], k), cb0 = readlane_f(gl.f[3], k);
        const float rlim = (float)(RU - ncu), clim = (float)(RV - ncv), rwf = (float)RW;
        const float *w0 = wt + (ua - uw) * RW + va - vw;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int dr = row + 4 * t, dc = lane;
            if (!full && (U0 + dr > U1 || V0 + dc > V1)) continue;
            // first candidate, relative to the window's origin, kept inside
            // the window (a rounding at the edge moves it by one); whole
            // numbers below 2^24, exact in FP32
            const float uq = fmaf((float)dr, g0f, fmaf((float)dc, g1f, ub0)) - euf;
            const float vq = fmaf((float)dr, g3f, fmaf((float)dc, g4f, vb0)) - evf;
            const float ous = __builtin_amdgcn_fmed3f(floorf(uq) + 1.f, 0.f, rlim);
            const float ovs = __builtin_amdgcn_fmed3f(floorf(vq) + 1.f, 0.f, clim);
            // its warped coordinate relative to the pixel
            const float d0r = fmaf(ous, m0f, fmaf(ovs, m1f, rb0)) - (float)dr;
            const float d0c = fmaf(ous, m3f, fmaf(ovs, m4f, cb0)) - (float)dc;
            const float *wb = w0 + (int)fmaf(ous, rwf, ovs);
            float a_t = 0.f;
            auto cand = [&](int a, int b) {
                const float ar = a ? fmaf((float)a, m0f, d0r) : d0r;
                const float ac = a ? fmaf((float)a, m3f, d0c) : d0c;
                const float dr = b ? fmaf((float)b, m1f, ar) : ar;
                const float dc = b ? fmaf((float)b, m4f, ac) : ac;
                // (clamped below; 1 - |d| never exceeds 1: one instruction each)
                const float wgt = __builtin_amdgcn_fmed3f(1.f - fabsf(dr), 0.f, 1.f) *
                                  __builtin_amdgcn_fmed3f(1.f - fabsf(dc), 0.f, 1.f);
                a_t = fmaf(wgt, wb[a * RW + b], a_t);
            };
            if (c33) {
#pragma unroll
                for (int a = 0; a < 3; ++a)
#pragma unroll
                    for (int b = 0; b < 3; ++b) cand(a, b);
            } else {
                for (int a = 0; a < ncu; ++a)
                    for (int b = 0; b < ncv; ++b) cand(a, b);
            }
            acc[t] += a_t;
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------ stored form

// (A v)_r for ELL row r of `rows`, with v(c) given by f(c)
// (entries in groups of four, every load of a group issued before its
// arithmetic, so that a thread keeps several HBM requests in flight)
template <class F>
FI float ell_row(const AS1 int *col, const AS1 float *val, int width, i64 rows, i64 r, F f) {
    float acc = 0.f;
    int q = 0;
    for (; q + 4 <= width; q += 4) {
        int c[4];
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const i64 at = (i64)(q + e) * rows + r;
            c[e] = col[at];
            v[e] = val[at];
        }
        float g[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) g[e] = f(c[e]);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = fmaf(v[e], g[e], acc);
    }
    for (; q < width; ++q) {
        const i64 at = (i64)q * rows + r;
        acc = fmaf(val[at], f(col[at]), acc);
    }
    return acc;
}

// Residual term of LR row r (frame value y[r]) at forward value ax: the term
// the adjoint consumes (2 r, or psi(r) for the Charbonnier L1 term) and, in
// e, the data cost of the row.
FI float gen_residual(const AS4 ScgState &st, float y, float ax, double &e) {
    const float rr = ax - y * st.wt.y_scale;
    if (st.wt.data_p == 2) {
        e = (double)rr * (double)rr;
        return 2.f * rr;
    }
    const float epsd = st.wt.eps_data;
    float ph, ps;
    phi_psi(rr, epsd, epsd * epsd, ph, ps);
    e = (double)ph;
    return ps;
}

// Residuals for mf_adjoint: of the trial point (from A x + alpha A p as they
// are read), and as stored.
struct TrialRes {
    const AS4 ScgState &st;
    const AS1 float *y, *ax, *ap;
    float af;
    struct Raw {
        float y, ax, ap;
    };
    FI Raw load(i64 row, unsigned j) const {
        return {*at32(y + row, j), *at32(ax + row, j), *at32(ap + row, j)};
    }
    FI float value(const Raw &v) const {
        double e;
        return gen_residual(st, v.y, fmaf(af, v.ap, v.ax), e);
    }
};
struct StoredRes {
    const AS1 float *r;
    using Raw = float;
    FI Raw load(i64 row, unsigned j) const { return *at32(r + row, j); }
    FI float value(Raw v) const { return v; }
};

// BTV prior at HR pixel (ui, vi) of x_t, given at offsets (dy, dx) from the
// pixel by xo(dy, dx): adds its gradient to g and returns its cost over the
// pairs (i, i + d) owned by the pixel.
// FAST: every pair lies inside the image, and eps > 0 (no branch per pair).
template <bool FAST, class X>
FI float gen_prior(const AS4 ScgState &st, int H, int W, int ui, int vi, X xo, float &g) {
    const float x0 = xo(0, 0), eps = st.wt.eps, e2 = eps * eps;
    float eb = 0.f;
    auto pair = [&](float z, float &ph, float &ps) {
        if (FAST)
            phi_psi_pos(z, eps, e2, ph, ps);
        else
            phi_psi(z, eps, e2, ph, ps);
    };
#pragma unroll
    for (int d = 0; d < 8; ++d) {
        const int dx = kGX[d], dy = kGY[d];
        const float gam = st.wt.gam[dy * 3 + dx];
        float ph, ps;
        if (FAST || (ui + dy < H && vi + dx < W)) {   // pair (i, i + d), owned by i
            pair(x0 - xo(dy, dx), ph, ps);
            g = fmaf(gam, ps, g);
            eb = fmaf(gam, ph, eb);
        }
        if (FAST || (ui - dy >= 0 && vi - dx >= 0)) {   // pair (i - d, i)
            pair(xo(-dy, -dx) - x0, ph, ps);
            g = fmaf(-gam, ps, g);
        }
    }
    return eb;
}

// Prior part of Moller's curvature at the new (x, p) over the pairs owned by
// HR pixel (ui, vi): lambda sum gamma q^2 Q(z, sigma_k q), the new x and p
// at offsets (dy, dx) given by xo, po.
// FAST: every pair lies inside the image, and eps > 0: the pairs take the
// series of psi_quot; its closed form runs only for a pixel with a pair that
// needs it.
template <bool FAST, class X, class Pf>
FI float gen_prior_curv(const AS4 ScgState &st, int H, int W, int ui, int vi, X xo, Pf po) {
    const float x0 = xo(0, 0), p0 = po(0, 0);
    const float eps = st.wt.eps, e2 = eps * eps, sk = st.sigk_f;
    float a = 0.f;
    if (FAST) {
        float Qv[8], q[8], far = 0.f;
#pragma unroll
        for (int d = 0; d < 8; ++d) {
            const float z = x0 - xo(kGY[d], kGX[d]);
            q[d] = p0 - po(kGY[d], kGX[d]);
            const float rB = rsq(fmaf(z, z, e2)), h = sk * q[d];
            Qv[d] = psi_series(z, h, rB, e2);
            far = fmaxf(far, fabsf(h * rB));
        }
        if (!(far < 1e-3f)) {
#pragma unroll 1
            for (int d = 0; d < 8; ++d) {
                const float z = x0 - xo(kGY[d], kGX[d]), qd = p0 - po(kGY[d], kGX[d]);
                const float rB = rsq(fmaf(z, z, e2)), h = sk * qd;
                if (!(fabsf(h * rB) < 1e-3f)) {
                    const float c = psi_closed(z, h, rB, e2);
#pragma unroll
                    for (int n = 0; n < 8; ++n) Qv[n] = n == d ? c : Qv[n];
                }
            }
        }
#pragma unroll
        for (int d = 0; d < 8; ++d)
            a = fmaf(st.wt.gam[kGY[d] * 3 + kGX[d]] * q[d] * q[d], Qv[d], a);
        return a;
    }
#pragma unroll 1
    for (int d = 0; d < 8; ++d) {
        const int dx = kGX[d], dy = kGY[d];
        if (ui + dy < H && vi + dx < W) {
            const float z = x0 - xo(dy, dx), q = p0 - po(dy, dx);
            a = fmaf(st.wt.gam[dy * 3 + dx] * q * q, psi_quot(z, sk * q, eps, e2), a);
        }
    }
    return a;
}

// Update at HR pixel u = (ui, vi) of the stored form: x <- x + alpha p,
// p <- -g_t + beta p into the other buffers; returns the prior part of the
// curvature at the new (x, p), with |p|^2 and p.r.
FI float gen_update(const AS4 ScgState &st, const AS4 Proj &P, int H, int W, i64 u, int ui, int vi,
                    double &pp, double &pr) {
    const int src = st.upd_src, dst = src ^ 1;
    const AS1 float *x = glb((const float *)P.x[src]);
    const AS1 float *p = glb(P.p[src]);
    const AS1 float *gt = glb(P.g[st.cur]);
    const float af = st.alpha_f, bf = st.beta_f;
    auto xn = [&](int dy, int dx) {
        const i64 c = u + (i64)dy * W + dx;
        return fmaf(af, p[c], x[c]);
    };
    auto pn = [&](int dy, int dx) {
        const i64 c = u + (i64)dy * W + dx;
        return fmaf(bf, p[c], -gt[c]);
    };
    const float x0 = xn(0, 0), p0 = pn(0, 0);
    glbw((float *)P.x[dst])[u] = x0;
    glbw(P.p[dst])[u] = p0;
    pp += (double)p0 * (double)p0;
    pr += -(double)p0 * (double)gt[u];
    return gen_prior_curv<false>(st, H, W, ui, vi, xn, pn);
}

// Data part of the curvature of one LR row at A p (ap) and A x (ax) of the
// new iterate: 2 (A_k p)^2 for the L2 term, (A_k p)^2 Q(A_k x - y_k,
// sigma_k A_k p) for the Charbonnier L1 term.
FI double gen_data_curv(const AS4 ScgState &st, const AS4 Proj &P, i64 r, float ap, float ax) {
    if (st.wt.data_p == 2) return 2.0 * (double)ap * (double)ap;
    const float rr = ax - glb((const float *)P.y)[r] * st.wt.y_scale;
    const float epsd = st.wt.eps_data;
    return (double)(ap * ap * psi_quot(rr, st.sigk_f * ap, epsd, epsd * epsd));
}

// trial / cost+gradient, LR rows (an LR tile, or kGenRows ELL rows): the
// forward at x_t = x + alpha p (mode 1) or x (mode 0), the residual term and
// the data cost.  Matrix-free (mode 0 only): applies A to x and keeps A x (and
// A p = 0 for the zero start direction) for the trials, which take
// A x + alpha A p from the kept vectors (A is linear) with no forward.
template <int S>
__global__ void __launch_bounds__(kGenRows) k_gen_trial_lr(const Proj *projs, const Item *items,
                                                           const int *n_items, double *partials,
                                                           int mode) {
    __shared__ double red[kNV * (kGenRows / 64)];
    extern __shared__ float zs[];   // the forward's warped window, sized by the launch
    const int it = blockIdx.x;
    if (it >= *cst(n_items)) return;
    const AS4 Item &itm = cst(items)[it];
    if (itm.tx != 0) return;
    const AS4 Proj &P = cst(projs)[itm.proj];
    const AS4 ScgState &st = *cst(P.st);
    if (mode == 1 && !st.active) return;
    const AS4 OpDev &op = *cst(P.op);
    const int h = op.H / op.s, w = op.W / op.s;
    const int xc = st.xc;
    const AS1 float *x = glb((const float *)P.x[xc]);
    const AS1 float *p = glb(P.p[xc]);
    const float af = (mode == 1) ? st.alpha_f : 0.f;
    double e = 0.0, er;
    if (op.mf) {
        int k, ti, tj, i, j;
        {
            for (int q = 0; q < kMfLRG && mf_lr_tile(op, itm.ty, q, k, ti, tj); ++q) {
                float ax[kMfCPT];
                mf_forward<S>(op, k, ti, tj, [&](i64 b, unsigned c) { return *at32(x + b, c); }, zs, i,
                              j, ax);
#pragma unroll
                for (int c = 0; c < kMfCPT; ++c)
                    if (i + c < h && j < w) {
                        const i64 row = ((i64)k * h + i + c) * w + j;
                        glbw(P.res)[row] = gen_residual(st, glb((const float *)P.y)[row], ax[c], er);
                        e += er;
                        glbw(P.ax[xc])[row] = ax[c];
                        glbw(P.ap[xc])[row] = 0.f;
                    }
            }
        }
    } else {
        const i64 rows = (i64)op.K * h * w;
        const i64 r = (i64)itm.ty * kGenRows + threadIdx.x;
        // mode 0 reads x alone: p is not yet initialised there
        if (r < rows) {
            glbw(P.res)[r] = gen_residual(
                st, glb((const float *)P.y)[r],
                ell_row(glb(op.a_col), glb(op.a_val), op.a_w, rows, r,
                        [&](i64 c) { return mode == 1 ? fmaf(af, p[c], x[c]) : x[c]; }),
                er);
            e = er;
        }
    }
    double v[5] = {e, 0.0, 0.0, 0.0, 0.0};
    block_sum_store<5, kGenRows>(v, partials + (i64)it * kNV, red);
}

// trial / cost+gradient, HR rows (an HR tile, or kGenRows ELL rows):
// g_t = A^T (residual term) + the BTV gradient at x_t; writes g_t to
// g[cur ^ 1] with {E_data, E_reg, |g_t|^2, g_t.g_k, g_t.p} (mode 0: p[xc] = 0,
// the start direction buffer).  Matrix-free, mode 1: the residual is formed
// from A x + alpha A p as its window is staged (LR pixels shared by
// neighbouring tiles by each of them), so the trial is this one launch; the
// data cost goes by the LR items, each of which counts kGenRows kMfCPT rows.
// Bound by instructions (the prior's eight pairs, the 9 candidates of each
// pixel and frame) with waits at three barriers a frame: the matrix-core cells,
// a frame's residuals loaded under the frame before, the geometry of all
// frames at once.  1024^2 image, s = 2, 4 frames: 48 us after a 7 us launch
// that only formed the residual -> 41 us in all; 633 x 909, s = 3, 9 frames,
// mode 0: 81 -> 56 us.
template <int S>
__global__ void __launch_bounds__(kGenRows) k_gen_trial_hr(const Proj *projs, const Item *items,
                                                           const int *n_items, double *partials,
                                                           int mode) {
    __shared__ double red[kNV * (kGenRows / 64)];
    __shared__ float lds[kMfWin + kMfQP * kMfQP];
    // from the end of the list, where a solve's HR tiles are: they take 20 us
    // and its LR items 4, which fill in behind them (LR items first: 44.4 us
    // on a 1024^2 image, HR tiles first: 40.6)
    const int it = *cst(n_items) - 1 - (int)blockIdx.x;
    if (it < 0) return;
    const AS4 Item &itm = cst(items)[it];
    const AS4 Proj &P = cst(projs)[itm.proj];
    const AS4 OpDev &op = *cst(P.op);
    if (itm.tx != 1 && !(op.mf && mode == 1)) return;
    const AS4 ScgState &st = *cst(P.st);
    if (mode == 1 && !st.active) return;
    const int H = op.H, W = op.W, h = H / op.s, w = W / op.s;
    const i64 n = (i64)H * W;
    const int xc = st.xc, cur = st.cur;
    const AS1 float *x = glb((const float *)P.x[xc]);
    const AS1 float *p = glb(P.p[xc]);
    const AS1 float *res = glb((const float *)P.res);
    const AS1 float *ax = glb((const float *)P.ax[xc]), *ap = glb((const float *)P.ap[xc]);
    const float af = (mode == 1) ? st.alpha_f : 0.f;
    auto xt = [&](i64 c) { return mode == 1 ? fmaf(af, p[c], x[c]) : x[c]; };
    double ed = 0.0, er = 0.0, gg = 0.0, ggk = 0.0, gp = 0.0;
    if (itm.tx != 1) {
        // data cost: item t takes LR rows [t B, (t + 1) B), B = kGenRows kMfCPT
        // (there are at least as many LR items as such blocks)
#pragma unroll
        for (int c = 0; c < kMfCPT; ++c) {
            const i64 r = ((i64)itm.ty * kMfCPT + c) * kGenRows + threadIdx.x;
            double e;
            if (r < (i64)op.K * h * w) {
                (void)gen_residual(st, glb((const float *)P.y)[r], fmaf(af, ap[r], ax[r]), e);
                ed += e;
            }
        }
        double v[5] = {ed, 0.0, 0.0, 0.0, 0.0};
        block_sum_store<5, kGenRows>(v, partials + (i64)it * kNV, red);
        return;
    }
    // gradient of one pixel from its data part: prior (x_t at offsets from
    // the pixel given by xo), store, inner products (gk, pk: g_k and p there)
    auto finish = [&](i64 u, int ui, int vi, float g, auto xo, auto fast, float gk, float pk) {
        er += (double)gen_prior<decltype(fast)::value>(st, H, W, ui, vi, xo, g);
        glbw(P.g[cur ^ 1])[u] = g;
        gg += (double)g * (double)g;
        if (mode == 1) {
            ggk += (double)g * (double)gk;
            gp += (double)g * (double)pk;
        } else {
            glbw(P.p[xc])[u] = 0.f;
        }
    };
    if (op.mf) {
        const int ntv = (W + kMfTV - 1) / kMfTV;
        const int tu = itm.ty / ntv, tv = itm.ty - tu * ntv;
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
        {
            if (mode == 1)
                mf_adjoint<S>(op, tu, tv, TrialRes{st, glb((const float *)P.y), ax, ap, af}, lds,
                              acc);
            else
                mf_adjoint<S>(op, tu, tv, StoredRes{res}, lds, acc);
        }
        // x_t on the tile and two pixels around it, for the prior's pairs,
        // and g_k, p of the thread's pixels: every load before its use
        constexpr int WR = kMfTU + 4, WC = kMfTV + 4, NE = (WR * WC + kGenRows - 1) / kGenRows;
        const int U0 = tu * kMfTU - 2, V0 = tv * kMfTV - 2;
        float gk[4] = {0.f, 0.f, 0.f, 0.f}, pk[4] = {0.f, 0.f, 0.f, 0.f};
        if (mode == 1) {
            const AS1 float *gc = glb(P.g[cur]);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int pr = min(tu * kMfTU + (int)(threadIdx.x >> 6) + 4 * t, H - 1);
                const int pc = min(tv * kMfTV + (int)(threadIdx.x & 63), W - 1);
                gk[t] = gc[(i64)pr * W + pc];
                pk[t] = p[(i64)pr * W + pc];
            }
        }
        float xw[NE];
#pragma unroll
        for (int n = 0; n < NE; ++n) {
            const int e = threadIdx.x + n * kGenRows, a = e / WC, u = U0 + a, v = V0 + e - a * WC;
            const float t = xt((i64)min(max(u, 0), H - 1) * W + min(max(v, 0), W - 1));
            xw[n] = (u >= 0 && u < H && v >= 0 && v < W) ? t : 0.f;
        }
#pragma unroll
        for (int n = 0; n < NE; ++n)
            if (threadIdx.x + n * kGenRows < WR * WC) lds[threadIdx.x + n * kGenRows] = xw[n];
        __syncthreads();
        auto pixel = [&](int t, float at, auto fast, float gkt, float pkt) {
            const int a = (threadIdx.x >> 6) + 4 * t, b = threadIdx.x & 63;
            const int pr = tu * kMfTU + a, pc = tv * kMfTV + b;
            const float *wp = lds + (a + 2) * WC + b + 2;
            if (decltype(fast)::value || (pr < H && pc < W))
                finish((i64)pr * W + pc, pr, pc, at,
                       [&](int dy, int dx) { return wp[dy * WC + dx]; }, fast, gkt, pkt);
        };
        if (U0 >= 0 && V0 >= 0 && U0 + WR <= H && V0 + WC <= W && st.wt.eps != 0.f) {
#pragma unroll
            for (int t = 0; t < 4; ++t) pixel(t, acc[t], std::true_type{}, gk[t], pk[t]);
        } else {
#pragma unroll 1
            for (int t = 0; t < 4; ++t) {
                auto at = [&](const float (&v)[4]) {
                    return t == 0 ? v[0] : t == 1 ? v[1] : t == 2 ? v[2] : v[3];
                };
                pixel(t, at(acc), std::false_type{}, at(gk), at(pk));
            }
        }
    } else {
        const i64 u = (i64)itm.ty * kGenRows + threadIdx.x;
        if (u < n) {
            const int ui = (int)(u / W), vi = (int)(u - (i64)ui * W);
            const float gk = mode == 1 ? glb(P.g[cur])[u] : 0.f, pk = mode == 1 ? p[u] : 0.f;
            finish(u, ui, vi, ell_row(glb(op.t_col), glb(op.t_val), op.t_w, n, u,
                                      [&](int c) { return res[c]; }),
                   [&](int dy, int dx) { return xt(u + (i64)dy * W + dx); }, std::false_type{},
                   gk, pk);
        }
    }
    double v[5] = {0.0, er, gg, ggk, gp};
    block_sum_store<5, kGenRows>(v, partials + (i64)it * kNV, red);
}

// matrix-free update of an HR tile: x <- x + alpha p,
// p <- -g_t + beta p (into the other buffer of each pair), with {prior
// curvature, |p|^2, p.r}: the prior part of Moller's curvature at the new
// (x, p), lambda sum gamma q^2 Q(z, sigma_k q) over the pairs (i, i + d)
// owned by i
FI void gen_upd_hr(const AS4 Item &itm, const AS4 Proj &P, const AS4 ScgState &st, const AS4 OpDev &op,
                   float *lds, double (&out)[4]) {
    const int H = op.H, W = op.W;
    double pp = 0.0, pr = 0.0;
    // the new x and p on the tile and the two pixels below and right of
    // it (the pairs a pixel owns), each formed once, every load first
    constexpr int WR = kMfTU + 2, WC = kMfTV + 2, NE = (WR * WC + kGenRows - 1) / kGenRows;
    float *xw = lds, *pw = lds + WR * WC;
    const int ntv = (W + kMfTV - 1) / kMfTV;
    const int tu = itm.ty / ntv, tv = itm.ty - tu * ntv;
    const int src = st.upd_src, dst = src ^ 1;
    const AS1 float *x = glb((const float *)P.x[src]);
    const AS1 float *p = glb(P.p[src]);
    const AS1 float *gt = glb(P.g[st.cur]);
    const float af = st.alpha_f, bf = st.beta_f;
    float xr[NE], pr0[NE], gr[NE];
#pragma unroll
    for (int n = 0; n < NE; ++n) {
        const int e = threadIdx.x + n * kGenRows, a = e / WC;
        const int u = min(tu * kMfTU + a, H - 1), v = min(tv * kMfTV + e - a * WC, W - 1);
        const i64 c = (i64)u * W + v;
        xr[n] = x[c];
        pr0[n] = p[c];
        gr[n] = gt[c];
    }
#pragma unroll
    for (int n = 0; n < NE; ++n) {
        const int e = threadIdx.x + n * kGenRows;
        if (e < WR * WC) {
            xw[e] = fmaf(af, pr0[n], xr[n]);
            pw[e] = fmaf(bf, pr0[n], -gr[n]);
        }
    }
    float g4[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int ui = min(tu * kMfTU + (int)(threadIdx.x >> 6) + 4 * t, H - 1);
        const int vi = min(tv * kMfTV + (int)(threadIdx.x & 63), W - 1);
        g4[t] = gt[(i64)ui * W + vi];
    }
    __syncthreads();
    const bool fast = (tu + 1) * kMfTU + 2 <= H && (tv + 1) * kMfTV + 2 <= W && st.wt.eps != 0.f;
    float a = 0.f;
    // (rolled: the eight pairs of a pixel are enough in flight)
#pragma unroll 1
    for (int t = 0; t < 4; ++t) {
        const int ra = (threadIdx.x >> 6) + 4 * t, cb = threadIdx.x & 63;
        const int ui = tu * kMfTU + ra, vi = tv * kMfTV + cb;
        if (ui >= H || vi >= W) continue;
        const i64 u = (i64)ui * W + vi;
        const int o = ra * WC + cb;
        const float x0 = xw[o], p0 = pw[o];
        const float g0 = t == 0 ? g4[0] : t == 1 ? g4[1] : t == 2 ? g4[2] : g4[3];
        glbw((float *)P.x[dst])[u] = x0;
        glbw(P.p[dst])[u] = p0;
        pp += (double)p0 * (double)p0;
        pr += -(double)p0 * (double)g0;
        auto xo = [&](int dy, int dx) { return xw[o + dy * WC + dx]; };
        auto po = [&](int dy, int dx) { return pw[o + dy * WC + dx]; };
        a += fast ? gen_prior_curv<true>(st, H, W, ui, vi, xo, po)
                  : gen_prior_curv<false>(st, H, W, ui, vi, xo, po);
    }
    out[0] = 0.0;
    out[1] = (double)a;
    out[2] = pp;
    out[3] = pr;
}

// matrix-free update of an LR item: the data part of the curvature along the new p (x, p
// the new iterate and direction).  Matrix-free: A p of the new direction by
// the forward, which forms p <- -g_t + beta p at the pixels it samples (the HR
// items write it elsewhere in the same launch), A x of the new iterate as
// A x + alpha A p of the old one; both kept for the next trial.
template <int S>
FI void gen_upd_lr_mf(const AS4 Item &itm, const AS4 Proj &P, const AS4 ScgState &st, const AS4 OpDev &op,
                      float *zs, double (&out)[4]) {
    const int h = op.H / op.s, w = op.W / op.s;
    const int src = st.upd_src, dst = src ^ 1;
    const AS1 float *p = glb(P.p[src]);
    const AS1 float *gt = glb(P.g[st.cur]);
    const float af = st.alpha_f, bf = st.beta_f;
    double dd = 0.0;
    int k, ti, tj, i, j;
    {
        for (int q = 0; q < kMfLRG && mf_lr_tile(op, itm.ty, q, k, ti, tj); ++q) {
            float ap[kMfCPT];
            mf_forward<S>(op, k, ti, tj, [&](i64 b, unsigned c) {
                return fmaf(bf, *at32(p + b, c), -*at32(gt + b, c));
            }, zs, i, j, ap);
#pragma unroll
            for (int c = 0; c < kMfCPT; ++c)
                if (i + c < h && j < w) {
                    const i64 row = ((i64)k * h + i + c) * w + j;
                    const float ax = fmaf(af, glb(P.ap[src])[row], glb(P.ax[src])[row]);
                    glbw(P.ax[dst])[row] = ax;
                    glbw(P.ap[dst])[row] = ap[c];
                    dd += gen_data_curv(st, P, row, ap[c], ax);
                }
        }
    }
    out[0] = dd;
    out[1] = out[2] = out[3] = 0.0;
}

// The update pass of matrix-free operators: HR and LR items in one launch
// (they write different vectors and read only the old ones).
template <int S>
__global__ void __launch_bounds__(kGenRows) k_mf_upd(const Proj *projs, const Item *items,
                                                     const int *n_items, double *partials) {
    __shared__ double red[kNV * (kGenRows / 64)];
    extern __shared__ float dyn[];   // an HR item's windows or an LR item's warped window
    const int it = blockIdx.x;
    if (it >= *cst(n_items)) return;
    const AS4 Item &itm = cst(items)[it];
    const AS4 Proj &P = cst(projs)[itm.proj];
    const AS4 ScgState &st = *cst(P.st);
    if (!st.do_update) return;
    const AS4 OpDev &op = *cst(P.op);
    double v[4];
    if (itm.tx == 1)
        gen_upd_hr(itm, P, st, op, dyn, v);
    else
        gen_upd_lr_mf<S>(itm, P, st, op, dyn, v);
    block_sum_store<4, kGenRows>(v, partials + (i64)it * kNV, red);
}

// The update pass of stored operators: HR items, then LR items (which read
// the new x and p).
__global__ void __launch_bounds__(kGenRows) k_gen_upd_hr(const Proj *projs, const Item *items,
                                                         const int *n_items, double *partials) {
    __shared__ double red[kNV * (kGenRows / 64)];
    const int it = blockIdx.x;
    if (it >= *cst(n_items)) return;
    const AS4 Item &itm = cst(items)[it];
    if (itm.tx != 1) return;
    const AS4 Proj &P = cst(projs)[itm.proj];
    const AS4 ScgState &st = *cst(P.st);
    if (!st.do_update) return;
    const AS4 OpDev &op = *cst(P.op);
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    const i64 u = (i64)itm.ty * kGenRows + threadIdx.x;
    if (u < (i64)op.H * op.W) {
        const int ui = (int)(u / op.W), vi = (int)(u - (i64)ui * op.W);
        v[1] = (double)gen_update(st, P, op.H, op.W, u, ui, vi, v[2], v[3]);
    }
    block_sum_store<4, kGenRows>(v, partials + (i64)it * kNV, red);
}

__global__ void __launch_bounds__(kGenRows) k_gen_upd_lr(const Proj *projs, const Item *items,
                                                         const int *n_items, double *partials) {
    __shared__ double red[kNV * (kGenRows / 64)];
    const int it = blockIdx.x;
    if (it >= *cst(n_items)) return;
    const AS4 Item &itm = cst(items)[it];
    if (itm.tx != 0) return;
    const AS4 Proj &P = cst(projs)[itm.proj];
    const AS4 ScgState &st = *cst(P.st);
    if (!st.do_update) return;
    const AS4 OpDev &op = *cst(P.op);
    const int h = op.H / op.s, w = op.W / op.s;
    const int dst = st.upd_src ^ 1;
    const AS1 float *xn = glb((const float *)P.x[dst]);
    const AS1 float *pn = glb(P.p[dst]);
    const bool l1 = st.wt.data_p != 2;
    double dd = 0.0;
    const i64 rows = (i64)op.K * h * w;
    const i64 r = (i64)itm.ty * kGenRows + threadIdx.x;
    if (r < rows) {
        const float ap = ell_row(glb(op.a_col), glb(op.a_val), op.a_w, rows, r,
                                 [&](i64 c) { return pn[c]; });
        const float ax = l1 ? ell_row(glb(op.a_col), glb(op.a_val), op.a_w, rows, r,
                                      [&](i64 c) { return xn[c]; })
                            : 0.f;
        dd = gen_data_curv(st, P, r, ap, ax);
    }
    double v[4] = {dd, 0.0, 0.0, 0.0};
    block_sum_store<4, kGenRows>(v, partials + (i64)it * kNV, red);
}

// standalone operators (FP32): y = A x over the LR rows, x = A^T r over the
// HR rows; matrix-free: one tile per workgroup
__global__ void __launch_bounds__(kGenRows) k_gen_forward(const OpDev *opp, const float *x,
                                                          float *y) {
    const AS4 OpDev &op = *cst(opp);
    const i64 rows = (i64)op.K * (op.H / op.s) * (op.W / op.s);
    for (i64 r = (i64)blockIdx.x * kGenRows + threadIdx.x; r < rows;
         r += (i64)gridDim.x * kGenRows)
        y[r] = ell_row(glb(op.a_col), glb(op.a_val), op.a_w, rows, r,
                       [&](int c) { return x[c]; });
}

__global__ void __launch_bounds__(kGenRows) k_gen_adjoint(const OpDev *opp, const float *r,
                                                          float *x) {
    const AS4 OpDev &op = *cst(opp);
    const i64 n = (i64)op.H * op.W;
    for (i64 u = (i64)blockIdx.x * kGenRows + threadIdx.x; u < n;
         u += (i64)gridDim.x * kGenRows)
        x[u] = ell_row(glb(op.t_col), glb(op.t_val), op.t_w, n, u,
                       [&](int c) { return r[c]; });
}

template <int S>
__global__ void __launch_bounds__(kGenRows) k_mf_forward(const OpDev *opp, const float *x,
                                                         float *y) {
    __shared__ float zs[mf_zwin(S)];
    const AS4 OpDev &op = *cst(opp);
    const int h = op.H / op.s, w = op.W / op.s;
    const AS1 float *xg = glb(x);
    int k, ti, tj, i, j;
    {
        for (int q = 0; q < kMfLRG && mf_lr_tile(op, blockIdx.x, q, k, ti, tj); ++q) {
            float ax[kMfCPT];
            mf_forward<S>(op, k, ti, tj, [&](i64 b, unsigned c) { return *at32(xg + b, c); }, zs, i, j,
                          ax);
#pragma unroll
            for (int c = 0; c < kMfCPT; ++c)
                if (i + c < h && j < w) y[((i64)k * h + i + c) * w + j] = ax[c];
        }
    }
}

template <int S>
__global__ void __launch_bounds__(kGenRows) k_mf_adjoint(const OpDev *opp, const float *r,
                                                         float *x) {
    __shared__ float lds[kMfWin + kMfQP * kMfQP];
    const AS4 OpDev &op = *cst(opp);
    const int H = op.H, W = op.W, h = H / op.s, w = W / op.s;
    const AS1 float *rg = glb(r);
    const int ntv = (W + kMfTV - 1) / kMfTV;
    const int tu = blockIdx.x / ntv, tv = blockIdx.x - tu * ntv;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    {
        mf_adjoint<S>(op, tu, tv, StoredRes{rg}, lds, acc);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int pr = tu * kMfTU + (threadIdx.x >> 6) + 4 * t;
        const int pc = tv * kMfTV + (threadIdx.x & 63);
        if (pr < H && pc < W && (threadIdx.x >> 6) + 4 * t < kMfTU) x[(i64)pr * W + pc] = acc[t];
    }
}

// Runs f with the scale as a compile-time constant.
template <class F>
void by_scale(int s, F f) {
    switch (s) {
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    default: f(std::integral_constant<int, 4>{}); break;
    }
}

// A pass over one class of general items.  Stored operators (ell): the trial
// and the cost+gradient run the LR rows then the HR rows, the update the HR
// rows then the LR rows.  Matrix-free ones: the cost+gradient likewise, the
// trial and the update in one launch each.
hipError_t launch_general(int grid, hipStream_t stream, const Proj *projs, const Item *items,
                          const int *n_items, double *partials, int kind, int S, bool ell) {
    if (grid <= 0) return hipSuccess;
    // the forward's warped window for the class's scale (any P)
    const size_t zb = (size_t)mf_zwin(S) * sizeof(float);
    const size_t ub = 2 * (kMfTU + 2) * (kMfTV + 2) * sizeof(float);
    const dim3 g(grid), b(kGenRows);
    by_scale(S, [&](auto sc) {
        constexpr int s = decltype(sc)::value;
        if (kind == 2 && ell) {
            hipLaunchKernelGGL(k_gen_upd_hr, g, b, 0, stream, projs, items, n_items, partials);
            hipLaunchKernelGGL(k_gen_upd_lr, g, b, 0, stream, projs, items, n_items, partials);
        } else if (kind == 2) {
            hipLaunchKernelGGL(k_mf_upd<s>, g, b, zb > ub ? zb : ub, stream, projs, items, n_items,
                               partials);
        } else {
            const int mode = kind == 1 ? 1 : 0;
            if (ell || mode == 0)
                hipLaunchKernelGGL(k_gen_trial_lr<s>, g, b, ell ? 0 : zb, stream, projs, items,
                                   n_items, partials, mode);
            hipLaunchKernelGGL(k_gen_trial_hr<s>, g, b, 0, stream, projs, items, n_items, partials,
                               mode);
        }
    });
    return hipGetLastError();
}

hipError_t launch_general_forward(hipStream_t stream, const OpDev *op, long long rows,
                                  const float *x, float *y, long long mf_tiles, int S) {
    if (mf_tiles > 0) {
        by_scale(S, [&](auto sc) {
            hipLaunchKernelGGL(k_mf_forward<decltype(sc)::value>, dim3((unsigned)mf_tiles),
                               dim3(kGenRows), 0, stream, op, x, y);
        });
        return hipGetLastError();
    }
    long long blocks = (rows + kGenRows - 1) / kGenRows;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_gen_forward, dim3((unsigned)blocks), dim3(kGenRows), 0, stream, op, x,
                       y);
    return hipGetLastError();
}

hipError_t launch_general_adjoint(hipStream_t stream, const OpDev *op, long long n,
                                  const float *r, float *x, long long mf_tiles, int S) {
    if (mf_tiles > 0) {
        by_scale(S, [&](auto sc) {
            hipLaunchKernelGGL(k_mf_adjoint<decltype(sc)::value>, dim3((unsigned)mf_tiles),
                               dim3(kGenRows), 0, stream, op, r, x);
        });
        return hipGetLastError();
    }
    long long blocks = (n + kGenRows - 1) / kGenRows;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_gen_adjoint, dim3((unsigned)blocks), dim3(kGenRows), 0, stream, op, r,
                       x);
    return hipGetLastError();
}

}  // namespace misr
