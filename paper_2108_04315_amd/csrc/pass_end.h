// pass_end.h -- the end of a pass: sums over a workgroup and over a solve's
// workgroups, and the device-resident SCG state machine (Moller's scalar
// steps in FP64) that the last workgroup of each pass runs.
#pragma once

#include "device_common.h"

namespace misr {

// ------------------------------------------------------ Moller's scalar steps
FI void scg_init(ScgScalars &s, const double *v) {
    s.E = v[0] + v[1];
    s.E0 = s.E;
    s.rr = v[2];
    s.pi = v[2];
    s.mu = v[2];
    s.alpha = 0.0;
    s.beta = 0.0;
    s.alpha_f = 0.f;
    s.beta_f = 0.f;
    s.lam_bar = 0.0;
    s.k = 1;
    s.it = 0;
    s.n_success = 0;
    s.stop = 0;
    if (!isfinite(s.E) || !isfinite(s.rr)) {
        s.active = 0;
        s.stop = 2;
        s.do_update = 0;
        return;
    }
    s.active = (s.n_iter > 0);
    s.success = 1;
    s.cur ^= 1;          // the gradient at x0 went to g[cur ^ 1]
    s.upd_src = s.xc;    // p[xc] is zero: the update pass sets p = -g0, x unchanged
    s.xc ^= 1;
    s.do_update = 1;
    s.sigk = (s.pi > 0.0) ? s.sigma / sqrt(s.pi) : 0.0;
    s.sigk_f = (float)s.sigk;
}

// steps 1-5 of the pass
FI void scg_phase_a(ScgScalars &s, const double *v) {
    s.do_update = 0;
    if (!s.active) return;
    if (s.success) {
        s.delta = v[0] + v[1];
        s.pi = v[2];
        s.mu = v[3];
    }
    if (s.rr == 0.0) {
        s.active = 0;
        s.stop = 1;
        return;
    }
    if (!isfinite(s.delta)) {
        s.active = 0;
        s.stop = 2;
        return;
    }
    double d = s.delta + (s.lam - s.lam_bar) * s.pi;
    if (d <= 0.0) {
        s.lam_bar = 2.0 * (s.lam - d / s.pi);
        d = -d + s.lam * s.pi;
        s.lam = s.lam_bar;
    }
    s.delta = d;
    s.alpha = s.mu / d;
    if (!isfinite(s.alpha)) {
        s.active = 0;
        s.stop = 2;
        return;
    }
    s.alpha_f = (float)s.alpha;
    s.rseed = mix32(0x51ed270bu + (unsigned)s.it);
}

// steps 6-9 of the pass
FI void scg_phase_b(ScgScalars &s, const double *v, IterRec *trace) {
    s.do_update = 0;
    if (!s.active) return;
    const double rr0 = s.rr;   // |r|^2 at the pass's start (mu = p . r used this r)
    const double Et = v[0] + v[1];
    s.E_t = Et;
    if (!isfinite(Et)) {
        s.active = 0;
        s.stop = 2;
        s.Delta = 0.0;
    } else {
        const double Delta = 2.0 * s.delta * (s.E - Et) / (s.mu * s.mu);
        s.Delta = Delta;
        if (Delta >= 0.0) {
            const double gg = v[2], ggk = v[3], gp = v[4];
            s.E = Et;
            s.lam_bar = 0.0;
            s.success = 1;
            s.n_success++;
            s.beta = (s.k % s.N == 0) ? 0.0 : (gg - ggk) / s.mu;
            s.rr = gg;
            s.cur ^= 1;
            s.upd_src = s.xc;
            s.xc ^= 1;
            s.do_update = 1;
            s.beta_f = (float)s.beta;
            const double pn = gg - 2.0 * s.beta * gp + s.beta * s.beta * s.pi;
            s.sigk = (pn > 0.0) ? s.sigma / sqrt(pn) : 0.0;
            s.sigk_f = (float)s.sigk;
            if (Delta >= 0.75) s.lam *= 0.25;
        } else {
            s.lam_bar = s.lam;
            s.success = 0;
        }
        if (Delta < 0.25) s.lam += s.delta * (1.0 - Delta) / s.pi;
    }
    if (trace) {
        IterRec &r = trace[s.it];
        r.E = s.E;
        r.E_t = s.E_t;
        r.delta = s.delta;
        r.mu = s.mu;
        r.alpha = s.alpha;
        r.Delta = s.Delta;
        r.lam = s.lam;
        r.pi = s.pi;
        r.rr = rr0;
        r.success = (s.do_update != 0);
        r.pad_ = 0;
    }
    s.k++;
    s.it++;
    if (s.it >= s.n_iter) s.active = 0;
}

// ------------------------------------------------------------- pass end
// Threads that sum a solve's rows of partial sums (four rows each in flight
// per round; 1024 threads measured slower).
constexpr int kEndRows = kNT;

// Sums rows 0..n-1 of N partial sums (of kNV) over the workgroup's first
// kEndRows threads in a fixed order, wave by wave into red[wave N + i]; row
// loads as ld(address).  Four rows per thread and step, all their loads issued
// before the additions; past the end a row is loaded from a valid address and
// counted as zero, so each thread adds its rows in the same order whatever the
// count, and in one memory round trip per 4 x kEndRows rows.
template <int N, class Ld>
FI void sum_rows(const AS1 double *pt, int n, double *red, Ld ld) {
    constexpr int kSU = 4;   // (eight measured slower)
    double t[N];
#pragma unroll
    for (int q = 0; q < N; ++q) t[q] = 0.0;
    for (int i = threadIdx.x; i < n; i += kSU * kEndRows) {
        double l[kSU][N];
#pragma unroll
        for (int a = 0; a < kSU; ++a) {
            const int j = (i + a * kEndRows < n) ? i + a * kEndRows : i;
#pragma unroll
            for (int q = 0; q < N; ++q) l[a][q] = ld(pt + (i64)j * kNV + q);
        }
#pragma unroll
        for (int a = 0; a < kSU; ++a)
#pragma unroll
            for (int q = 0; q < N; ++q) t[q] += (i + a * kEndRows < n) ? l[a][q] : 0.0;
    }
    wave_sums<N>(t, red + (threadIdx.x >> 6) * N);
}

// The SCG steps after a pass, by one thread, from sum_rows' sums: pass 0 cost
// and gradient at the start point, 1 trial, 2 update.  fold: the steps that
// wait for nothing but a rejected trial follow it at once (a rejection leaves
// nothing to update).  The scalars go by 8-byte words: in with one memory
// round trip, out with one.
template <int N>
FI void scg_steps(const AS4 SolveRef *rp, const double *red, int pass, bool fold) {
    double t[kNV] = {0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < N; ++q)
#pragma unroll
        for (int w = 0; w < kEndRows / 64; ++w) t[q] += red[w * N + q];
    constexpr int NW = sizeof(ScgScalars) / 8;
    static_assert(sizeof(ScgScalars) % 8 == 0, "state copied by 8-byte words");
    unsigned long long w[NW];
    const AS4 unsigned long long *gr = cst((const unsigned long long *)rp->st);
#pragma unroll
    for (int i = 0; i < NW; ++i) w[i] = gr[i];
    ScgScalars s;
    __builtin_memcpy(&s, w, sizeof s);
    if (pass == 0) {
        scg_init(s, t);
    } else if (pass == 1) {
        scg_phase_b(s, t, rp->trace);
        if (fold && !s.do_update) scg_phase_a(s, t);
    } else {
        scg_phase_a(s, t);
    }
    __builtin_memcpy(w, &s, sizeof s);
    AS1 unsigned long long *gw = glbw((unsigned long long *)rp->st);
#pragma unroll
    for (int i = 0; i < NW; ++i) gw[i] = w[i];
}

// Ends a workgroup of a banded operator's pass: sums N per-thread values over
// its NT threads in a fixed order, stores them to out[0..N) (a row of the
// partial sums) and, in a solve (P.ref), counts the workgroup as arrived; the
// last of the solve's workgroups sums the rows and runs the SCG steps that
// follow the pass.  red: LDS scratch of kNV * NT/64 doubles.
//
// As launches of their own (k_scalar, which general operators keep) the steps
// took 4.7 us after each of a pass's two launches, mostly the launch and two
// round trips to memory.  Here they cost every workgroup a store and an
// addition in memory, about 2 us at its end, and the last one the sums:
// 100-pass solves of 1024^2 LR (s = 2) 11.31 -> 10.98 ms, of 3072^2 LR even;
// 50 passes of 64^2 LR 1.73 -> 1.54 ms.  A general operator's pass is made of many
// short workgroups, which the 2 us cost more than the launch saves (1024^2
// HR: 9.44 -> 9.86 ms), and an evaluation of cost and gradient alone gains
// nothing (27.3 -> 28.1 us).
//
// Order between workgroups (8 XCDs, each with its own L2): a row goes out by
// agent-scope stores, which write through to memory, and the addition to the
// count follows only when those have completed; the last workgroup reads the
// rows by agent-scope loads.  The state is read through this XCD's caches
// (an earlier launch wrote it) and written for the next launch.  Every
// workgroup that reads the state counts itself afterwards, so nobody reads it
// while it changes.
template <int N, int NT>
FI void pass_end(double (&v)[N], double *out, double *red, const AS4 Proj &P, int pass) {
    static_assert(N < kNV && NT >= kEndRows && NT % 64 == 0, "");
    int *last = reinterpret_cast<int *>(red + kNV * (NT / 64) - 1);
    const int wid = threadIdx.x >> 6;
    wave_sums<N>(v, red + wid * N);
    __syncthreads();
    const AS4 SolveRef *rp = cst(P.ref);
    if (wid == 0) {
        if (threadIdx.x < N) {
            double s = 0.0;
#pragma unroll
            for (int w = 0; w < NT / 64; ++w) s += red[w * N + threadIdx.x];
            __hip_atomic_store(glbw(out) + threadIdx.x, s, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        }
        if (rp) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (threadIdx.x == 0) {
                AS1 unsigned *c = glbw(&rp->st->arrived);
                const unsigned n = pass == 2 ? rp->nitemsu : rp->nitems;
                const bool l = __hip_atomic_fetch_add(c, 1u, __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT) == n - 1u;
                if (l) __hip_atomic_store(c, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                *last = l;
            }
        }
    }
    if (!rp) return;
    __syncthreads();
    if (!*last) return;   // uniform
    asm volatile("" ::: "memory");
    if (threadIdx.x < kEndRows)
        sum_rows<N>(glb((const double *)(pass == 2 ? rp->part_u : rp->part)),
                    pass == 2 ? rp->nitemsu : rp->nitems, red, [](const AS1 double *a) {
                        return __hip_atomic_load(a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    });
    __syncthreads();
    if (threadIdx.x == 0) scg_steps<N>(rp, red, pass, true);
}

}  // namespace misr
