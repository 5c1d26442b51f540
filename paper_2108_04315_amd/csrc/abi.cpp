// abi.cpp -- the C ABI of libmisr.so: validation, operator construction,
// workspace management and the device-resident SCG solve driver.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <new>
#include <thread>

#include "runtime.h"

using namespace misr;

namespace misr {

static thread_local std::string g_err;

misr_status set_error(misr_status st, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return st;
}

misr_status hip_fail(hipError_t e, const char *what) {
    return set_error(e == hipErrorOutOfMemory ? MISR_E_NOMEM : MISR_E_HIP, "%s: %s", what,
                     hipGetErrorString(e));
}

size_t dtype_size(misr_dtype dt) { return dt == MISR_F32 ? 4 : 2; }

bool capturing(hipStream_t stream) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &cap) != hipSuccess) (void)hipGetLastError();
    return cap != hipStreamCaptureStatusNone;
}

hipError_t PlanDev::upload(Plan &pl, int n_iter, hipStream_t stream) {
    hipError_t e;
    const size_t np = pl.projs.size(), ni = pl.items.size(), nu = pl.items_u.size(),
                 ns = pl.states.size(), nh = pl.halos.size();
    if ((e = projs.ensure(np * sizeof(Proj))) != hipSuccess) return e;
    if ((e = items.ensure(ni * sizeof(Item))) != hipSuccess) return e;
    if ((e = items_u.ensure(nu * sizeof(Item))) != hipSuccess) return e;
    if ((e = counts.ensure(pl.counts.size() * sizeof(int))) != hipSuccess) return e;
    if ((e = states.ensure(ns * sizeof(ScgState))) != hipSuccess) return e;
    if ((e = partials.ensure(ni * kNV * sizeof(double))) != hipSuccess) return e;
    if ((e = partials_u.ensure(nu * kNV * sizeof(double))) != hipSuccess) return e;
    if ((e = refs.ensure(ns * sizeof(SolveRef))) != hipSuccess) return e;
    if ((e = halos.ensure(nh * sizeof(HaloCopy))) != hipSuccess) return e;
    // per-pass records of each solve (only solves write them)
    const size_t per = (size_t)(n_iter > 0 ? n_iter : 0);
    if (per > 0 && (e = traces.ensure(ns * per * sizeof(IterRec))) != hipSuccess) return e;
    n_iter_max = (int)per;
    ScgState *sd = states.as<ScgState>();
    for (size_t j = 0; j < np; ++j) {
        pl.projs[j].st = sd + pl.proj_solve[j];
        const int i = pl.proj_solve[j];
        pl.projs[j].ref = pl.steps && !pl.apart[i] ? refs.as<SolveRef>() + i : nullptr;
    }
    pl.refs.resize(ns);
    for (size_t i = 0; i < ns; ++i)
        pl.refs[i] = SolveRef{sd + i, per ? traces.as<IterRec>() + i * per : nullptr,
                              partials.as<double>() + (size_t)pl.item0[i] * kNV,
                              partials_u.as<double>() + (size_t)pl.item0u[i] * kNV,
                              pl.nitems[i], pl.nitemsu[i], pl.apart[i], 0};
    // A call uploads the arrays whose bytes differ from what the device holds.
    // A repeated call on an operator differs in the views (its buffers) and,
    // after a solve, in the states: short arrays, which go with one launch
    // (launch_put).  Seven copies from pageable memory cost a call about 20 us
    // of host time.  (An operator's first call allocates the arrays and uploads
    // all of them.)
    struct Up {
        DevMem &d;
        const void *h;
        size_t n;
    } ups[] = {{projs, pl.projs.data(), np * sizeof(Proj)},
               {items, pl.items.data(), ni * sizeof(Item)},
               {items_u, pl.items_u.data(), nu * sizeof(Item)},
               {counts, pl.counts.data(), pl.counts.size() * sizeof(int)},
               {refs, pl.refs.data(), ns * sizeof(SolveRef)},
               {halos, pl.halos.data(), nh * sizeof(HaloCopy)},
               {states, pl.states.data(), ns * sizeof(ScgState)}};
    // A call captured into the caller's graph writes these arrays whenever that
    // graph is replayed: from then on nothing is known about what they hold.
    // The graph goes on using these blocks, and its copies read their source
    // when they run: both stay as they are now (Kept).
    const bool cap = kept && capturing(stream);
    captured |= cap;
    if (cap)
        for (DevMem *m : {&projs, &items, &items_u, &counts, &states, &partials, &partials_u,
                          &traces, &refs, &halos})
            m->keep(*kept);
    constexpr int kStates = 6;
    if (states_dirty) held[kStates].p = nullptr;
    if (captured)
        for (auto &hd : held) hd.p = nullptr;
    PutArgs put;
    put.n = 0;
    size_t at = 0;   // bytes in put
    for (int i = 0; i < 7; ++i) {
        Up &u = ups[i];
        Held &hd = held[i];
        if (!u.n || (hd.p == u.d.p && hd.b.size() == u.n && !std::memcmp(hd.b.data(), u.h, u.n)))
            continue;
        hd.p = nullptr;   // (not held while the upload may fail)
        if (at + u.n <= kPutBytes && u.n % 4 == 0) {
            put.dst[put.n] = u.d.as<unsigned>();
            put.words[put.n++] = (int)(u.n / 4);
            std::memcpy((unsigned char *)put.w + at, u.h, u.n);
            at += u.n;
        } else {
            const void *src = cap ? kept->copy(u.h, u.n) : u.h;
            e = hipMemcpyAsync(u.d.p, src, u.n, hipMemcpyHostToDevice, stream);
            if (e != hipSuccess) return e;
        }
        hd.b.assign((const unsigned char *)u.h, (const unsigned char *)u.h + u.n);
    }
    if (put.n && (e = launch_put(stream, put)) != hipSuccess) return e;
    for (int i = 0; i < 7; ++i)
        if (ups[i].n) held[i].p = ups[i].d.p;
    states_dirty = false;
    return hipSuccess;
}

}  // namespace misr

// ------------------------------------------------------------------- checks
static bool finite_pos(double v) { return std::isfinite(v) && v > 0; }

extern "C" const char *misr_last_error(void) { return g_err.c_str(); }

extern "C" void misr_params_default(misr_params *p) {
    if (!p) return;
    std::memset(p, 0, sizeof *p);
    p->lambda_reg = 0.01;
    p->alpha_btv = 0.4;
    p->eps = 1e-3;
    p->btv_w = 3;
    p->data_p = 2;
    p->eps_data = 1e-3;
    p->scg_sigma = 1e-4;
    p->scg_lambda1 = 1e-6;
    p->n_iter = 50;
    p->img_dtype = MISR_F32;
    p->tile_lr = 0;
    p->halo_lr = 8;
}

int misr::band_length(const misr_geometry *g) {
    bool frac = false;
    for (int k = 0; k < g->n_frames; ++k)
        for (int a = 0; a < 2; ++a) {
            const double t = g->scale * g->shifts_lr[2 * k + a];
            if (t != std::floor(t)) frac = true;
        }
    return g->scale + g->psf_size - (frac ? 0 : 1);
}

extern "C" misr_status misr_geometry_check(const misr_geometry *g) {
    if (!g) return set_error(MISR_E_INVAL, "geometry is NULL");
    if (g->scale < 1 || g->scale > 4)
        return set_error(MISR_E_INVAL, "scale %d outside [1, 4]", g->scale);
    if (g->hr_h < 1 || g->hr_w < 1 || g->hr_h % g->scale || g->hr_w % g->scale)
        return set_error(MISR_E_INVAL, "HR size %dx%d must be positive and divisible by s=%d",
                         g->hr_h, g->hr_w, g->scale);
    if ((long long)g->hr_h * g->hr_w >= (1LL << 31))
        return set_error(MISR_E_INVAL, "HR image too large (>= 2^31 pixels)");
    if (g->n_frames < 1 || g->n_frames > kMaxK)
        return set_error(MISR_E_INVAL, "n_frames %d outside [1, %d]", g->n_frames, kMaxK);
    if (!g->shifts_lr && !g->warps) return set_error(MISR_E_INVAL, "shifts_lr is NULL");
    if (g->shifts_lr)
        for (int i = 0; i < 2 * g->n_frames; ++i)
            if (!std::isfinite(g->shifts_lr[i]) || std::fabs(g->shifts_lr[i]) > 1.0)
                return set_error(MISR_E_INVAL, "shift %d (%g) not finite or |shift| > 1 LR px",
                                 i, g->shifts_lr[i]);
    if (g->psf_size < 1 || g->psf_size > 15 || g->psf_size % 2 == 0)
        return set_error(MISR_E_INVAL, "psf_size %d must be odd in [1, 15]", g->psf_size);
    if (!g->psf_1d && !g->psf_2d) return set_error(MISR_E_INVAL, "psf_1d is NULL");
    if (g->psf_1d)
        for (int i = 0; i < g->psf_size; ++i)
            if (!std::isfinite(g->psf_1d[i]))
                return set_error(MISR_E_INVAL, "psf tap %d not finite", i);
    if (g->psf_frames)
        for (int i = 0; i < 2 * g->n_frames * g->psf_size; ++i)
            if (!std::isfinite(g->psf_frames[i]))
                return set_error(MISR_E_INVAL, "psf_frames tap %d not finite", i);
    if (g->psf_2d)
        for (int i = 0; i < g->n_frames * g->psf_size * g->psf_size; ++i)
            if (!std::isfinite(g->psf_2d[i]))
                return set_error(MISR_E_INVAL, "psf_2d entry %d not finite", i);
    if (g->warps) {
        for (int i = 0; i < 6 * g->n_frames; ++i)
            if (!std::isfinite(g->warps[i]) || std::fabs(g->warps[i]) > 1e6)
                return set_error(MISR_E_INVAL, "warp coefficient %d not finite or > 1e6", i);
    }
    if (g->warps || g->psf_2d) return MISR_OK;   // general operator: no band constraints
    const int L = band_length(g);
    const int Lp = padded_band(g->scale, L);
    if (Lp < 0)
        return set_error(MISR_E_INVAL, "band length %d unsupported at scale %d", L, g->scale);
    // the update/curvature window needs every frame's band start within
    // [-EXT, s-1] relative to the tile (EXT = max(Lp-1, 2))
    const int EXT = Lp - 1 > 2 ? Lp - 1 : 2;
    const int R = (g->psf_size - 1) / 2;
    for (int k = 0; k < g->n_frames; ++k)
        for (int a = 0; a < 2; ++a) {
            const int off = (int)std::floor(g->scale * g->shifts_lr[2 * k + 1 - a]) - R;
            if (off < -EXT || off > g->scale - 1)
                return set_error(MISR_E_INVAL, "frame %d shift moves the band outside the "
                                 "supported window", k);
        }
    return MISR_OK;
}

extern "C" misr_status misr_params_check(const misr_params *p) {
    if (!p) return set_error(MISR_E_INVAL, "params is NULL");
    if (!std::isfinite(p->lambda_reg) || p->lambda_reg < 0)
        return set_error(MISR_E_INVAL, "lambda_reg must be finite and >= 0");
    if (!(p->alpha_btv > 0 && p->alpha_btv < 1))
        return set_error(MISR_E_INVAL, "alpha_btv must lie in (0, 1)");
    if (!std::isfinite(p->eps) || p->eps < 0) return set_error(MISR_E_INVAL, "eps must be >= 0");
    if (p->btv_w < 1 || p->btv_w > 3) return set_error(MISR_E_INVAL, "btv_w must be in [1, 3]");
    if (p->data_p != 1 && p->data_p != 2) return set_error(MISR_E_INVAL, "data_p must be 1 or 2");
    if (!std::isfinite(p->eps_data) || p->eps_data < 0)
        return set_error(MISR_E_INVAL, "eps_data must be >= 0");
    if (!finite_pos(p->scg_sigma)) return set_error(MISR_E_INVAL, "scg_sigma must be > 0");
    if (!finite_pos(p->scg_lambda1)) return set_error(MISR_E_INVAL, "scg_lambda1 must be > 0");
    if (p->n_iter < 0) return set_error(MISR_E_INVAL, "n_iter must be >= 0");
    if (p->img_dtype != MISR_F32 && p->img_dtype != MISR_F16 && p->img_dtype != MISR_BF16)
        return set_error(MISR_E_INVAL, "img_dtype invalid");
    if (p->tile_lr < 0 || p->halo_lr < 0)
        return set_error(MISR_E_INVAL, "tile_lr and halo_lr must be >= 0");
    if (p->x_rounding != 0 && p->x_rounding != 1)
        return set_error(MISR_E_INVAL, "x_rounding must be 0 or 1");
    if (p->x_work != 0 && p->x_work != 1) return set_error(MISR_E_INVAL, "x_work must be 0 or 1");
    if (p->x_init < 0 || p->x_init > 2) return set_error(MISR_E_INVAL, "x_init must be 0, 1 or 2");
    if (p->y_u16 != 0 && p->y_u16 != 1) return set_error(MISR_E_INVAL, "y_u16 must be 0 or 1");
    if (p->y_u16 && !(std::isfinite(p->y_scale) && p->y_scale > 0))
        return set_error(MISR_E_INVAL, "y_scale must be finite and > 0 with y_u16");
    if (p->y_u16 && p->img_dtype != MISR_F32)
        return set_error(MISR_E_INVAL, "uint16 frames go with an FP32 image (img_dtype F32)");
    if (p->y_u16 && p->x_init != 0)
        return set_error(MISR_E_INVAL, "x_init reads frames stored in img_dtype (y_u16 = 0)");
    return MISR_OK;
}

// -------------------------------------------------------------------- ctx
extern "C" misr_status misr_ctx_create(int dev, misr_ctx **out) {
    if (!out) return set_error(MISR_E_INVAL, "out is NULL");
    *out = nullptr;
    int n = 0;
    hipError_t e = hipGetDeviceCount(&n);
    if (e != hipSuccess || n == 0) return set_error(MISR_E_HIP, "no HIP device available");
    if (dev < 0 || dev >= n) return set_error(MISR_E_INVAL, "device %d outside [0, %d)", dev, n);
    MISR_HIP(hipSetDevice(dev));
    hipDeviceProp_t prop;
    MISR_HIP(hipGetDeviceProperties(&prop, dev));
    auto *c = new misr_ctx();
    c->dev = dev;
    c->ncu = prop.multiProcessorCount;
    if (hipStreamCreateWithFlags(&c->stream, hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&c->ev_in, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&c->ev_out, hipEventDisableTiming) != hipSuccess) {
        delete c;
        return set_error(MISR_E_HIP, "stream/event creation failed");
    }
    // the workspace of misr_cost_grad_noalloc on this device
    if ((e = scratch_init(dev)) != hipSuccess) {
        (void)hipEventDestroy(c->ev_in);
        (void)hipEventDestroy(c->ev_out);
        (void)hipStreamDestroy(c->stream);
        delete c;
        return hip_fail(e, "hipGetSymbolAddress (no-allocation workspace)");
    }
    *out = c;
    return MISR_OK;
}

// Gives back what batches on the context keep (with BatchCache below).
static void drop_batch(const misr_ctx *c);

extern "C" misr_status misr_ctx_destroy(misr_ctx *c) {
    if (!c) return set_error(MISR_E_INVAL, "ctx is NULL");
    if (c->users.load() > 0)
        return set_error(MISR_E_BUSY, "%d ops/servers still use this context", c->users.load());
    (void)hipStreamSynchronize(c->stream);
    drop_batch(c);
    (void)hipEventDestroy(c->ev_in);
    (void)hipEventDestroy(c->ev_out);
    (void)hipStreamDestroy(c->stream);
    delete c;
    return MISR_OK;
}

static hipError_t set_device(int dev) {
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    return cur == dev ? hipSuccess : hipSetDevice(dev);
}

// --------------------------------------------------------------------- op
// One axis of A_k = C_y (x) C_x: LR index i reads HR samples
// s*i + off + l, l in [0, Lp).  Built from the three 1-D factors in FP64:
// bilinear translation by t HR px (zero outside [0, N)), "same" convolution
// with the taps (zero padding), mean over s samples.
static void band_weights(int N, int s, double t, int P, const double *psf, int Lp, int off,
                         float *out) {
    const int R = (P - 1) / 2;
    const double fl = std::floor(t), f = t - fl;
    const int ifl = (int)fl;
    std::vector<double> acc((size_t)Lp);
    for (int i = 0; i < N / s; ++i) {
        std::fill(acc.begin(), acc.end(), 0.0);
        for (int b = 0; b < s; ++b) {
            const int u = s * i + b;                // output of the blur, inside [0, N)
            for (int a = -R; a <= R; ++a) {
                const int z = u - a;                // blur input = warp output index
                if (z < 0 || z >= N) continue;      // warp output exists on [0, N) only
                for (int e = 0; e < 2; ++e) {
                    const double wgt = e ? f : 1.0 - f;
                    const int v = z + ifl + e;      // HR sample read by the warp
                    if (wgt == 0.0 || v < 0 || v >= N) continue;
                    acc[v - (s * i + off)] += psf[a + R] * wgt / s;
                }
            }
        }
        for (int l = 0; l < Lp; ++l) out[(size_t)i * Lp + l] = (float)acc[l];
    }
}

// Weights of an LR row that the image edge does not cut (the same sums as
// band_weights, in its order), and the run [lo, hi) of rows, around the
// middle one, that equal them at every tap inside the image.
static void canonical_row(int N, int s, double t, int P, const double *psf, int Lp, int off,
                          const float *rows, float *cw, int *lo, int *hi) {
    const int R = (P - 1) / 2, n = N / s;
    const double fl = std::floor(t), f = t - fl;
    std::vector<double> acc((size_t)Lp, 0.0);
    for (int b = 0; b < s; ++b)
        for (int a = -R; a <= R; ++a)
            for (int e = 0; e < 2; ++e) {
                const double wgt = e ? f : 1.0 - f;
                if (wgt != 0.0) acc[b - a + (int)fl + e - off] += psf[a + R] * wgt / s;
            }
    for (int l = 0; l < kMaxL; ++l) cw[l] = l < Lp ? (float)acc[l] : 0.f;
    auto same = [&](int i) {
        for (int l = 0; l < Lp; ++l) {
            const int v = s * i + off + l;
            if (v >= 0 && v < N && !(rows[(size_t)i * Lp + l] == cw[l])) return false;
        }
        return true;
    };
    *lo = *hi = n / 2;
    while (*hi < n && same(*hi)) ++*hi;
    while (*lo > 0 && *hi > n / 2 && same(*lo - 1)) --*lo;
    if (*hi == *lo) *lo = *hi = 0;   // none: every row takes the table's
}

// ---------------------------------------------------- general operators
// Row (k, i, j) of A = [A_0; ...; A_{K-1}] for an affine warp and a P x P PSF:
// D averages the s x s block of HR samples (U, V) = (s i + a, s j + b); B
// takes h[pa + R][pb + R] times the warped image at (U - pa, V - pb), zero
// off the grid; M samples x bilinearly at the affine position of that pixel,
// zero off the grid.  Contributions to one HR pixel are merged (FP64).
static void general_row(const misr_op *op, const double *m, const double *hk, int P, int i,
                        int j, std::vector<std::pair<int, double>> &ent) {
    const int H = op->H, W = op->W, s = op->s, R = (P - 1) / 2;
    const double inv = 1.0 / ((double)s * s);
    ent.clear();
    for (int a = 0; a < s; ++a)
        for (int b = 0; b < s; ++b)
            for (int pa = -R; pa <= R; ++pa)
                for (int pb = -R; pb <= R; ++pb) {
                    const int u = s * i + a - pa, v = s * j + b - pb;
                    if (u < 0 || u >= H || v < 0 || v >= W) continue;
                    const double hw = hk[(pa + R) * P + (pb + R)] * inv;
                    if (hw == 0.0) continue;
                    const double r = m[0] * u + m[1] * v + m[2], c = m[3] * u + m[4] * v + m[5];
                    const double r0 = std::floor(r), c0 = std::floor(c);
                    const double fa = r - r0, fb = c - c0;
                    const double wq[4] = {(1 - fa) * (1 - fb), (1 - fa) * fb, fa * (1 - fb),
                                          fa * fb};
                    const double rq[4] = {r0, r0, r0 + 1, r0 + 1}, cq[4] = {c0, c0 + 1, c0, c0 + 1};
                    for (int q = 0; q < 4; ++q) {
                        if (wq[q] == 0.0 || rq[q] < 0 || rq[q] >= H || cq[q] < 0 || cq[q] >= W)
                            continue;
                        ent.emplace_back((int)rq[q] * W + (int)cq[q], hw * wq[q]);
                    }
                }
    std::sort(ent.begin(), ent.end(),
              [](const std::pair<int, double> &x, const std::pair<int, double> &y) {
                  return x.first < y.first;
              });
    size_t o = 0;
    for (size_t e = 0; e < ent.size(); ++e) {
        if (o > 0 && ent[o - 1].first == ent[e].first)
            ent[o - 1].second += ent[e].second;
        else
            ent[o++] = ent[e];
    }
    ent.resize(o);
}

// Frame k's warp of a general geometry (its shift as a translation when no
// warps are given) and its P x P PSF.
static void general_warp(const misr_geometry *g, int k, double m[6]) {
    if (g->warps) {
        std::copy(g->warps + 6 * k, g->warps + 6 * k + 6, m);
        return;
    }
    const double s = g->scale;
    const double ty = g->shifts_lr ? s * g->shifts_lr[2 * k + 1] : 0.0;
    const double tx = g->shifts_lr ? s * g->shifts_lr[2 * k] : 0.0;
    const double mm[6] = {1.0, 0.0, ty, 0.0, 1.0, tx};
    std::copy(mm, mm + 6, m);
}

static void general_psf(const misr_geometry *g, int k, double *hk) {
    const int P = g->psf_size;
    if (g->psf_2d) {
        std::copy(g->psf_2d + (size_t)k * P * P, g->psf_2d + (size_t)(k + 1) * P * P, hk);
        return;
    }
    const double *vy = g->psf_frames ? g->psf_frames + (size_t)k * 2 * P : g->psf_1d;
    const double *vx = g->psf_frames ? vy + P : g->psf_1d;
    for (int a = 0; a < P; ++a)
        for (int b = 0; b < P; ++b) hk[a * P + b] = vy[a] * vx[b];
}

long long misr::mf_lr_tiles(int H, int W, int s, int K) {
    const long long h = H / s, w = W / s;
    const long long nt = ((h + mf_ti(s) - 1) / mf_ti(s)) * ((w + kMfTJ - 1) / kMfTJ);
    return (long long)K * ((nt + kMfLRG - 1) / kMfLRG);
}

long long misr::mf_hr_tiles(int H, int W) {
    return (long long)((H + kMfTU - 1) / kMfTU) * ((W + kMfTV - 1) / kMfTV);
}

// Matrix-free form of a general operator (Eq. sisr, A_k = D B_k M_k from its
// factors).  Per frame: the inverse warp; the half extents eu, ev of the
// preimage of a pixel's bilinear support (|r - pr| < 1, |c - pc| < 1 maps to
// |u - u(pr, pc)| < |gi0| + |gi1|); the candidates per axis (floor(2 eu) + 1
// from floor(u - eu) + 1); the caps on an adjoint tile's back-projection
// window (every candidate of the tile's pixels: floor of the preimage's
// extent plus 2, one position of slack) and its residual window, which with
// the padded kernel must fit the kernel's LDS.  The blur-and-bin kernel: LR pixel
// (i, j) averages the s x s block (s i + a, s j + b) of the PSF-blurred
// warped image, and the blur takes h[pa + R][pb + R] times the warped image
// at (U - pa, V - pb), so the warped image at (s i + al - R, s j + be - R)
// weighs C[al][be] = sum over a, b < s of h[a + 2R - al][b + 2R - be] / s^2
// (terms outside the PSF dropped).
bool misr::general_mf_plan(const misr_geometry *g, OpDev *hd, std::vector<float> *ker) {
    if (g->general_ell) return false;
    const int s = g->scale, K = g->n_frames, P = g->psf_size, Q = s + P - 1, R = (P - 1) / 2;
    if (Q > kMfQmax || K > kMaxK) return false;
    OpDev tmp;
    OpDev &d = hd ? *hd : tmp;
    for (int k = 0; k < K; ++k) {
        double m[6];
        general_warp(g, k, m);
        const double det = m[0] * m[4] - m[1] * m[3];
        if (!(std::fabs(det) > 1e-9)) return false;
        const double gi[6] = {m[4] / det, -m[1] / det, 0.0, -m[3] / det, m[0] / det, 0.0};
        const double eu = std::fabs(gi[0]) + std::fabs(gi[1]);
        const double ev = std::fabs(gi[3]) + std::fabs(gi[4]);
        if (!(eu <= 64.0 && ev <= 64.0)) return false;
        const double lu = (kMfTU - 1) * std::fabs(gi[0]) + (kMfTV - 1) * std::fabs(gi[1]) + 2 * eu;
        const double lv = (kMfTU - 1) * std::fabs(gi[3]) + (kMfTV - 1) * std::fabs(gi[4]) + 2 * ev;
        const long long ru = (long long)std::floor(lu) + 3, rv = (long long)std::floor(lv) + 3;
        const long long nt = (Q + s - 1) / s;
        const long long ni = (ru + s - 1) / s + nt, nj = (rv + s - 1) / s + nt;
        if (ru * rv + ni * nj > kMfWin || s * nt > kMfQP) return false;
        std::copy(m, m + 6, d.gm[k]);
        d.gi[k][0] = gi[0];
        d.gi[k][1] = gi[1];
        d.gi[k][2] = -(gi[0] * m[2] + gi[1] * m[5]);
        d.gi[k][3] = gi[3];
        d.gi[k][4] = gi[4];
        d.gi[k][5] = -(gi[3] * m[2] + gi[4] * m[5]);
        d.eu[k] = eu;
        d.ev[k] = ev;
        d.ncu[k] = (int)std::floor(2 * eu) + 1;
        d.ncv[k] = (int)std::floor(2 * ev) + 1;
        d.ru[k] = (int)ru;
        d.rv[k] = (int)rv;
    }
    d.mf = 1;
    d.P = P;
    d.Q = Q;
    if (ker) {
        ker->assign((size_t)K * Q * Q, 0.f);
        std::vector<double> hk((size_t)P * P);
        for (int k = 0; k < K; ++k) {
            general_psf(g, k, hk.data());
            for (int al = 0; al < Q; ++al)
                for (int be = 0; be < Q; ++be) {
                    double c = 0.0;
                    for (int a = 0; a < s; ++a)
                        for (int b = 0; b < s; ++b) {
                            const int ia = a + 2 * R - al, ib = b + 2 * R - be;
                            if (ia >= 0 && ia < P && ib >= 0 && ib < P) c += hk[ia * P + ib];
                        }
                    (*ker)[((size_t)k * Q + al) * Q + be] = (float)(c / ((double)s * s));
                }
        }
    }
    return true;
}

// Builds a general operator: matrix-free where general_mf_plan takes it,
// else A and A^T as ELL matrices (host, FP64 weights rounded to FP32 once),
// uploaded.
static misr_status build_general(misr_op *op, const misr_geometry *g) {
    op->general = true;
    op->L = op->Lp = op->TH = op->TW = op->TWt = 0;
    const int H = op->H, W = op->W, s = op->s, K = op->K, P = g->psf_size;
    const int h = H / s, w = W / s;
    const long long rows = (long long)K * h * w, n = (long long)H * W;
    op->shifts.assign(2 * (size_t)K, 0.0);
    if (g->shifts_lr) op->shifts.assign(g->shifts_lr, g->shifts_lr + 2 * K);
    {
        OpDev &hd = op->host;
        std::memset(&hd, 0, sizeof hd);
        hd.H = H;
        hd.W = W;
        hd.s = s;
        hd.K = K;
        std::vector<float> ker;
        if (general_mf_plan(g, &hd, &ker)) {
            // the kernels, then their taps by position phase (zero past Q):
            // taps (t, t2) of phase (a, b) are C[a + s t][b + s t2]
            const int Q = hd.Q, NT = (Q + s - 1) / s, QP = s * NT;
            std::vector<float> both(ker);
            both.resize((size_t)K * (Q * Q + QP * QP), 0.f);
            float *pk = both.data() + (size_t)K * Q * Q;
            for (int k = 0; k < K; ++k)
                for (int al = 0; al < Q; ++al)
                    for (int be = 0; be < Q; ++be) {
                        const int ph = (al % s) * s + be % s, tp = (al / s) * NT + be / s;
                        pk[((size_t)k * s * s + ph) * NT * NT + tp] =
                            ker[((size_t)k * Q + al) * Q + be];
                    }
            MISR_HIP(op->gker.ensure(both.size() * 4));
            MISR_HIP(hipMemcpy(op->gker.p, both.data(), both.size() * 4, hipMemcpyHostToDevice));
            hd.gker = op->gker.as<float>();
            hd.gkp = hd.gker + (size_t)K * Q * Q;
            MISR_HIP(op->opdev.ensure(sizeof(OpDev)));
            MISR_HIP(hipMemcpy(op->opdev.p, &hd, sizeof hd, hipMemcpyHostToDevice));
            return MISR_OK;
        }
    }
    std::vector<double> warp(6 * (size_t)K), psf((size_t)K * P * P);
    for (int k = 0; k < K; ++k) {
        general_warp(g, k, warp.data() + 6 * k);
        general_psf(g, k, psf.data() + (size_t)k * P * P);
    }
    op->tv = kGenEll;   // a class of launches of its own
    // rows in parallel chunks: (columns, weights) per row, then the ELL width
    const int nt = (int)std::max(1u, std::min(16u, std::thread::hardware_concurrency()));
    std::vector<std::vector<int>> cc(nt), len(nt);
    std::vector<std::vector<double>> vv(nt);
    std::atomic<bool> oom{false};
    auto work = [&](int t) {
        try {
            std::vector<std::pair<int, double>> ent;
            const long long r0 = rows * t / nt, r1 = rows * (t + 1) / nt;
            for (long long r = r0; r < r1 && !oom; ++r) {
                const int k = (int)(r / ((long long)h * w));
                const long long q = r - (long long)k * h * w;
                general_row(op, warp.data() + 6 * k, psf.data() + (size_t)k * P * P, P,
                            (int)(q / w), (int)(q % w), ent);
                len[t].push_back((int)ent.size());
                for (auto &e : ent) {
                    cc[t].push_back(e.first);
                    vv[t].push_back(e.second);
                }
            }
        } catch (const std::bad_alloc &) {
            oom = true;
        }
    };
    {
        std::vector<std::thread> th;
        for (int t = 1; t < nt; ++t) th.emplace_back(work, t);
        work(0);
        for (auto &x : th) x.join();
    }
    if (oom) throw std::bad_alloc();
    int aw = 1;
    for (auto &l : len)
        for (int x : l) aw = std::max(aw, x);
    std::vector<int> acol((size_t)aw * rows, 0), tcnt(n, 0), rlen(rows, 0);
    std::vector<float> aval((size_t)aw * rows, 0.f);
    {
        long long r = 0;
        for (int t = 0; t < nt; ++t) {
            size_t e = 0;
            for (int l : len[t]) {
                rlen[r] = l;
                for (int q = 0; q < aw; ++q) {
                    const size_t at = (size_t)q * rows + r;
                    if (q < l) {
                        acol[at] = cc[t][e + q];
                        aval[at] = (float)vv[t][e + q];
                        tcnt[cc[t][e + q]]++;
                    } else {
                        acol[at] = l > 0 ? cc[t][e] : 0;   // weight 0 on one of the row's columns
                    }
                }
                e += l;
                ++r;
            }
            std::vector<int>().swap(cc[t]);
            std::vector<double>().swap(vv[t]);
        }
    }
    int tw = 1;
    for (int x : tcnt) tw = std::max(tw, x);
    std::vector<int> tcol((size_t)tw * n, -1);
    std::vector<float> tval((size_t)tw * n, 0.f);
    std::fill(tcnt.begin(), tcnt.end(), 0);
    for (long long r = 0; r < rows; ++r)
        for (int q = 0; q < rlen[r]; ++q) {
            const size_t at = (size_t)q * rows + r;
            const int c = acol[at];
            const int slot = tcnt[c]++;
            tcol[(size_t)slot * n + c] = (int)r;
            tval[(size_t)slot * n + c] = aval[at];
        }
    for (long long c = 0; c < n; ++c) {
        const int first = tcnt[c] > 0 ? tcol[c] : 0;
        for (int q = tcnt[c]; q < tw; ++q) tcol[(size_t)q * n + c] = first;
    }
    MISR_HIP(op->a_col.ensure(acol.size() * 4));
    MISR_HIP(op->a_val.ensure(aval.size() * 4));
    MISR_HIP(op->t_col.ensure(tcol.size() * 4));
    MISR_HIP(op->t_val.ensure(tval.size() * 4));
    MISR_HIP(hipMemcpy(op->a_col.p, acol.data(), acol.size() * 4, hipMemcpyHostToDevice));
    MISR_HIP(hipMemcpy(op->a_val.p, aval.data(), aval.size() * 4, hipMemcpyHostToDevice));
    MISR_HIP(hipMemcpy(op->t_col.p, tcol.data(), tcol.size() * 4, hipMemcpyHostToDevice));
    MISR_HIP(hipMemcpy(op->t_val.p, tval.data(), tval.size() * 4, hipMemcpyHostToDevice));
    OpDev &hd = op->host;
    std::memset(&hd, 0, sizeof hd);   // mf = 0: the stored form
    hd.H = H;
    hd.W = W;
    hd.s = s;
    hd.K = K;
    hd.a_w = aw;
    hd.t_w = tw;
    hd.a_col = op->a_col.as<int>();
    hd.a_val = op->a_val.as<float>();
    hd.t_col = op->t_col.as<int>();
    hd.t_val = op->t_val.as<float>();
    MISR_HIP(op->opdev.ensure(sizeof(OpDev)));
    MISR_HIP(hipMemcpy(op->opdev.p, &hd, sizeof hd, hipMemcpyHostToDevice));
    return MISR_OK;
}

// An image takes the narrow tiles while they are so few that the wide ones
// would leave CUs idle, also with a few more images in the same launch: up to
// 320 at scale 2 (48 x 32; 512^2 HR 54.4 -> 38.7 us a pass, 666^2 54.5 -> 45.3,
// ten of 512^2 147 -> 143, but 1024^2 57.7 -> 61.6), up to 128 at the other
// scales, whose narrow tile does a quarter more work per pixel (scale 3: 576^2
// and smaller 66 -> 55 us a pass, ten of 510^2 98 -> 104).  The rule takes the
// geometry alone, so that a solve has the same tiles by itself, in a batch and
// served.
bool misr::use_narrow(int S, int Lp, int H, int W) {
    const int th = tile_hr(S, Lp), tw = tile_wr(S, Lp | (kNarrow << 8));
    if (th <= 0 || tw <= 0 || tw >= tile_wr(S, Lp)) return false;
    const long long n = (long long)((H + th - 1) / th) * ((W + tw - 1) / tw);
    return n <= (S == 2 ? 320 : 128);
}

// Sets the operator's tiles: variant tv, or (nar) variant 0's kernels on
// narrow tiles.
static void set_tile_variant(misr_op *op, int tv, bool nar) {
    op->tv = tv;
    op->nar = nar;
    const int key = nar ? op->Lp | (kNarrow << 8) : op->kernel_key();
    op->TH = tile_hr(op->s, key);
    op->TW = tile_wr(op->s, key);
    op->TWt = nar ? op->TW : tile_wt(op->s, key);
}

extern "C" misr_status misr_op_create(misr_ctx *ctx, const misr_geometry *g, misr_op **out) {
    if (!ctx || !out) return set_error(MISR_E_INVAL, "ctx/out is NULL");
    *out = nullptr;
    misr_status st = misr_geometry_check(g);
    if (st != MISR_OK) return st;
    MISR_HIP(set_device(ctx->dev));
    auto op = std::make_unique<misr_op>();
    op->ctx = ctx;
    op->pdev.kept = &op->kept;
    op->H = g->hr_h;
    op->W = g->hr_w;
    op->s = g->scale;
    op->K = g->n_frames;
    op->P = g->psf_size;
    if (g->warps || g->psf_2d) {
        try {
            st = build_general(op.get(), g);
        } catch (const std::bad_alloc &) {
            st = set_error(MISR_E_NOMEM, "host memory for the general operator's matrices");
        }
        if (st != MISR_OK) return st;
        ctx->users++;
        *out = op.release();
        return MISR_OK;
    }
    op->L = band_length(g);
    op->Lp = padded_band(op->s, op->L);
    set_tile_variant(op.get(), 0, use_narrow(op->s, op->Lp, op->H, op->W));
    op->shifts.assign(g->shifts_lr, g->shifts_lr + 2 * g->n_frames);
    // taps per frame and axis: [K][2][P], vertical then horizontal
    if (g->psf_frames) {
        op->psf.assign(g->psf_frames, g->psf_frames + 2 * (size_t)op->K * op->P);
    } else {
        op->psf.clear();
        for (int k = 0; k < 2 * op->K; ++k)
            op->psf.insert(op->psf.end(), g->psf_1d, g->psf_1d + g->psf_size);
    }
    const int h = op->H / op->s, w = op->W / op->s, R = (op->P - 1) / 2;
    const int fsy = h + 2 * kPadRows, fsx = w + 2 * kPadRows;
    const size_t fy = (size_t)fsy * op->Lp, fx = (size_t)fsx * op->Lp;
    std::vector<float> wy((size_t)op->K * fy, 0.f), wx((size_t)op->K * fx, 0.f);
    OpDev &hd = op->host;
    std::memset(&hd, 0, sizeof hd);
    for (int k = 0; k < op->K; ++k) {
        const double tx = op->s * op->shifts[2 * k], ty = op->s * op->shifts[2 * k + 1];
        hd.offy[k] = (int)std::floor(ty) - R;
        hd.offx[k] = (int)std::floor(tx) - R;
        const double *taps = op->psf.data() + (size_t)k * 2 * op->P;
        band_weights(op->H, op->s, ty, op->P, taps, op->Lp, hd.offy[k],
                     wy.data() + k * fy + (size_t)kPadRows * op->Lp);
        band_weights(op->W, op->s, tx, op->P, taps + op->P, op->Lp, hd.offx[k],
                     wx.data() + k * fx + (size_t)kPadRows * op->Lp);
        canonical_row(op->H, op->s, ty, op->P, taps, op->Lp, hd.offy[k],
                      wy.data() + k * fy + (size_t)kPadRows * op->Lp, hd.cwy[k], &hd.loy[k],
                      &hd.hiy[k]);
        canonical_row(op->W, op->s, tx, op->P, taps + op->P, op->Lp, hd.offx[k],
                      wx.data() + k * fx + (size_t)kPadRows * op->Lp, hd.cwx[k], &hd.lox[k],
                      &hd.hix[k]);
    }
    MISR_HIP(op->wy.ensure(wy.size() * 4));
    MISR_HIP(op->wx.ensure(wx.size() * 4));
    MISR_HIP(op->opdev.ensure(sizeof(OpDev)));
    MISR_HIP(hipMemcpy(op->wy.p, wy.data(), wy.size() * 4, hipMemcpyHostToDevice));
    MISR_HIP(hipMemcpy(op->wx.p, wx.data(), wx.size() * 4, hipMemcpyHostToDevice));
    hd.wy = op->wy.as<float>() + (size_t)kPadRows * op->Lp;
    hd.wx = op->wx.as<float>() + (size_t)kPadRows * op->Lp;
    hd.H = op->H;
    hd.W = op->W;
    hd.s = op->s;
    hd.K = op->K;
    hd.L = op->Lp;
    hd.fsy = fsy;
    hd.fsx = fsx;
    MISR_HIP(hipMemcpy(op->opdev.p, &hd, sizeof hd, hipMemcpyHostToDevice));
    ctx->users++;
    *out = op.release();
    return MISR_OK;
}

extern "C" misr_status misr_op_destroy(misr_op *op) {
    if (!op) return set_error(MISR_E_INVAL, "op is NULL");
    misr_ctx *ctx = op->ctx;
    (void)set_device(ctx->dev);
    // work of this op still queued anywhere on the device finishes first; a
    // device error it (or earlier work) raised is reported here, after the
    // op is freed
    const hipError_t e = hipDeviceSynchronize();
    delete op;
    ctx->users--;
    if (e != hipSuccess) return hip_fail(e, "device error seen while destroying an operator");
    return MISR_OK;
}

extern "C" int misr_op_band(const misr_op *op) { return op ? op->L : -1; }

extern "C" misr_status misr_op_sparse_width(const misr_op *op, int32_t *a_w, int32_t *t_w) {
    if (!op || !a_w || !t_w) return set_error(MISR_E_INVAL, "NULL argument");
    *a_w = op->general ? op->host.a_w : 0;
    *t_w = op->general ? op->host.t_w : 0;
    return MISR_OK;
}

// General operator checks: FP32 images, untiled, no interpolation start point.
static misr_status check_general(const misr_op *op, const misr_params &p) {
    if (!op->general) return MISR_OK;
    if (p.img_dtype != MISR_F32 || p.y_u16)
        return set_error(MISR_E_INVAL, "general operators take FP32 images (img_dtype f32, "
                         "y_u16 = 0)");
    if (p.tile_lr > 0) return set_error(MISR_E_INVAL, "general operators run untiled");
    if (p.x_init == 2)
        return set_error(MISR_E_INVAL, "multi-image interpolation needs translational frames");
    return MISR_OK;
}

// LR vectors of a general solve (kGenVecs x K h w floats).
static hipError_t ensure_res(const misr_op *op, SolveBufs &b) {
    if (!op->general) return hipSuccess;
    return b.res.ensure((size_t)kGenVecs * op->K * (op->H / op->s) * (op->W / op->s) * 4);
}

// ------------------------------------------------------------- plan build
void misr::init_state(ScgState &s, const misr_params &p, long long N) {
    std::memset(&s, 0, sizeof s);
    s.lam = p.scg_lambda1;
    s.lam_bar = 0.0;
    s.sigma = p.scg_sigma;
    s.N = N;
    s.n_iter = p.n_iter;
    s.success = 1;
    s.active = 1;
    for (int dy = 0; dy < 3; ++dy)
        for (int dx = 0; dx < 3; ++dx)
            s.wt.gam[dy * 3 + dx] = (dx == 0 && dy == 0) || dx >= p.btv_w || dy >= p.btv_w
                                        ? 0.f
                                        : (float)(p.lambda_reg * std::pow(p.alpha_btv, dx + dy));
    s.wt.eps = (float)p.eps;
    s.wt.eps_data = (float)p.eps_data;
    s.wt.data_p = p.data_p;
    s.wt.x_rounding = p.x_rounding;
    s.wt.y_scale = p.y_u16 ? (float)p.y_scale : 1.f;
}

struct SolveIn {
    const misr_op *op;
    misr_params prm;
    const void *y;
    void *x;
    SolveBufs *bufs;     // untiled: the view's workspace
    TileSet *tiles;      // tiled (prm.tile_lr > 0): per-tile buffers
};

TileGrid misr::tile_grid(const misr_op *op, const misr_params &p) {
    TileGrid g;
    g.T = p.tile_lr * op->s;
    g.Hh = p.halo_lr * op->s;
    g.ny = (op->H + g.T - 1) / g.T;
    g.nx = (op->W + g.T - 1) / g.T;
    return g;
}

misr_status misr::check_tiling(const misr_op *op, const misr_params &p) {
    if (p.tile_lr <= 0) return MISR_OK;
    const int need = std::max(op->L - 1, 2);
    if (p.halo_lr * op->s < need)
        return set_error(MISR_E_INVAL, "halo of %d LR px (%d HR px) is below the %d HR px the "
                         "operator and prior reach", p.halo_lr, p.halo_lr * op->s, need);
    return MISR_OK;
}

hipError_t misr::ensure_tiles(const misr_op *op, const misr_params &p, TileSet &ts) {
    const TileGrid g = tile_grid(op, p);
    const size_t es = view_esize(p);
    const int nt = g.ny * g.nx;
    if (ts.tile_lr != p.tile_lr || ts.halo_lr != p.halo_lr || ts.es != es ||
        (int)ts.bufs.size() != nt) {
        ts.bufs.clear();
        ts.x0.clear();
        ts.tile_lr = p.tile_lr;
        ts.halo_lr = p.halo_lr;
        ts.es = es;
    }
    for (int a = 0; a < g.ny; ++a)
        for (int b = 0; b < g.nx; ++b) {
            const int t = a * g.nx + b;
            const int r0 = std::max(0, a * g.T - g.Hh), r1 = std::min(op->H, (a + 1) * g.T + g.Hh);
            const int c0 = std::max(0, b * g.T - g.Hh), c1 = std::min(op->W, (b + 1) * g.T + g.Hh);
            const long long n = (long long)(r1 - r0) * (c1 - c0);
            if ((int)ts.bufs.size() <= t) {
                ts.bufs.emplace_back(new SolveBufs());
                ts.x0.emplace_back(new DevMem());
                ts.bufs.back()->set_pool(ts.pool);
                ts.x0.back()->pool = ts.pool;
            }
            hipError_t e = ts.bufs[t]->ensure(n, es);
            if (e == hipSuccess) e = ts.x0[t]->ensure(n * es);
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

// Tiles of a view in work-list order (strip_tile).  Each XCD takes a
// contiguous run of the list, and a tile re-reads its window's margin rows
// from the tiles above and below it: a wide image is listed in strips of a
// few tile columns, so that those neighbours are a few items apart and their
// rows still in the XCD's L2, instead of a whole tile row apart (the windows
// of the 64 tiles of a 6144-px row fill an XCD's 4 MB L2).
static void add_items(std::vector<Item> &items, int pj, int rows, int cols, int TH, int TW,
                      bool nar) {
    const int nty = (rows + TH - 1) / TH, ntx = (cols + TW - 1) / TW;
    for (int i = 0; i < nty * ntx; ++i) {
        int ty, tx;
        strip_tile(i, nty, ntx, ty, tx);
        items.push_back(Item{pj, ty, tx, nar ? 1 : 0});
    }
}

void misr::add_views(const misr_op *op, const misr_params &prm, const void *y, void *x,
                     SolveBufs *bufs, TileSet *tiles, std::vector<Proj> &projs,
                     std::vector<Item> &items, std::vector<Item> &items_u,
                     std::vector<HaloCopy> &halos) {
    Proj P;
    std::memset(&P, 0, sizeof P);
    P.y = y;
    P.op = op->opdev.as<OpDev>();
    if (op->general) {
        // one untiled FP32 view; LR items (role 0) then HR items (role 1),
        // in both lists
        P.x[0] = x;
        P.x[1] = bufs->x1.p;
        P.p[0] = bufs->p0.as<float>();
        P.p[1] = bufs->p1.as<float>();
        P.g[0] = bufs->g0.as<float>();
        P.g[1] = bufs->g1.as<float>();
        const size_t m = (size_t)op->K * (op->H / op->s) * (op->W / op->s);
        P.res = bufs->res.as<float>();
        P.ax[0] = P.res + m;
        P.ax[1] = P.res + 2 * m;
        P.ap[0] = P.res + 3 * m;
        P.ap[1] = P.res + 4 * m;
        P.ld = P.Wb = op->W;
        P.Hb = op->H;
        P.oy1 = P.uy1 = op->H;
        P.ox1 = P.ux1 = op->W;
        const int pj = (int)projs.size();
        projs.push_back(P);
        // matrix-free: LR tiles (all frames) then HR tiles; stored: blocks
        // of kGenRows LR rows then HR rows
        const long long rows = (long long)op->K * (op->H / op->s) * (op->W / op->s);
        const long long n = (long long)op->H * op->W;
        const long long nlr = op->host.mf ? mf_lr_tiles(op->H, op->W, op->s, op->K)
                                          : (rows + kGenRows - 1) / kGenRows;
        const long long nhr = op->host.mf ? mf_hr_tiles(op->H, op->W) : (n + kGenRows - 1) / kGenRows;
        for (auto *lst : {&items, &items_u}) {
            for (long long b = 0; b < nlr; ++b) lst->push_back(Item{pj, (int)b, 0, 0});
            for (long long b = 0; b < nhr; ++b) lst->push_back(Item{pj, (int)b, 1, 0});
        }
        return;
    }
    if (prm.tile_lr <= 0) {
        P.x[0] = iterate_fp32(prm) ? bufs->x0w.p : x;
        P.x[1] = bufs->x1.p;
        P.p[0] = bufs->p0.as<float>();
        P.p[1] = bufs->p1.as<float>();
        P.g[0] = bufs->g0.as<float>();
        P.g[1] = bufs->g1.as<float>();
        P.ld = P.Wb = op->W;
        P.Hb = op->H;
        P.oy1 = P.uy1 = op->H;
        P.ox1 = P.ux1 = op->W;
        P.ntx = (op->W + op->TW - 1) / op->TW;
        const int pj = (int)projs.size();
        projs.push_back(P);
        add_items(items, pj, op->H, op->W, op->TH, op->TWt, op->nar);
        add_items(items_u, pj, op->H, op->W, op->TH, op->TW, op->nar);
        return;
    }
    const TileGrid g = tile_grid(op, prm);
    const int v0 = (int)projs.size();
    for (int a = 0; a < g.ny; ++a)
        for (int b = 0; b < g.nx; ++b) {
            const int t = a * g.nx + b;
            SolveBufs &tb = *tiles->bufs[t];
            const int R0 = a * g.T, R1 = std::min(op->H, (a + 1) * g.T);
            const int C0 = b * g.T, C1 = std::min(op->W, (b + 1) * g.T);
            const int r0 = std::max(0, R0 - g.Hh), r1 = std::min(op->H, R1 + g.Hh);
            const int c0 = std::max(0, C0 - g.Hh), c1 = std::min(op->W, C1 + g.Hh);
            Proj Q = P;
            Q.x[0] = tiles->x0[t]->p;
            Q.x[1] = tb.x1.p;
            Q.p[0] = tb.p0.as<float>();
            Q.p[1] = tb.p1.as<float>();
            Q.g[0] = tb.g0.as<float>();
            Q.g[1] = tb.g1.as<float>();
            Q.ld = Q.Wb = c1 - c0;
            Q.Hb = r1 - r0;
            Q.gy0 = r0;
            Q.gx0 = c0;
            Q.oy0 = R0 - r0;
            Q.oy1 = R1 - r0;
            Q.ox0 = C0 - c0;
            Q.ox1 = C1 - c0;
            Q.uy0 = 0;
            Q.uy1 = Q.Hb;
            Q.ux0 = 0;
            Q.ux1 = Q.Wb;
            Q.ntx = (C1 - C0 + op->TW - 1) / op->TW;
            const int pj = (int)projs.size();
            projs.push_back(Q);
            add_items(items, pj, R1 - R0, C1 - C0, op->TH, op->TWt, op->nar);
            add_items(items_u, pj, Q.Hb, Q.Wb, op->TH, op->TW, op->nar);
        }
    // halo exchanges: every view's halo from the views that own it
    const int v1 = (int)projs.size();
    for (int bi = v0; bi < v1; ++bi)
        for (int ai = v0; ai < v1; ++ai) {
            if (ai == bi) continue;
            const Proj &A = projs[ai], &B = projs[bi];
            const int gy0 = std::max(B.gy0, A.gy0 + A.oy0);
            const int gy1 = std::min(B.gy0 + B.Hb, A.gy0 + A.oy1);
            const int gx0 = std::max(B.gx0, A.gx0 + A.ox0);
            const int gx1 = std::min(B.gx0 + B.Wb, A.gx0 + A.ox1);
            if (gy1 > gy0 && gx1 > gx0)
                halos.push_back(HaloCopy{ai, bi, gy0, gx0, gy1 - gy0, gx1 - gx0});
        }
}

// Builds the work lists: solves grouped by kernel class (S, Lp), each solve's
// items contiguous so that its partial sums form one range.
static void build_plan(Plan &pl, const std::vector<SolveIn> &in) {
    pl.projs.clear();
    pl.items.clear();
    pl.items_u.clear();
    pl.states.clear();
    pl.classes.clear();
    pl.classes_u.clear();
    pl.proj_solve.clear();
    pl.refs.clear();
    pl.halos.clear();
    pl.tiled = false;
    pl.staged = false;
    pl.inits.clear();
    pl.steps = true;
    pl.apart.assign(in.size(), 0);
    pl.vt = in.empty() ? (int)ST_F32 : view_stype(in[0].prm);
    pl.gt = in.empty() ? (int)ST_F32 : (int)in[0].prm.img_dtype;
    pl.yt = in.empty() ? (int)ST_F32 : frame_stype(in[0].prm);
    const size_t ns = in.size();
    pl.item0.assign(ns, 0);
    pl.nitems.assign(ns, 0);
    pl.item0u.assign(ns, 0);
    pl.nitemsu.assign(ns, 0);
    std::map<std::pair<int, int>, std::vector<int>> groups;
    std::vector<std::pair<int, int>> order;
    for (int i = 0; i < (int)ns; ++i) {
        auto key = std::make_pair(in[i].op->s, in[i].op->kernel_key());
        if (!groups.count(key)) order.push_back(key);
        groups[key].push_back(i);
    }
    pl.states.resize(ns);
    for (auto &key : order) {
        Plan::Cls c{key.first, key.second, (int)pl.items.size(), 0};
        Plan::Cls cu{key.first, key.second, (int)pl.items_u.size(), 0};
        for (int i : groups[key]) {
            const SolveIn &si = in[i];
            const misr_op *op = si.op;
            init_state(pl.states[i], si.prm, (long long)op->H * op->W);
            pl.apart[i] = op->general;
            pl.item0[i] = (int)pl.items.size();
            pl.item0u[i] = (int)pl.items_u.size();
            if (si.prm.tile_lr > 0 || iterate_fp32(si.prm)) {
                pl.tiled |= si.prm.tile_lr > 0;
                pl.staged = true;
                pl.states[i].xglob = si.x;
                pl.states[i].ldg = op->W;
            }
            if (si.prm.x_init > 0)
                pl.inits.push_back(Plan::Init{si.prm.x_init, init_args(op), si.y, si.x,
                                              (int)si.prm.img_dtype});
            add_views(op, si.prm, si.y, si.x, si.bufs, si.tiles, pl.projs, pl.items, pl.items_u,
                      pl.halos);
            pl.proj_solve.resize(pl.projs.size(), i);
            pl.nitems[i] = (int)pl.items.size() - pl.item0[i];
            pl.nitemsu[i] = (int)pl.items_u.size() - pl.item0u[i];
        }
        c.count = (int)pl.items.size() - c.start;
        cu.count = (int)pl.items_u.size() - cu.start;
        pl.classes.push_back(c);
        pl.classes_u.push_back(cu);
    }
    pl.finish_counts();
}

// Everything a captured solve bakes in as launch arguments: pass count,
// storage codes, counts and class ranges.  The caller's buffers are not among
// them (the views hold those; the start-point kernels that take them directly
// are launched before the graph), so a captured solve serves new frames.
static std::string plan_key(const Plan &pl, int n_iter) {
    std::string k = std::to_string(n_iter) + "/" + std::to_string(pl.code()) + "," +
                    std::to_string(pl.gt) + "/" + std::to_string(pl.states.size()) + "/" +
                    std::to_string(pl.projs.size()) + "/" + std::to_string(pl.halos.size()) +
                    (pl.staged ? "S" : "U");
    for (auto &c : pl.classes)
        k += ":" + std::to_string(c.S) + "," + std::to_string(c.Lp) + "," +
             std::to_string(c.start) + "," + std::to_string(c.count);
    for (auto &c : pl.classes_u)
        k += ";" + std::to_string(c.start) + "," + std::to_string(c.count);
    return k;
}

// Launch helpers over a plan's device mirror.
struct Launcher {
    const Plan &pl;
    PlanDev &pd;
    hipStream_t s;
    const int *cnt() const { return pd.counts.as<int>(); }
    hipError_t image(int kind) const {
        for (int c = 0; c < (int)pl.classes.size(); ++c) {
            hipError_t e = image(kind, c, s);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    // one launch class's pass
    hipError_t image(int kind, int c, hipStream_t s) const {
        const bool upd = kind == KIND_UPCURV;
        const auto &cls = upd ? pl.classes_u : pl.classes;
        const Item *items = upd ? pd.items_u.as<Item>() : pd.items.as<Item>();
        double *part = upd ? pd.partials_u.as<double>() : pd.partials.as<double>();
        const int off = upd ? (int)pl.classes.size() : 0;
        // band length 0: the classes of general operators
        return (cls[c].Lp & 255) == 0
                   ? launch_general(cls[c].count, s, pd.projs.as<Proj>(), items + cls[c].start,
                                    cnt() + off + c, part + (size_t)cls[c].start * kNV, kind,
                                    cls[c].S, cls[c].Lp >> 8 == kGenEll)
                   : launch_image(cls[c].S, cls[c].Lp, cls[c].count, s, pd.projs.as<Proj>(),
                                  items + cls[c].start, cnt() + off + c,
                                  part + (size_t)cls[c].start * kNV, kind, pl.code());
    }
    // the SCG steps after a pass, of the solves whose passes do not end with them
    hipError_t scalar(int kind) const {
        if (!pl.any_apart(1)) return hipSuccess;
        return launch_scalar((int)pl.states.size(), s, pd.refs.as<SolveRef>(), kind, 1);
    }
    hipError_t halo() const {
        if (pl.halos.empty()) return hipSuccess;
        return launch_halo(s, pd.projs.as<Proj>(), pd.halos.as<HaloCopy>(),
                           cnt() + pl.n_halos_idx(), (int)pl.halos.size());
    }
};

// Streams and events that only a capture uses: its branches.
struct Branches {
    std::vector<hipStream_t> st;
    std::vector<hipEvent_t> ev;
    ~Branches() {
        for (auto e : ev) (void)hipEventDestroy(e);
        for (auto s : st) (void)hipStreamDestroy(s);
    }
    hipError_t fork(hipStream_t from, hipStream_t *to) {
        hipStream_t b;
        hipError_t e = hipStreamCreateWithFlags(&b, hipStreamNonBlocking);
        if (e != hipSuccess) return e;
        st.push_back(b);
        *to = b;
        return order(from, b);
    }
    // work on `after` from here on follows the work on `s` so far
    hipError_t order(hipStream_t s, hipStream_t after) {
        hipEvent_t v;
        hipError_t e = hipEventCreateWithFlags(&v, hipEventDisableTiming);
        if (e != hipSuccess) return e;
        ev.push_back(v);
        if ((e = hipEventRecord(v, s)) != hipSuccess) return e;
        return hipStreamWaitEvent(after, v, 0);
    }
};
// Branches of a batch's graph at most (the device has four queues per process).
constexpr int kMaxBranches = 4;

// Enqueues the whole solve (init + n_iter passes + result copy) on `s` (being
// captured, with `br` for branches); last: where the final state of a single
// solve is kept, or NULL.
static hipError_t enqueue_solve(const Plan &pl, PlanDev &pd, int n_iter, ScgState *last,
                                hipStream_t s, Branches &br) {
    const Launcher Lr{pl, pd, s};
    const int np = (int)pl.projs.size();
    hipError_t e = hipSuccess;
#define STEP(x)                          \
    if ((e = (x)) != hipSuccess) return e;
    if (pl.staged) STEP(launch_scatter(s, pd.projs.as<Proj>(), np, pl.vt, pl.gt));
    const int nc = (int)pl.classes.size();
    if (nc > 1 && pl.halos.empty() && !pl.any_apart(1)) {
        // Solves of different launch classes (scales, band lengths) share
        // nothing and their passes end with their own steps: each class is a
        // branch of the graph, so that one's last workgroups do not leave the
        // device idle before the next (6 solves, 4 of scale 2 and 2 of scale 3, LR
        // 768 x 512 and less, 60 passes: 15.7 -> 12.0 ms)
        std::vector<hipStream_t> bs(std::min(nc, kMaxBranches), s);
        for (size_t b = 1; b < bs.size(); ++b) STEP(br.fork(s, &bs[b]));
        for (int c = 0; c < nc; ++c) {
            const hipStream_t b = bs[c % bs.size()];
            STEP(Lr.image(KIND_COSTGRAD, c, b));
            STEP(Lr.image(KIND_UPCURV, c, b));
            for (int it = 0; it < n_iter; ++it) {
                STEP(Lr.image(KIND_TRIAL, c, b));
                STEP(Lr.image(KIND_UPCURV, c, b));
            }
        }
        for (size_t b = 1; b < bs.size(); ++b) STEP(br.order(bs[b], s));
        n_iter = -1;   // (all passes enqueued)
    } else {
        STEP(Lr.image(KIND_COSTGRAD));
        STEP(Lr.halo());
        STEP(Lr.scalar(KIND_COSTGRAD));
        STEP(Lr.image(KIND_UPCURV));
    }
    for (int it = 0; it < n_iter; ++it) {
        STEP(Lr.scalar(KIND_UPCURV));
        STEP(Lr.image(KIND_TRIAL));
        STEP(Lr.halo());
        STEP(Lr.scalar(KIND_TRIAL));
        STEP(Lr.image(KIND_UPCURV));
    }
    if (last) STEP(launch_copy_state(s, last, pd.states.as<ScgState>()));
#undef STEP
    // staged views: owned parts back into the caller's image (rounded to its
    // storage); an unstaged view copies its workspace buffer back when the
    // iterate ended there
    return pl.staged ? launch_gather(s, pd.projs.as<Proj>(), np, pl.vt, pl.gt, 0)
                     : launch_finalize(s, pd.projs.as<Proj>(), np, pl.vt);
}

// A solve is a graph of its own, which HIP launches at once also where the
// stream is being captured: it would run now, on whatever the operator's
// arrays hold, and not when the caller's graph does.
static misr_status check_not_capturing(hipStream_t s) {
    return capturing(s) ? set_error(MISR_E_HIP, "a solve cannot be captured: the stream is "
                                    "recording a graph")
                        : MISR_OK;
}

// Runs a plan; the solve is captured into a graph (on the context's library
// stream) once per plan shape and replayed.  A single solve replays on the
// caller's stream: its workspace is the operator's, whose calls the caller
// orders.  A batch, whose workspace all batches share, replays on the library
// stream, ordered after the caller's stream and before its later work.
static misr_status run_plan(misr_ctx *ctx, Plan &pl, PlanDev &pd, int n_iter, ScgState *last,
                            bool shared, hipStream_t user) {
    hipStream_t s = shared ? ctx->stream : user;
    if (shared) {
        MISR_HIP(hipEventRecord(ctx->ev_in, user));
        MISR_HIP(hipStreamWaitEvent(s, ctx->ev_in, 0));
    }
    MISR_HIP(pd.upload(pl, n_iter, s));
    // the graph bakes in the device addresses of the plan arrays
    char ptrs[256];
    snprintf(ptrs, sizeof ptrs, "|%p,%p,%p,%p,%p,%p,%p,%p,%p,%p", pd.projs.p, pd.items.p,
             pd.items_u.p, pd.counts.p, pd.states.p, pd.partials.p, pd.partials_u.p, pd.refs.p,
             pd.halos.p, (void *)last);
    const std::string key = plan_key(pl, n_iter) + ptrs;
    if (!pd.exec || pd.graph_key != key) {
        if (pd.exec) {
            (void)hipGraphExecDestroy(pd.exec);
            pd.exec = nullptr;
        }
        hipGraph_t graph = nullptr;
        MISR_HIP(hipStreamBeginCapture(ctx->stream, hipStreamCaptureModeThreadLocal));
        Branches br;
        hipError_t e = enqueue_solve(pl, pd, n_iter, last, ctx->stream, br);
        hipError_t e2 = hipStreamEndCapture(ctx->stream, &graph);
        if (e != hipSuccess) {
            if (graph) (void)hipGraphDestroy(graph);
            return hip_fail(e, "enqueue_solve (capture)");
        }
        if (e2 != hipSuccess) return hip_fail(e2, "hipStreamEndCapture");
        e = hipGraphInstantiate(&pd.exec, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        if (e != hipSuccess) {
            pd.exec = nullptr;
            return hip_fail(e, "hipGraphInstantiate");
        }
        pd.graph_key = key;
    }
    pd.states_dirty = true;   // from here on the kernels write them
    for (auto &it : pl.inits) MISR_HIP(launch_init(s, it.kind, it.a, it.y, it.x, it.st));
    MISR_HIP(hipGraphLaunch(pd.exec, s));
    if (shared) {
        MISR_HIP(hipEventRecord(ctx->ev_out, s));
        MISR_HIP(hipStreamWaitEvent(user, ctx->ev_out, 0));
    }
    return MISR_OK;
}

static misr_status fetch_trace(PlanDev &pd, int idx, misr_scg_trace *tr, hipStream_t user) {
    ScgState st;
    MISR_HIP(hipMemcpyAsync(&st, pd.states.as<ScgState>() + idx, sizeof st, hipMemcpyDeviceToHost,
                            user));
    MISR_HIP(hipStreamSynchronize(user));
    tr->n_passes = st.it;
    tr->n_success = st.n_success;
    tr->stop = st.stop;
    tr->E0 = st.E0;
    tr->E_final = st.E;
    if (tr->iters && tr->capacity > 0 && st.it > 0) {
        const int n = st.it < tr->capacity ? st.it : tr->capacity;
        static_assert(sizeof(IterRec) == sizeof(misr_scg_iter), "trace record layout");
        MISR_HIP(hipMemcpy(tr->iters, pd.traces.as<IterRec>() + (size_t)idx * pd.n_iter_max,
                           n * sizeof(IterRec), hipMemcpyDeviceToHost));
    }
    return st.stop == 2 ? set_error(MISR_E_NUMERIC, "non-finite cost or curvature at pass %d",
                                    st.it)
                        : MISR_OK;
}

// ------------------------------------------------------------ operators
// The plan of a standalone operator; its buffers go with the launch.
static void single_view(misr_op *op, Plan &pl) {
    SolveIn si{op, {}, nullptr, nullptr, &op->bufs, nullptr};
    misr_params_default(&si.prm);
    si.prm.n_iter = 0;
    build_plan(pl, {si});
}

extern "C" misr_status misr_forward(const misr_op *cop, misr_dtype dt, const void *x, void *y,
                                    void *stream) {
    misr_op *op = const_cast<misr_op *>(cop);
    if (!op || !x || !y) return set_error(MISR_E_INVAL, "NULL argument");
    if (dt != MISR_F32 && dt != MISR_F16 && dt != MISR_BF16)
        return set_error(MISR_E_INVAL, "dtype invalid");
    std::lock_guard<std::mutex> lk(op->mu);
    MISR_HIP(set_device(op->ctx->dev));
    if (op->general) {
        if (dt != MISR_F32) return set_error(MISR_E_INVAL, "general operators take FP32 images");
        MISR_HIP(launch_general_forward(
            (hipStream_t)stream, op->opdev.as<OpDev>(),
            (long long)op->K * (op->H / op->s) * (op->W / op->s), (const float *)x, (float *)y,
            op->host.mf ? mf_lr_tiles(op->H, op->W, op->s, op->K) : 0, op->s));
        return MISR_OK;
    }
    Plan &pl = op->plan;
    single_view(op, pl);
    PlanDev &pd = op->pdev;
    hipStream_t s = (hipStream_t)stream;
    MISR_HIP(pd.upload(pl, 0, s));
    // the update list: tiles of the operator's (update-pass) shape
    MISR_HIP(launch_forward(op->s, op->kernel_key(), (int)pl.items_u.size(), s,
                            pd.projs.as<Proj>(), pd.items_u.as<Item>(), (int)pl.items_u.size(),
                            (int)dt, x, y));
    return MISR_OK;
}

extern "C" misr_status misr_adjoint(const misr_op *cop, misr_dtype dt, const void *r, float *x,
                                    void *stream) {
    misr_op *op = const_cast<misr_op *>(cop);
    if (!op || !x || !r) return set_error(MISR_E_INVAL, "NULL argument");
    if (dt != MISR_F32 && dt != MISR_F16 && dt != MISR_BF16)
        return set_error(MISR_E_INVAL, "dtype invalid");
    std::lock_guard<std::mutex> lk(op->mu);
    MISR_HIP(set_device(op->ctx->dev));
    if (op->general) {
        if (dt != MISR_F32) return set_error(MISR_E_INVAL, "general operators take FP32 images");
        MISR_HIP(launch_general_adjoint((hipStream_t)stream, op->opdev.as<OpDev>(),
                                        (long long)op->H * op->W, (const float *)r, x,
                                        op->host.mf ? mf_hr_tiles(op->H, op->W) : 0, op->s));
        return MISR_OK;
    }
    Plan &pl = op->plan;
    single_view(op, pl);
    PlanDev &pd = op->pdev;
    hipStream_t s = (hipStream_t)stream;
    MISR_HIP(pd.upload(pl, 0, s));
    MISR_HIP(launch_adjoint(op->s, op->kernel_key(), (int)pl.items_u.size(), s,
                            pd.projs.as<Proj>(), pd.items_u.as<Item>(), (int)pl.items_u.size(),
                            (int)dt, r, x));
    return MISR_OK;
}

InitArgs misr::init_args(const misr_op *op) {
    InitArgs a;
    std::memset(&a, 0, sizeof a);
    a.H = op->H;
    a.W = op->W;
    a.s = op->s;
    a.K = op->K;
    for (int k = 0; k < op->K; ++k) {
        a.tx[k] = (int)std::lround(op->s * op->shifts[2 * k + 0]);
        a.ty[k] = (int)std::lround(op->s * op->shifts[2 * k + 1]);
    }
    return a;
}

static misr_status start_point(const misr_op *op, int kind, misr_dtype dt, const void *y,
                               void *x, void *stream) {
    if (!op || !y || !x) return set_error(MISR_E_INVAL, "NULL argument");
    if (dt != MISR_F32 && dt != MISR_F16 && dt != MISR_BF16)
        return set_error(MISR_E_INVAL, "dtype invalid");
    MISR_HIP(set_device(op->ctx->dev));
    MISR_HIP(launch_init((hipStream_t)stream, kind, init_args(op), y, x, (int)dt));
    return MISR_OK;
}

extern "C" misr_status misr_interpolate(const misr_op *op, misr_dtype dt, const void *y, void *x,
                                        void *stream) {
    if (op && op->general)
        return set_error(MISR_E_INVAL, "multi-image interpolation needs translational frames");
    return start_point(op, 2, dt, y, x, stream);
}

extern "C" misr_status misr_upsample(const misr_op *op, misr_dtype dt, const void *y, void *x,
                                     void *stream) {
    return start_point(op, 1, dt, y, x, stream);
}

extern "C" misr_status misr_cost_grad(const misr_op *cop, const misr_params *prm, const void *x,
                                      const void *y, float *g, double *cost_dev, void *stream) {
    misr_op *op = const_cast<misr_op *>(cop);
    if (!op || !x || !y || !g || !cost_dev) return set_error(MISR_E_INVAL, "NULL argument");
    misr_status st = misr_params_check(prm);
    if (st != MISR_OK) return st;
    if ((st = check_general(op, *prm)) != MISR_OK) return st;
    if ((st = check_tiling(op, *prm)) != MISR_OK) return st;
    std::lock_guard<std::mutex> lk(op->mu);
    MISR_HIP(set_device(op->ctx->dev));
    const size_t es = dtype_size(prm->img_dtype);
    const long long n = (long long)op->H * op->W;
    MISR_HIP(op->bufs.ensure(n, es));
    MISR_HIP(ensure_res(op, op->bufs));
    if (prm->tile_lr > 0) MISR_HIP(ensure_tiles(op, *prm, op->tiles));
    Plan &pl = op->plan;
    SolveIn si{op, *prm, y, const_cast<void *>(x), &op->bufs, &op->tiles};
    si.prm.n_iter = 0;
    si.prm.x_work = 1;   // evaluated at x as stored: no FP32 copy
    si.prm.x_init = 0;
    build_plan(pl, {si});
    if (pl.tiled)
        pl.states[0].gglob = g;
    else
        pl.projs[0].g[1] = g;   // the init pass writes g[cur ^ 1] with cur = 0
    pl.steps = false;
    PlanDev &pd = op->pdev;
    hipStream_t s = (hipStream_t)stream;
    if (capturing(s)) {
        op->bufs.keep(op->kept);
        if (prm->tile_lr > 0) op->tiles.keep(op->kept);
    }
    MISR_HIP(pd.upload(pl, 0, s));
    const Launcher Lr{pl, pd, s};
    const int np = (int)pl.projs.size();
    if (pl.staged) MISR_HIP(launch_scatter(s, pd.projs.as<Proj>(), np, pl.vt, pl.gt));
    MISR_HIP(Lr.image(KIND_COSTGRAD));
    MISR_HIP(launch_cost_out(s, pd.partials.as<double>(), (int)pl.items.size(), cost_dev));
    if (pl.staged) MISR_HIP(launch_gather(s, pd.projs.as<Proj>(), np, pl.vt, pl.gt, 1));
    return MISR_OK;
}

// ----------------------------------------------------------------- solves
extern "C" misr_status misr_scg_solve(const misr_op *cop, const misr_params *prm, const void *y,
                                      void *x, misr_scg_trace *trace, void *stream) {
    misr_op *op = const_cast<misr_op *>(cop);
    if (!op || !y || !x) return set_error(MISR_E_INVAL, "NULL argument");
    misr_status st = misr_params_check(prm);
    if (st != MISR_OK) return st;
    if ((st = check_general(op, *prm)) != MISR_OK) return st;
    if ((st = check_tiling(op, *prm)) != MISR_OK) return st;
    if ((st = check_not_capturing((hipStream_t)stream)) != MISR_OK) return st;
    std::lock_guard<std::mutex> lk(op->mu);
    std::lock_guard<std::mutex> lc(op->ctx->mu);
    MISR_HIP(set_device(op->ctx->dev));
    const long long n = (long long)op->H * op->W;
    if (prm->tile_lr > 0)
        MISR_HIP(ensure_tiles(op, *prm, op->tiles));
    else
        MISR_HIP(op->bufs.ensure_view(n, *prm));
    MISR_HIP(ensure_res(op, op->bufs));
    Plan &pl = op->plan;
    build_plan(pl, {SolveIn{op, *prm, y, x, &op->bufs, &op->tiles}});
    hipStream_t s = (hipStream_t)stream;
    // the final state goes to last_state, kept for misr_scg_status (later calls
    // on the op reuse the plan's state buffer)
    MISR_HIP(op->last_state.ensure(sizeof(ScgState)));
    st = run_plan(op->ctx, pl, op->pdev, prm->n_iter, op->last_state.as<ScgState>(), false, s);
    if (st != MISR_OK) return st;
    op->have_last = true;
    if (trace) return fetch_trace(op->pdev, 0, trace, s);
    return MISR_OK;
}

extern "C" misr_status misr_scg_status(const misr_op *cop, misr_scg_trace *summary,
                                       void *stream) {
    misr_op *op = const_cast<misr_op *>(cop);
    if (!op) return set_error(MISR_E_INVAL, "op is NULL");
    std::lock_guard<std::mutex> lk(op->mu);
    if (!op->have_last) return set_error(MISR_E_INVAL, "no solve has run on this operator");
    MISR_HIP(set_device(op->ctx->dev));
    hipStream_t s = (hipStream_t)stream;
    ScgState st;
    MISR_HIP(hipMemcpyAsync(&st, op->last_state.p, sizeof st, hipMemcpyDeviceToHost, s));
    MISR_HIP(hipStreamSynchronize(s));
    if (summary) {
        summary->n_passes = st.it;
        summary->n_success = st.n_success;
        summary->stop = st.stop;
        summary->E0 = st.E0;
        summary->E_final = st.E;
    }
    return st.stop == 2 ? set_error(MISR_E_NUMERIC, "non-finite cost or curvature at pass %d",
                                    st.it)
                        : MISR_OK;
}

namespace {
struct BatchCache {
    misr_ctx *ctx = nullptr;
    std::vector<std::unique_ptr<SolveBufs>> bufs;
    PlanDev pdev;
    Plan plan;
};
std::mutex g_batch_mu;
BatchCache *g_batch = nullptr;

// Device bytes of one batch entry's buffers.
size_t batch_bytes(const misr_op *op, const misr_params &p) {
    const size_t n = (size_t)op->H * op->W;
    size_t b = n * (view_esize(p) + 16 + (iterate_fp32(p) ? 4 : 0));
    if (op->general) b += (size_t)kGenVecs * op->K * (op->H / op->s) * (op->W / op->s) * 4;
    return b;
}
}  // namespace

// (a later context may have this one's address, and another device)
static void drop_batch(const misr_ctx *c) {
    std::lock_guard<std::mutex> lk(g_batch_mu);
    if (!g_batch || g_batch->ctx != c) return;
    delete g_batch;
    g_batch = nullptr;
}

extern "C" misr_status misr_scg_solve_batch(int n, const misr_op *const *ops,
                                            const misr_params *prm, const void *const *y,
                                            void *const *x, misr_scg_trace *traces,
                                            void *stream) {
    if (n < 1 || !ops || !prm || !y || !x) return set_error(MISR_E_INVAL, "bad batch arguments");
    misr_ctx *ctx = nullptr;
    for (int i = 0; i < n; ++i) {
        if (!ops[i] || !y[i] || !x[i]) return set_error(MISR_E_INVAL, "NULL entry %d", i);
        misr_status st = misr_params_check(&prm[i]);
        if (st != MISR_OK) return st;
        if ((st = check_general(ops[i], prm[i])) != MISR_OK) return st;
        if (prm[i].tile_lr > 0)
            return set_error(MISR_E_INVAL, "batch entry %d: batched solves are untiled", i);
        if (prm[i].img_dtype != prm[0].img_dtype || prm[i].x_work != prm[0].x_work ||
            prm[i].y_u16 != prm[0].y_u16)
            return set_error(MISR_E_INVAL, "batch entries must share img_dtype, x_work, y_u16");
        if (ctx && ops[i]->ctx != ctx) return set_error(MISR_E_INVAL, "ops span contexts");
        ctx = ops[i]->ctx;
    }
    const misr_status cap = check_not_capturing((hipStream_t)stream);
    if (cap != MISR_OK) return cap;
    std::lock_guard<std::mutex> lk(g_batch_mu);
    std::lock_guard<std::mutex> lc(ctx->mu);
    MISR_HIP(set_device(ctx->dev));
    // one context's batches at a time (another's stream does not wait for
    // this one's; freeing the buffers waits for the device)
    if (g_batch && g_batch->ctx != ctx) {
        delete g_batch;
        g_batch = nullptr;
    }
    if (!g_batch) {
        g_batch = new BatchCache();
        g_batch->ctx = ctx;
    }
    BatchCache &bc = *g_batch;
    // Batches share one set of buffers per entry, grown as needed (a program
    // that alternates between batches allocates nothing), and given back when
    // they hold more than twice what the batch at hand needs.
    size_t need = 0, have = 0;
    for (int i = 0; i < n; ++i)
        need += batch_bytes(ops[i], prm[i]);
    for (auto &b : bc.bufs) have += b->bytes();
    if (have > 2 * need) bc.bufs.clear();
    int n_iter = 0;
    for (int i = 0; i < n; ++i) n_iter = std::max(n_iter, prm[i].n_iter);
    std::vector<SolveIn> in;
    for (int i = 0; i < n; ++i) {
        if ((int)bc.bufs.size() <= i) bc.bufs.emplace_back(new SolveBufs());
        MISR_HIP(bc.bufs[i]->ensure_view((long long)ops[i]->H * ops[i]->W, prm[i]));
        MISR_HIP(ensure_res(ops[i], *bc.bufs[i]));
        in.push_back(SolveIn{ops[i], prm[i], y[i], x[i], bc.bufs[i].get(), nullptr});
    }
    build_plan(bc.plan, in);
    hipStream_t s = (hipStream_t)stream;
    misr_status st = run_plan(ctx, bc.plan, bc.pdev, n_iter, nullptr, true, s);
    if (st != MISR_OK) return st;
    misr_status worst = MISR_OK;
    if (traces)
        for (int i = 0; i < n; ++i) {
            misr_status t = fetch_trace(bc.pdev, i, &traces[i], s);
            if (t != MISR_OK) worst = t;
        }
    return worst;
}

// ------------------------------------------------------------- measurement
// One image pass timed with HIP events (caller holds op->mu and the ctx lock).
static misr_status time_pass_impl(misr_op *op, const misr_params *prm, const void *y, void *x,
                                  int which, int reps, double *avg_us, void *stream) {
    const long long n = (long long)op->H * op->W;
    MISR_HIP(op->bufs.ensure(n, dtype_size(prm->img_dtype)));
    MISR_HIP(ensure_res(op, op->bufs));
    Plan &pl = op->plan;
    misr_params p1 = *prm;
    p1.n_iter = 1;
    p1.x_work = 1;   // the passes over x as stored
    p1.x_init = 0;
    build_plan(pl, {SolveIn{op, p1, y, x, &op->bufs, nullptr}});
    PlanDev &pd = op->pdev;
    hipStream_t s = op->ctx->stream;
    MISR_HIP(hipEventRecord(op->ctx->ev_in, (hipStream_t)stream));
    MISR_HIP(hipStreamWaitEvent(s, op->ctx->ev_in, 0));
    MISR_HIP(pd.upload(pl, 1, s));
    pd.states_dirty = true;   // the SCG steps write them
    const Launcher Lr{pl, pd, s};
    MISR_HIP(Lr.image(KIND_COSTGRAD));
    MISR_HIP(Lr.scalar(KIND_COSTGRAD));
    MISR_HIP(Lr.image(KIND_UPCURV));
    MISR_HIP(Lr.scalar(KIND_UPCURV));
    // from here on the passes leave the state as it is, an update pending
    pl.projs[0].ref = nullptr;
    pd.held[0].p = nullptr;   // (the view on the device is not what upload put there)
    PutArgs put;
    put.n = 2;
    put.dst[0] = pd.projs.as<unsigned>();
    put.words[0] = (int)(sizeof(Proj) / 4);
    std::memcpy(put.w, &pl.projs[0], sizeof(Proj));
    put.dst[1] = (unsigned *)&pd.states.as<ScgState>()->do_update;
    put.words[1] = 1;
    put.w[put.words[0]] = 1;
    MISR_HIP(launch_put(s, put));
    hipEvent_t e0, e1;
    MISR_HIP(hipEventCreate(&e0));
    MISR_HIP(hipEventCreate(&e1));
    // which 2: a trial pass and then an update pass, as they follow each
    // other in a solve (the update writes the x and p the trial reads)
    auto pass = [&]() {
        hipError_t e1 = Lr.image(which == 1 ? KIND_UPCURV : KIND_TRIAL);
        if (e1 == hipSuccess && which == 2) e1 = Lr.image(KIND_UPCURV);
        return e1;
    };
    hipError_t e = pass();   // warm-up launch
    if (e == hipSuccess) e = hipEventRecord(e0, s);
    for (int r = 0; r < reps && e == hipSuccess; ++r) e = pass();
    if (e == hipSuccess) e = hipEventRecord(e1, s);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float ms = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (e != hipSuccess) return hip_fail(e, "misr_time_pass");
    *avg_us = 1e3 * ms / reps;
    return MISR_OK;
}

extern "C" misr_status misr_time_pass(const misr_op *cop, const misr_params *prm, const void *y,
                                      void *x, int which, int reps, double *avg_us,
                                      void *stream) {
    misr_op *op = const_cast<misr_op *>(cop);
    if (!op || !y || !x || !avg_us || reps < 1 || which < 0 || which > 2)
        return set_error(MISR_E_INVAL, "bad arguments");
    misr_status st = misr_params_check(prm);
    if (st != MISR_OK) return st;
    if (prm->tile_lr > 0) return set_error(MISR_E_INVAL, "timing runs untiled");
    if ((st = check_general(op, *prm)) != MISR_OK) return st;
    std::lock_guard<std::mutex> lk(op->mu);
    std::lock_guard<std::mutex> lc(op->ctx->mu);
    MISR_HIP(set_device(op->ctx->dev));
    return time_pass_impl(op, prm, y, x, which, reps, avg_us, stream);
}

// ------------------------------------------------------------ tile autotuner
extern "C" misr_status misr_op_tune(misr_op *op, const misr_params *prm, const void *y, void *x,
                                    int reps, int32_t *tile_h, int32_t *tile_w, void *stream) {
    if (!op || !y || !x || !tile_h || !tile_w || reps < 1)
        return set_error(MISR_E_INVAL, "bad arguments");
    misr_status st = misr_params_check(prm);
    if (st != MISR_OK) return st;
    if (prm->tile_lr > 0) return set_error(MISR_E_INVAL, "tuning runs untiled");
    if ((st = check_general(op, *prm)) != MISR_OK) return st;
    std::lock_guard<std::mutex> lk(op->mu);
    std::lock_guard<std::mutex> lc(op->ctx->mu);
    MISR_HIP(set_device(op->ctx->dev));
    if (!op->general) {
        // kept if a timing run fails
        const int prev = op->tv;
        const bool prev_nar = op->nar;
        const bool can_nar = use_narrow(op->s, op->Lp, op->H, op->W);
        double best = 0.0;
        int best_tv = -1;
        bool best_nar = false;
        for (int c = 0; c < 4; ++c) {
            // the three variants, then the narrow tiles of a small image
            const int tv = c < 3 ? c : 0;
            const bool nar = c == 3;
            if (nar ? !can_nar : tile_hr(op->s, op->Lp | (tv << 8)) <= 0) continue;
            set_tile_variant(op, tv, nar);
            // the two passes alternating, as in a solve: a trial tile that
            // lines up with the update tiles finds the update's output in its
            // XCD's L2, which timing each pass alone would not show
            double t_pair = 0.0;
            if ((st = time_pass_impl(op, prm, y, x, 2, reps, &t_pair, stream)) != MISR_OK) {
                set_tile_variant(op, prev, prev_nar);
                return st;
            }
            if (best_tv < 0 || t_pair < best) {
                best = t_pair;
                best_tv = tv;
                best_nar = nar;
            }
        }
        set_tile_variant(op, best_tv, best_nar);
    }
    return misr_op_tile(op, tile_h, tile_w);
}

extern "C" misr_status misr_op_set_tile(misr_op *op, int variant) {
    if (!op) return set_error(MISR_E_INVAL, "op is NULL");
    if (op->general) return set_error(MISR_E_INVAL, "a general operator has no tiles");
    if (variant < 0 || variant > 2 || tile_hr(op->s, op->Lp | (variant << 8)) <= 0)
        return set_error(MISR_E_INVAL, "tile variant %d not compiled", variant);
    std::lock_guard<std::mutex> lk(op->mu);
    set_tile_variant(op, variant, false);
    return MISR_OK;
}

extern "C" misr_status misr_op_tile(const misr_op *op, int32_t *tile_h, int32_t *tile_w) {
    if (!op || !tile_h || !tile_w) return set_error(MISR_E_INVAL, "NULL argument");
    // the variant's shape, also while a small image runs the narrow tiles
    *tile_h = op->general ? 0 : tile_hr(op->s, op->kernel_key());
    *tile_w = op->general ? 0 : tile_wr(op->s, op->kernel_key());
    return MISR_OK;
}

extern "C" misr_status misr_op_tile_variant(const misr_op *op, int32_t *variant,
                                            int32_t *trial_w) {
    if (!op || !variant || !trial_w) return set_error(MISR_E_INVAL, "NULL argument");
    *variant = op->general ? -1 : op->tv;
    *trial_w = op->general ? 0 : tile_wt(op->s, op->kernel_key());
    return MISR_OK;
}
