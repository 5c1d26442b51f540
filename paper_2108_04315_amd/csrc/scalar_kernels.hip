// scalar_kernels.hip -- the device-resident SCG state machine (Moller's
// scalar steps in FP64), small helper kernels, and the dispatch from a
// geometry's (scale, band length) to the image-kernel instances.
#include <hip/hip_runtime.h>

#include "device_common.h"
#include "pass_end.h"
#include "runtime.h"

namespace misr {

// ------------------------------------------------------------ scalar kernel
// The SCG steps after a pass of the general operators' solves, one workgroup
// per solve (banded operators run them at the end of the pass, pass_end.h);
// solves with apart >= least.
__global__ void __launch_bounds__(kEndRows) k_scalar(const SolveRef *refs, int pass,
                                                     int least) {
    __shared__ double red[kNV * (kEndRows / 64)];
    const AS4 SolveRef *rp = cst(refs) + blockIdx.x;
    if (rp->apart < least) return;
    sum_rows<5>(glb((const double *)(pass == 2 ? rp->part_u : rp->part)),
                pass == 2 ? rp->nitemsu : rp->nitems, red, [](const AS1 double *a) { return *a; });
    __syncthreads();
    if (threadIdx.x == 0) scg_steps<5>(rp, red, pass, false);
}

// Sums one solve's partials into out[0..3) = {J, E_data, E_reg} (cost only).
__global__ void __launch_bounds__(kNT) k_cost_out(const double *__restrict__ partials,
                                                  int nitems, double *out) {
    __shared__ double red[kNV * (kNT / 64)];
    __shared__ double tot[kNV];
    double v[kNV] = {0, 0, 0, 0, 0, 0};
    for (int i = threadIdx.x; i < nitems; i += kNT)
#pragma unroll
        for (int q = 0; q < kNV; ++q) v[q] += partials[(long long)i * kNV + q];
    block_sum_store<kNV, kNT>(v, tot, red);
    if (threadIdx.x == 0) {
        out[0] = tot[0] + tot[1];
        out[1] = tot[0];
        out[2] = tot[1];
    }
}

// ----------------------------------------------------------- small kernels
// Short plan arrays (views, states) travel with the launch: one kernel in
// stream order instead of a staged copy from pageable memory per array.
__global__ void __launch_bounds__(64) k_put(PutArgs a) {
    int at = 0;
    for (int i = 0; i < a.n; ++i) {
        for (int q = threadIdx.x; q < a.words[i]; q += 64) a.dst[i][q] = a.w[at + q];
        at += a.words[i];
    }
}

__global__ void __launch_bounds__(64) k_copy_state(ScgState *dst, const ScgState *src) {
    static_assert(sizeof(ScgState) % 8 == 0 && sizeof(ScgState) <= 512, "one wave copies a state");
    if (threadIdx.x < sizeof(ScgState) / 8)
        reinterpret_cast<unsigned long long *>(dst)[threadIdx.x] =
            reinterpret_cast<const unsigned long long *>(src)[threadIdx.x];
}

__global__ void k_fill_f32(float *p, long long n, float v) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        p[i] = v;
}

// Copies x[1] into x[0] for every view whose current iterate sits in the
// workspace buffer (decided on the device).
__global__ void k_finalize(const Proj *__restrict__ projs, int nproj, int stype) {
    for (int j = 0; j < nproj; ++j) {
        const Proj &P = projs[j];
        if (P.st->xc == 0) continue;
        const long long n = (long long)P.Hb * P.ld;
        const int es = (stype == ST_F32) ? 4 : 2;
        if (es == 4) {
            const float *a = (const float *)P.x[1];
            float *b = (float *)P.x[0];
            for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
                 i += (long long)gridDim.x * blockDim.x)
                b[i] = a[i];
        } else {
            const unsigned short *a = (const unsigned short *)P.x[1];
            unsigned short *b = (unsigned short *)P.x[0];
            for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
                 i += (long long)gridDim.x * blockDim.x)
                b[i] = a[i];
        }
    }
}

// ---------------------------------------------------- tiled-solve helpers
// Halo exchange: each copy moves a rectangle of the gradient g[cur] from the
// view that owns it into another view's halo.  It runs after the SCG steps that
// end a trial pass: an accepted trial's gradient is g[cur] by then; after a
// rejection the copy repeats values that are already there.  A copy between two
// neighbours is a strip as long as the view (2048 x 16 HR px at 1024^2-LR tiles
// with a halo of 8) and moves few bytes per launch, so the launch is bound by
// how many loads are in flight: kHaloPx pixels of a rectangle per workgroup
// (blockIdx.y), every load before the first store.
// One workgroup per copy took 74.8 us on four such tiles; this takes 8.1.
constexpr int kHaloPx = 2048;   // pixels per workgroup
__global__ void __launch_bounds__(256) k_halo(const Proj *__restrict__ projs,
                                              const HaloCopy *__restrict__ copies,
                                              const int *n_copies) {
    const int n = *n_copies;
    for (int c = blockIdx.x; c < n; c += gridDim.x) {
        const HaloCopy hc = copies[c];
        const Proj &A = projs[hc.src];
        const Proj &B = projs[hc.dst];
        const int g = A.st->cur;
        const long long lda = A.ld, ldb = B.ld;
        const float *__restrict__ src =
            A.g[g] + (long long)(hc.gy - A.gy0) * lda + hc.gx - A.gx0;
        float *__restrict__ dst = B.g[g] + (long long)(hc.gy - B.gy0) * ldb + hc.gx - B.gx0;
        const unsigned px = (unsigned)hc.rows * (unsigned)hc.cols;   // < 2^31, as the image
        for (unsigned q0 = blockIdx.y * kHaloPx; q0 < px; q0 += gridDim.y * kHaloPx) {
            float v[kHaloPx / 256];
            long long at[kHaloPx / 256];
#pragma unroll
            for (int e = 0; e < kHaloPx / 256; ++e) {
                const unsigned q = q0 + e * 256 + threadIdx.x;
                const unsigned r = q / (unsigned)hc.cols, cc = q - r * (unsigned)hc.cols;
                at[e] = q < px ? r * ldb + cc : -1;
                if (q < px) v[e] = src[r * lda + cc];
            }
#pragma unroll
            for (int e = 0; e < kHaloPx / 256; ++e)
                if (at[e] >= 0) dst[at[e]] = v[e];
        }
    }
}

// Element conversions between the storage types (round to nearest even
// into 16-bit; widening is exact).
__device__ __forceinline__ float ld_any(const void *b, long long i, int t) {
    if (t == ST_F32) return ((const float *)b)[i];
    if (t == ST_BF16) return __uint_as_float((unsigned)((const unsigned short *)b)[i] << 16);
    return (float)((const _Float16 *)b)[i];
}
__device__ __forceinline__ void st_any(void *b, long long i, int t, float v) {
    if (t == ST_F32) {
        ((float *)b)[i] = v;
    } else if (t == ST_BF16) {
        unsigned u = __float_as_uint(v);
        if ((u & 0x7fffffffu) > 0x7f800000u) {
            u = 0x7fc00000u;
        } else {
            u += 0x7fffu + ((u >> 16) & 1u);
        }
        ((unsigned short *)b)[i] = (unsigned short)(u >> 16);
    } else {
        ((_Float16 *)b)[i] = (_Float16)v;
    }
}

// Both copies below go by rows (blockIdx.x strides them), a thread's kRowE
// elements of a row in flight together; bound by memory.
constexpr int kRowE = 4;
template <class F>
__device__ __forceinline__ void row_elements(int n, F f) {
    for (int c0 = threadIdx.x; c0 < n; c0 += kRowE * 256) f(c0);
}

// Whole-image x (the solve's xglob, storage gt) into every view's x[0]
// (storage vt), halo included; p[0] cleared so that the first update starts
// from a zero direction.
__global__ void k_scatter(const Proj *__restrict__ projs, int nproj, int vt, int gt) {
    for (int j = blockIdx.y; j < nproj; j += gridDim.y) {
        const Proj &P = projs[j];
        const ScgState &st = *P.st;
        const int Wb = P.Wb;
        void *xo = P.x[0];
        float *po = P.p[0];
        const void *xg = st.xglob;
        for (int r = blockIdx.x; r < P.Hb; r += gridDim.x) {
            const long long src = (long long)(P.gy0 + r) * st.ldg + P.gx0;
            const long long dst = (long long)r * P.ld;
            row_elements(Wb, [&](int c0) {
                float v[kRowE];
#pragma unroll
                for (int e = 0; e < kRowE; ++e)
                    v[e] = ld_any(xg, src + min(c0 + 256 * e, Wb - 1), gt);
#pragma unroll
                for (int e = 0; e < kRowE; ++e)
                    if (c0 + 256 * e < Wb) {
                        st_any(xo, dst + c0 + 256 * e, vt, v[e]);
                        po[dst + c0 + 256 * e] = 0.f;
                    }
            });
        }
    }
}

// Owned part of every view's current x (which = 0; storage vt, written as
// gt) or trial gradient g[cur^1] (which = 1; FP32) back into the whole-image
// buffer.
__global__ void k_gather(const Proj *__restrict__ projs, int nproj, int vt, int gt, int which) {
    for (int j = blockIdx.y; j < nproj; j += gridDim.y) {
        const Proj &P = projs[j];
        const ScgState &st = *P.st;
        const int oh = P.oy1 - P.oy0, ow = P.ox1 - P.ox0;
        const void *srcb = which ? (const void *)P.g[st.cur ^ 1] : P.x[st.xc];
        void *dstb = which ? (void *)st.gglob : st.xglob;
        const int ts = which ? (int)ST_F32 : vt, td = which ? (int)ST_F32 : gt;
        for (int r = P.oy0 + blockIdx.x; r < P.oy0 + oh; r += gridDim.x) {
            const long long src = (long long)r * P.ld + P.ox0;
            const long long dst = (long long)(P.gy0 + r) * st.ldg + P.gx0 + P.ox0;
            row_elements(ow, [&](int c0) {
                float v[kRowE];
#pragma unroll
                for (int e = 0; e < kRowE; ++e)
                    v[e] = ld_any(srcb, src + min(c0 + 256 * e, ow - 1), ts);
#pragma unroll
                for (int e = 0; e < kRowE; ++e)
                    if (c0 + 256 * e < ow) st_any(dstb, dst + c0 + 256 * e, td, v[e]);
            });
        }
    }
}

// ------------------------------------------------------- start points
// Multi-image interpolation: frame k's pixel (i, j) lands on HR
// (s i + ty_k, s j + tx_k); mean of the samples landing on a pixel, in frame
// order; frame 0's covering pixel where none lands.
__global__ void k_interpolate(InitArgs a, const void *y, void *x, int st) {
    const int h = a.H / a.s, w = a.W / a.s;
    const long long n = (long long)a.H * a.W;
    for (long long q = blockIdx.x * (long long)blockDim.x + threadIdx.x; q < n;
         q += (long long)gridDim.x * blockDim.x) {
        const int u = (int)(q / a.W), v = (int)(q - (long long)u * a.W);
        float acc = 0.f;
        int cnt = 0;
        for (int k = 0; k < a.K; ++k) {
            const int r = u - a.ty[k], c = v - a.tx[k];
            if (r < 0 || c < 0 || r % a.s != 0 || c % a.s != 0) continue;
            const int i = r / a.s, j = c / a.s;
            if (i >= h || j >= w) continue;
            acc += ld_any(y, ((long long)k * h + i) * w + j, st);
            ++cnt;
        }
        st_any(x, q, st, cnt ? acc / (float)cnt : ld_any(y, (long long)(u / a.s) * w + v / a.s, st));
    }
}

// Keys cubic convolution weight (a = -1/2).
__device__ __forceinline__ float keys_w(float t) {
    t = fabsf(t);
    if (t <= 1.f) return (1.5f * t - 2.5f) * t * t + 1.f;
    if (t < 2.f) return ((-0.5f * t + 2.5f) * t - 4.f) * t + 2.f;
    return 0.f;
}

// Bicubic upsampling of frame 0: HR pixel u at LR coordinate (u + 1/2)/s - 1/2,
// 4 x 4 taps clamped to the frame.
__global__ void k_upsample(InitArgs a, const void *y, void *x, int st) {
    const int h = a.H / a.s, w = a.W / a.s;
    const long long n = (long long)a.H * a.W;
    for (long long q = blockIdx.x * (long long)blockDim.x + threadIdx.x; q < n;
         q += (long long)gridDim.x * blockDim.x) {
        const int u = (int)(q / a.W), v = (int)(q - (long long)u * a.W);
        const double cy = (u + 0.5) / a.s - 0.5, cx = (v + 0.5) / a.s - 0.5;
        const int iy = (int)floor(cy), ix = (int)floor(cx);
        const float fy = (float)(cy - iy), fx = (float)(cx - ix);
        float wy[4], wx[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            wy[t] = keys_w(fy - (t - 1));
            wx[t] = keys_w(fx - (t - 1));
        }
        float acc = 0.f;
#pragma unroll
        for (int ta = 0; ta < 4; ++ta) {
            const int i = min(max(iy + ta - 1, 0), h - 1);
            float row = 0.f;
#pragma unroll
            for (int tb = 0; tb < 4; ++tb) {
                const int j = min(max(ix + tb - 1, 0), w - 1);
                row = fmaf(wx[tb], ld_any(y, (long long)i * w + j, st), row);
            }
            acc = fmaf(wy[ta], row, acc);
        }
        st_any(x, q, st, acc);
    }
}

// ------------------------------------------------------------- dispatching
#define MISR_SCALES(X) X(1) X(2) X(3) X(4)
#define X(s)                                                                                   \
    int tile_dims_s##s(int Lp, int *th, int *tw);                                              \
    int tile_dims_trial_s##s(int Lp, int *th, int *tw);                                        \
    hipError_t launch_trial_s##s(int Lp, int stype, int grid, hipStream_t st, const Proj *projs, \
                                 const Item *items, const int *n_items, double *partials,      \
                                 int mode);                                                    \
    hipError_t launch_upcurv_s##s(int Lp, int stype, int grid, hipStream_t st,                 \
                                  const Proj *projs, const Item *items, const int *n_items,    \
                                  double *partials);                                           \
    hipError_t launch_forward_s##s(int Lp, int stype, int grid, hipStream_t st,                \
                                   const Proj *projs, const Item *items, int n, const void *x,  \
                                   void *y);                                                   \
    hipError_t launch_adjoint_s##s(int Lp, int stype, int grid, hipStream_t st,                \
                                   const Proj *projs, const Item *items, int n, const void *r, \
                                   float *x);
MISR_SCALES(X)
#undef X

// Band lengths instantiated per scale; an operator's L is rounded up to one.
static const int kBands[5][6] = {{0}, {4, 8, 16, 0}, {6, 8, 9, 12, 16, 0},
                                 {6, 9, 10, 12, 16, 0}, {12, 16, 0}};

int padded_band(int S, int L) {
    if (S < 1 || S > 4) return -1;
    for (int i = 0; kBands[S][i]; ++i)
        if (kBands[S][i] >= L) return kBands[S][i];
    return -1;
}

static int tile_dims(int S, int Lp, int *th, int *tw) {
    switch (S) {
    case 1: return tile_dims_s1(Lp, th, tw);
    case 2: return tile_dims_s2(Lp, th, tw);
    case 3: return tile_dims_s3(Lp, th, tw);
    case 4: return tile_dims_s4(Lp, th, tw);
    }
    return 0;
}

int tile_hr(int S, int Lp) {
    int th = -1, tw = -1;
    return tile_dims(S, Lp, &th, &tw) ? th : -1;
}

int tile_wr(int S, int Lp) {
    int th = -1, tw = -1;
    return tile_dims(S, Lp, &th, &tw) ? tw : -1;
}

int tile_wt(int S, int key) {
    int th = -1, tw = -1, ok = 0;
    switch (S) {
    case 1: ok = tile_dims_trial_s1(key, &th, &tw); break;
    case 2: ok = tile_dims_trial_s2(key, &th, &tw); break;
    case 3: ok = tile_dims_trial_s3(key, &th, &tw); break;
    case 4: ok = tile_dims_trial_s4(key, &th, &tw); break;
    }
    return ok ? tw : -1;
}

hipError_t launch_image(int S, int Lp, int grid, hipStream_t stream, const Proj *projs,
                        const Item *items, const int *n_items, double *partials, int kind,
                        int stype) {
#define X(s)                                                                                  \
    if (S == s)                                                                               \
        return kind == 2 ? launch_upcurv_s##s(Lp, stype, grid, stream, projs, items, n_items, \
                                              partials)                                       \
                         : launch_trial_s##s(Lp, stype, grid, stream, projs, items, n_items,  \
                                             partials, kind);
    MISR_SCALES(X)
#undef X
    return hipErrorInvalidValue;
}

hipError_t launch_forward(int S, int Lp, int grid, hipStream_t stream, const Proj *projs,
                          const Item *items, int n, int stype, const void *x, void *y) {
#define X(s) \
    if (S == s) return launch_forward_s##s(Lp, stype, grid, stream, projs, items, n, x, y);
    MISR_SCALES(X)
#undef X
    return hipErrorInvalidValue;
}

hipError_t launch_adjoint(int S, int Lp, int grid, hipStream_t stream, const Proj *projs,
                          const Item *items, int n, int stype, const void *r, float *x) {
#define X(s) \
    if (S == s) return launch_adjoint_s##s(Lp, stype, grid, stream, projs, items, n, r, x);
    MISR_SCALES(X)
#undef X
    return hipErrorInvalidValue;
}

hipError_t launch_scalar(int grid, hipStream_t stream, const SolveRef *refs, int pass,
                         int least) {
    hipLaunchKernelGGL(k_scalar, dim3(grid), dim3(kEndRows), 0, stream, refs, pass, least);
    return hipGetLastError();
}

hipError_t launch_halo(hipStream_t stream, const Proj *projs, const HaloCopy *copies,
                       const int *n_copies, int grid) {
    if (grid <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_halo, dim3(grid, 32), dim3(256), 0, stream, projs, copies, n_copies);
    return hipGetLastError();
}

// Workgroups of the view copies: enough of them to fill the device also where
// there is one view.  One 6144^2 view in half precision, with 256 workgroups
// and an element at a time: scatter 350 us, gather 415; now 77 and 81.
static dim3 view_grid(int nproj) {
    return dim3(nproj < 8 ? 2048 : 256, nproj < 65535 ? nproj : 65535);
}

hipError_t launch_scatter(hipStream_t stream, const Proj *projs, int nproj, int vt, int gt) {
    hipLaunchKernelGGL(k_scatter, view_grid(nproj), dim3(256), 0, stream, projs, nproj, vt, gt);
    return hipGetLastError();
}

hipError_t launch_gather(hipStream_t stream, const Proj *projs, int nproj, int vt, int gt,
                         int which) {
    hipLaunchKernelGGL(k_gather, view_grid(nproj), dim3(256), 0, stream, projs, nproj, vt, gt,
                       which);
    return hipGetLastError();
}

hipError_t launch_cost_out(hipStream_t stream, const double *partials, int nitems,
                           double *out) {
    hipLaunchKernelGGL(k_cost_out, dim3(1), dim3(kNT), 0, stream, partials, nitems, out);
    return hipGetLastError();
}

hipError_t launch_fill(hipStream_t stream, float *p, long long n, float v) {
    if (n <= 0) return hipSuccess;
    long long blocks = (n + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(k_fill_f32, dim3((unsigned)blocks), dim3(256), 0, stream, p, n, v);
    return hipGetLastError();
}

hipError_t launch_init(hipStream_t stream, int kind, const InitArgs &a, const void *y, void *x,
                       int st) {
    const long long n = (long long)a.H * a.W;
    long long blocks = (n + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    if (kind == 1)
        hipLaunchKernelGGL(k_upsample, dim3((unsigned)blocks), dim3(256), 0, stream, a, y, x, st);
    else
        hipLaunchKernelGGL(k_interpolate, dim3((unsigned)blocks), dim3(256), 0, stream, a, y, x,
                           st);
    return hipGetLastError();
}

hipError_t launch_put(hipStream_t stream, const PutArgs &a) {
    hipLaunchKernelGGL(k_put, dim3(1), dim3(64), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_copy_state(hipStream_t stream, ScgState *dst, const ScgState *src) {
    hipLaunchKernelGGL(k_copy_state, dim3(1), dim3(64), 0, stream, dst, src);
    return hipGetLastError();
}

hipError_t launch_finalize(hipStream_t stream, const Proj *projs, int nproj, int stype) {
    hipLaunchKernelGGL(k_finalize, dim3(1024), dim3(256), 0, stream, projs, nproj, stype);
    return hipGetLastError();
}

}  // namespace misr
