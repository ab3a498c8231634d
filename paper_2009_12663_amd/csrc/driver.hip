// Full-history BFGS on a quadratic, resident on the GPU (Alg. 1 with every pair
// kept and B_0 fixed, the search direction of eq. (1)), and the synthetic Hessian
// it runs on.
//
// The paper obtains its pairs from elastic FWI; here the misfit is the quadratic
// 1/2 m^T A m - b^T m whose Hessian A stands in for the wave-equation Hessian:
//   A = diag(D) + P (x) (G_z (x) G_x),   P = I + c (1 1^T - I) over the parameter fields,
// with G_x, G_z the truncated Gaussian smoothers (weights exp(-t^2 / (2 sigma^2)),
// |t| <= half, normalised to sum 1, zero outside the grid), applied by a stencil.
//
// One iteration:  p = -B_k g (bfgs_apply_Hinv with one column; p = -g before the
// first pair when B_0 = gamma I), the exact line search alpha = -g^T p / p^T A p,
// s = alpha p, y = A s = alpha A p (formed from A p, not by differencing
// gradients), m += s, g += y, then (s, y) is pushed.  Dot products are fixed-order
// block reductions in float64, so a run is deterministic.
//
// What bounds an iteration on all but the largest models is the launches and the one wait
// for the pair's check, so the kernels between them are few: the smoothing (both passes
// through LDS), the coupling with both dot products, and one that takes the step, stores
// the pair and sums g^T g (q = -p is kept instead of p).  Nothing is allocated after the first
// direction: the apply's workspaces are sized for the handle's capacity.  30 iterations at
// n = 90,000, float64: 4.1 ms with 20 launches and two waits an iteration, 2.9 with 11 and one
// and two workspaces replaced for every pair, 2.3 now.
#include <cmath>
#include <new>
#include <type_traits>
#include <vector>

#include "common.h"

struct bfgsuq_gridop {
    int64_t nx = 0, nz = 0, n = 0;
    int32_t nparam = 0, half = 0;
    double coupling = 0.0;
    hipStream_t stream = nullptr;
    double* D = nullptr;       // n
    double* w = nullptr;       // 2 half + 1 normalised weights
    double* tmp = nullptr;     // 2 n (x pass, z pass)
};

namespace {

constexpr int kRedBlocks = 256;

int blocks_for(int64_t n) {
    const int64_t g = (n + 255) / 256;
    return (int)(g > 4096 ? 4096 : (g < 1 ? 1 : g));
}

template <typename T>
__global__ void stencil_x(int64_t nx, int64_t rows, int half, const double* __restrict__ w, const T* __restrict__ x,
                          double* __restrict__ out) {
    const int64_t total = rows * nx;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t ix = e % nx;
        const T* src = x + (e - ix);
        double s = 0.0;
        const int lo = (int)max((int64_t)-half, -ix), hi = (int)min((int64_t)half, nx - 1 - ix);
        for (int t = lo; t <= hi; ++t) s = fma(w[t + half], (double)src[ix + t], s);
        out[e] = s;
    }
}

__global__ void stencil_z(int64_t nx, int64_t nz, int64_t nparam, int half, const double* __restrict__ w,
                          const double* __restrict__ x, double* __restrict__ out) {
    const int64_t total = nparam * nz * nx;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t ix = e % nx, iz = (e / nx) % nz, p = e / (nx * nz);
        const double* src = x + p * nz * nx + ix;
        double s = 0.0;
        const int lo = (int)max((int64_t)-half, -iz), hi = (int)min((int64_t)half, nz - 1 - iz);
        for (int u = lo; u <= hi; ++u) s = fma(w[u + half], src[(iz + u) * nx], s);
        out[e] = s;
    }
}

// Both passes of the smoother on one field through LDS: a tile of 32 x 32 points with its
// half-width halo (zero outside the grid), four neighbouring outputs to a thread in the x
// pass and one in the z pass.  Sums run over the taps in order, as in stencil_x and
// stencil_z, which serve wider smoothers and thin grids (smooth_in_tiles).  A small grid's
// tiles are far fewer than the CUs, so a tile's own latency counts: 300 x 100 x 3 points,
// half 20: 9 us, 19 for the two stencils.
constexpr int SM_T = 32, SM_HALF = 20, SM_IN = SM_T + 2 * SM_HALF, SM_PITCH = SM_IN + 1;

template <typename T>
__global__ void __launch_bounds__(SM_T* SM_T) smooth_tile(int64_t nx, int64_t nz, int half,
                                                          const double* __restrict__ w, const T* __restrict__ x,
                                                          double* __restrict__ out) {
    __shared__ double in[SM_IN][SM_PITCH];
    __shared__ double xs[SM_IN][SM_T];
    __shared__ double ws[2 * SM_HALF + 1];
    const int64_t x0 = (int64_t)blockIdx.x * SM_T, z0 = (int64_t)blockIdx.y * SM_T;
    const T* src = x + (int64_t)blockIdx.z * nz * nx;
    const int ext = SM_T + 2 * half, taps = 2 * half + 1;
    if ((int)threadIdx.x < taps) ws[threadIdx.x] = w[threadIdx.x];
#pragma unroll
    for (int q = 0; q < (SM_IN * SM_IN + SM_T * SM_T - 1) / (SM_T * SM_T); ++q) {
        const int e = threadIdx.x + q * SM_T * SM_T, iz = e / ext, ix = e % ext;
        const int64_t gz = z0 + iz - half, gx = x0 + ix - half;
        const bool there = iz < ext && gz >= 0 && gz < nz && gx >= 0 && gx < nx;
        const double v = there ? (double)src[gz * nx + gx] : 0.0;
        if (iz < ext) in[iz][ix] = v;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < ext * (SM_T / 4); e += SM_T * SM_T) {
        const int iz = e / (SM_T / 4), o = e % (SM_T / 4) * 4;
        double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
        double a0 = in[iz][o], a1 = in[iz][o + 1], a2 = in[iz][o + 2];
#pragma unroll 8
        for (int t = 0; t < taps; ++t) {
            const double a3 = in[iz][o + 3 + t], wt = ws[t];
            s0 = fma(wt, a0, s0);
            s1 = fma(wt, a1, s1);
            s2 = fma(wt, a2, s2);
            s3 = fma(wt, a3, s3);
            a0 = a1;
            a1 = a2;
            a2 = a3;
        }
        xs[iz][o] = s0;
        xs[iz][o + 1] = s1;
        xs[iz][o + 2] = s2;
        xs[iz][o + 3] = s3;
    }
    __syncthreads();
    const int ix = threadIdx.x % SM_T, iz = threadIdx.x / SM_T;
    double sum = 0.0;
#pragma unroll 8
    for (int t = 0; t < taps; ++t) sum = fma(ws[t], xs[iz + t][ix], sum);
    if (x0 + ix < nx && z0 + iz < nz) out[(int64_t)blockIdx.z * nz * nx + (z0 + iz) * nx + x0 + ix] = sum;
}

// Whether the tiles are the faster smoother.  A tile costs the same however many of its
// points exist, the stencils only what exists, so the tiles have to be filled, the more so the
// fewer taps there are.  us in tiles | as stencils, half 20, 10, 5, 2, 0:
//   1700 x 350 x 3 (98 %)   48 | 156    35 | 93     28 | 60     26 | 40     25 | 26
//   111,562 x 16 (50 %)     73 | 115    48 | 78     37 | 52     33 | 34     30 | 24
//   65 x 65 x 400 (46 %)   294 | 355   265 | 295   254 | 262   249 | 244   243 | 235
//   74,375 x 8 x 3 (25 %)  139 | 104    88 | 67     65 | 50     56 | 36     48 | 26
//   1,785,000 x 1 (3 %)    929 | 91    538 | 58    373 | 40    306 | 30    248 | 25
// Up to 256 tiles run at once, one to a CU, and take 9 us where the two launches of the
// stencils take 10, full or not; two to a CU do so with fewer taps (384 of them with half 10:
// 9 us, 13 with half 20; 512 with half 5: 8).  A launch holds fewer than 2^32 threads along x,
// and 65535 blocks along y and z.
bool smooth_in_tiles(int64_t nx, int64_t nz, int32_t nparam, int32_t half) {
    const int64_t tx = (nx + SM_T - 1) / SM_T, tz = (nz + SM_T - 1) / SM_T;
    if (half > SM_HALF || nparam > 65535 || tz > 65535 || tx * SM_T * SM_T >= (int64_t)1 << 32) return false;
    if (tx * tz * nparam <= (half <= 5 ? 512 : half <= 10 ? 384 : 256)) return true;
    const double filled = (double)nx * nz / ((double)tx * tz * SM_T * SM_T);
    return filled >= (half < 2 ? 0.875 : half < 5 ? 0.45 : 0.35);
}

// Sum of v over a workgroup of 256, in thread 0.
__device__ __forceinline__ double block_sum256(double v, double* sh) {
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
        __syncthreads();
    }
    const double t = sh[0];
    __syncthreads();
    return t;
}

// y = D o x + (1 - c) g + c sum_q g_q, g the smoothed fields (coupling P applied per point).
// DOTS: also the workgroup's part of r^T x (dots[block]) and x^T y (dots[blocks + block]).
template <typename T, bool DOTS>
__global__ void __launch_bounds__(256) couple(int64_t npt, int nparam, double c, const double* __restrict__ D,
                                              const T* __restrict__ x, const double* __restrict__ g,
                                              double* __restrict__ y, const double* __restrict__ r,
                                              double* __restrict__ dots) {
    __shared__ double sh[256];
    double rx = 0.0, xy = 0.0;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < npt; e += (int64_t)gridDim.x * blockDim.x) {
        double sum = 0.0;
        for (int p = 0; p < nparam; ++p) sum += g[(int64_t)p * npt + e];
        for (int p = 0; p < nparam; ++p) {
            const int64_t i = (int64_t)p * npt + e;
            const double xe = (double)x[i];
            const double ye = fma(D[i], xe, fma(1.0 - c, g[i], c * sum));
            y[i] = ye;
            if (DOTS) {
                rx = fma(r[i], xe, rx);
                xy = fma(xe, ye, xy);
            }
        }
    }
    if (!DOTS) return;
    rx = block_sum256(rx, sh);
    xy = block_sum256(xy, sh);
    if (threadIdx.x == 0) {
        dots[blockIdx.x] = rx;
        dots[gridDim.x + blockIdx.x] = xy;
    }
}

// A fixed-order dot product's parts, one to a workgroup.
__global__ void dot_partial(int64_t n, const double* __restrict__ a, const double* __restrict__ b,
                            double* __restrict__ part) {
    __shared__ double sh[256];
    double s = 0.0;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
        s = fma(a[e], b[e], s);
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// The step from q = -p, Aq = A q and the parts of g^T q and q^T A q (couple): alpha =
// damping g^T q / q^T A q, s = -alpha q, y = -alpha A q, m += s, g += y; s and y go to the
// pair's columns in the storage type (one rounding), and gg[block] is the workgroup's part
// of the new g^T g.  Every workgroup sums the parts itself, in the same order.
template <typename T, typename Ts>
__global__ void __launch_bounds__(256) line_step(int64_t n, int nb, const double* __restrict__ dots, double damping,
                                                 const T* __restrict__ q, const double* __restrict__ Aq,
                                                 Ts* __restrict__ s, Ts* __restrict__ y, double* __restrict__ m,
                                                 double* __restrict__ g, double* __restrict__ gg) {
    __shared__ double sh[256];
    double gq = 0.0, qAq = 0.0;
    for (int b = threadIdx.x; b < nb; b += 256) {
        gq += dots[b];
        qAq += dots[nb + b];
    }
    gq = block_sum256(gq, sh);
    qAq = block_sum256(qAq, sh);
    const double alpha = damping * (gq / qAq);
    double sum = 0.0;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const double se = -alpha * (double)q[e], ye = -alpha * Aq[e];
        s[e] = from_f64<Ts>(se);
        y[e] = from_f64<Ts>(ye);
        m[e] += se;
        const double ge = g[e] + ye;
        g[e] = ge;
        sum = fma(ge, ge, sum);
    }
    sum = block_sum256(sum, sh);
    if (threadIdx.x == 0) gg[blockIdx.x] = sum;
}

// out[0] (host memory) = the sum of nb parts.
__global__ void __launch_bounds__(256) sum_to_host(int nb, const double* __restrict__ part, double* __restrict__ out) {
    __shared__ double sh[256];
    double t = 0.0;
    for (int b = threadIdx.x; b < nb; b += 256) t += part[b];
    t = block_sum256(t, sh);
    if (threadIdx.x == 0) out[0] = t;
}

__global__ void negate_to(int64_t n, const double* __restrict__ x, double* __restrict__ out) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
        out[e] = -x[e];
}

__global__ void to_f32(int64_t n, const double* __restrict__ x, float* __restrict__ out) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
        out[e] = (float)x[e];
}

// y = A x; with r also the workgroups' parts of r^T x and x^T y (kRedBlocks each in dots).
template <typename T>
int gridop_apply_impl(bfgsuq_gridop* op, const T* x, double* y, hipStream_t st, const double* r = nullptr,
                      double* dots = nullptr) {
    const int64_t n = op->n, npt = op->nx * op->nz;
    double* tz = op->tmp + n;
    if (smooth_in_tiles(op->nx, op->nz, op->nparam, op->half)) {
        hipLaunchKernelGGL(smooth_tile<T>, dim3((unsigned)ceil_div(op->nx, SM_T), ceil_div(op->nz, SM_T), op->nparam),
                           dim3(SM_T * SM_T), 0, st, op->nx, op->nz, op->half, op->w, x, tz);
    } else {
        double* tx = op->tmp;
        hipLaunchKernelGGL(stencil_x<T>, dim3(blocks_for(n)), dim3(256), 0, st, op->nx, op->nz * (int64_t)op->nparam,
                           op->half, op->w, x, tx);
        hipLaunchKernelGGL(stencil_z, dim3(blocks_for(n)), dim3(256), 0, st, op->nx, op->nz, (int64_t)op->nparam,
                           op->half, op->w, tx, tz);
    }
    if (r)
        hipLaunchKernelGGL((couple<T, true>), dim3(kRedBlocks), dim3(256), 0, st, npt, op->nparam, op->coupling, op->D,
                           x, tz, y, r, dots);
    else
        hipLaunchKernelGGL((couple<T, false>), dim3(blocks_for(npt)), dim3(256), 0, st, npt, op->nparam, op->coupling,
                           op->D, x, tz, y, nullptr, nullptr);
    return hipGetLastError() == hipSuccess ? BFGS_OK : BFGS_ERR_HIP;
}

}  // namespace

extern "C" {

int bfgs_gridop_destroy(bfgs_gridop_t op) {
    if (!op) return BFGS_OK;
    (void)hipStreamSynchronize(op->stream);
    if (op->D) (void)hipFree(op->D);
    if (op->w) (void)hipFree(op->w);
    if (op->tmp) (void)hipFree(op->tmp);
    delete op;
    return BFGS_OK;
}

int bfgs_gridop_create(int64_t nx, int64_t nz, int32_t nparam, const double* D, double sigma, int32_t half,
                       double coupling, void* stream, bfgs_gridop_t* out) {
    if (!out || !D || nx < 1 || nz < 1 || nparam < 1 || !(sigma > 0.0) || !std::isfinite(sigma) || half < 0 ||
        half > 4096 || !std::isfinite(coupling))
        return BFGS_ERR_ARG;
    *out = nullptr;
    bfgsuq_gridop* op = new (std::nothrow) bfgsuq_gridop();
    if (!op) return BFGS_ERR_ALLOC;
    op->nx = nx;
    op->nz = nz;
    op->nparam = nparam;
    op->n = nx * nz * (int64_t)nparam;
    op->half = half;
    op->coupling = coupling;
    op->stream = (hipStream_t)stream;
    std::vector<double> w(2 * half + 1);
    double sum = 0.0;
    for (int t = -half; t <= half; ++t) sum += (w[t + half] = std::exp(-0.5 * (t / sigma) * (t / sigma)));
    for (double& v : w) v /= sum;
    if (hipMalloc(&op->D, op->n * 8) != hipSuccess || hipMalloc(&op->w, w.size() * 8) != hipSuccess ||
        hipMalloc(&op->tmp, 2 * op->n * 8) != hipSuccess) {
        bfgs_gridop_destroy(op);
        return BFGS_ERR_ALLOC;
    }
    if (hipMemcpyAsync(op->D, D, op->n * 8, hipMemcpyDeviceToDevice, op->stream) != hipSuccess ||
        hipMemcpyAsync(op->w, w.data(), w.size() * 8, hipMemcpyHostToDevice, op->stream) != hipSuccess ||
        hipStreamSynchronize(op->stream) != hipSuccess) {
        bfgs_gridop_destroy(op);
        return BFGS_ERR_HIP;
    }
    *out = op;
    return BFGS_OK;
}

int bfgs_gridop_apply(bfgs_gridop_t op, const double* x, int32_t ncols, double* y) {
    if (!op || !x || !y || ncols < 1 || x == y) return BFGS_ERR_ARG;
    for (int j = 0; j < ncols; ++j) {
        const int rc = gridop_apply_impl(op, x + (int64_t)j * op->n, y + (int64_t)j * op->n, op->stream);
        if (rc != BFGS_OK) return rc;
    }
    return BFGS_OK;
}

int bfgs_minimize_quadratic(bfgs_t h, bfgs_gridop_t op, const double* b, int32_t max_iter, double rel_tol, double* m,
                            double* gnorm, int32_t* iters) {
    return bfgs_minimize_quadratic_ex(h, op, b, max_iter, rel_tol, 0, 1.0, m, gnorm, iters);
}

int bfgs_minimize_quadratic_ex(bfgs_t h, bfgs_gridop_t op, const double* b, int32_t max_iter, double rel_tol,
                               int32_t memory, double damping, double* m, double* gnorm, int32_t* iters) {
    if (!h || !op || !b || !m || !iters || max_iter < 0 || !(rel_tol >= 0.0) || op->n != h->n) return BFGS_ERR_ARG;
    if (memory < 0 || memory > h->kmax || !(damping > 0.0 && damping <= 1.0)) return BFGS_ERR_ARG;
    if (memory > 0 && h->streamed) return BFGS_ERR_STATE;   // the window moves in device memory
    if (h->storage == BFGS_BF16) return BFGS_ERR_ARG;   // a bfloat16 gradient cannot reach small tolerances
    if (h->k != 0) return BFGS_ERR_STATE;                // the run starts from m = 0 with an empty history
    if (op->stream != h->stream) return BFGS_ERR_ARG;
    *iters = 0;
    const int64_t n = h->n;
    hipStream_t st = h->stream;
    const bool f32 = h->storage == BFGS_F32;
    // g, q, Aq (float64), the float32 copies of g and q, a streamed history's pair, the
    // parts of the dot products
    void* ws = nullptr;
    const size_t pair_bytes = h->streamed ? 2 * (size_t)n * 8 : 0;
    const size_t bytes = (size_t)3 * n * 8 + pair_bytes + (f32 ? 2 * (size_t)n * 4 : 0) + 4 * kRedBlocks * 8;
    if (hipMalloc(&ws, bytes) != hipSuccess) return BFGS_ERR_ALLOC;
    double* g = (double*)ws;
    double* q = g + n;
    double* Aq = q + n;
    double* s64 = Aq + n;                 // a streamed history's s and y
    float* g32 = (float*)((char*)s64 + pair_bytes);
    float* q32 = g32 + n;
    double* dots = (double*)((char*)g32 + (f32 ? 2 * (size_t)n * 4 : 0));   // g^T q, q^T A q
    double* gg = dots + 2 * kRedBlocks;
    volatile double* gg_host = h->host_sc + 4;   // written by the device, read after a wait
    int rc = BFGS_OK;
    auto norm = [&](double* out) -> int {
        *out = std::sqrt(*gg_host);
        return std::isfinite(*out) ? BFGS_OK : BFGS_ERR_NONFINITE;
    };
    hipLaunchKernelGGL(negate_to, dim3(blocks_for(n)), dim3(256), 0, st, n, b, g);   // g_0 = A 0 - b
    hipLaunchKernelGGL(dot_partial, dim3(kRedBlocks), dim3(256), 0, st, n, g, g, gg);
    hipLaunchKernelGGL(sum_to_host, dim3(1), dim3(256), 0, st, kRedBlocks, gg, h->host_sc + 4);
    if (hipMemsetAsync(m, 0, n * 8, st) != hipSuccess || hipStreamSynchronize(st) != hipSuccess) rc = BFGS_ERR_HIP;
    double gn0 = 0.0;
    if (rc == BFGS_OK) rc = norm(&gn0);
    if (rc == BFGS_OK && gnorm) gnorm[0] = gn0;
    int it = 0;
    while (rc == BFGS_OK && it < max_iter && (memory > 0 || h->k < h->kmax)) {
        const bool first = h->k == 0 && h->gamma_mode;   // gamma unknown: p = -g
        if (first) {
            rc = gridop_apply_impl(op, g, Aq, st, g, dots);
        } else if (f32) {
            hipLaunchKernelGGL(to_f32, dim3(blocks_for(n)), dim3(256), 0, st, n, g, g32);
            if ((rc = apply_block(h, g32, 1, q32, false)) != BFGS_OK) break;
            rc = gridop_apply_impl(op, q32, Aq, st, g, dots);
        } else {
            if ((rc = apply_block(h, g, 1, q, false)) != BFGS_OK) break;
            rc = gridop_apply_impl(op, q, Aq, st, g, dots);
        }
        if (rc != BFGS_OK) break;
        // the limited-memory form keeps the last `memory` pairs
        if (memory > 0 && h->k == memory && (rc = pop_oldest(h)) != BFGS_OK) break;
        const int64_t col = (int64_t)h->k * h->ld;
        auto step = [&](const auto* dir, auto* s, auto* y) {
            typedef std::remove_cv_t<std::remove_pointer_t<decltype(dir)>> T;
            typedef std::remove_pointer_t<decltype(s)> Ts;
            hipLaunchKernelGGL((line_step<T, Ts>), dim3(kRedBlocks), dim3(256), 0, st, n, kRedBlocks, dots, damping, dir,
                               Aq, s, y, m, g, gg);
        };
        // a direction that is g itself is copied first: the step updates g
        if (first && hipMemcpyAsync(q, g, n * 8, hipMemcpyDeviceToDevice, st) != hipSuccess) rc = BFGS_ERR_HIP;
        if (rc != BFGS_OK) break;
        if (h->streamed) {
            if (f32 && !first) step(q32, s64, s64 + n);
            else step(q, s64, s64 + n);
        } else if (f32) {
            float *S = (float*)h->S + col, *Y = (float*)h->Y + col;
            if (first) step(q, S, Y);
            else step(q32, S, Y);
        } else {
            step(q, (double*)h->S + col, (double*)h->Y + col);
        }
        hipLaunchKernelGGL(sum_to_host, dim3(1), dim3(256), 0, st, kRedBlocks, gg, h->host_sc + 4);
        if (hipGetLastError() != hipSuccess) {
            rc = BFGS_ERR_HIP;
            break;
        }
        rc = h->streamed ? push_enqueue(h, s64, s64 + n, BFGS_F64) : push_stored(h);
        if (rc == BFGS_OK) rc = push_finish(h);   // waits
        if (rc != BFGS_OK) break;
        ++it;
        double gn = 0.0;
        if ((rc = norm(&gn)) != BFGS_OK) break;
        if (gnorm) gnorm[it] = gn;
        if (gn <= rel_tol * gn0) break;
    }
    *iters = it;
    (void)hipStreamSynchronize(st);
    (void)hipFree(ws);
    return rc;
}

}  // extern "C"
