// B_k V for a block of ncols vectors through the compact form of the inverse
// BFGS matrix (Byrd, Nocedal & Schnabel 1994), which reaches the eq. (3)
// recursion / Alg. 2 two-loop result with two streaming passes over S and Y
// instead of 2k sequential ones:
//
//   B_k = B_0 + [S  B_0 Y] [ R^-T (D + Y^T B_0 Y) R^-1   -R^-T ] [ S^T     ]
//                          [ -R^-1                        0    ] [ Y^T B_0 ]
//   with R = triu(S^T Y), D = diag(S^T Y).
//
// Pass 1 (gemm1):  Z = [S^T V ; Y^T (h0 o V)]          2k x c, float64 partials
// reduce:          fixed-order sum of the partials
// small solve:     P = R^-1 Z_s,  T = R^-T ((D + Y^T B_0 Y) P - Z_y)     (float64)
// Pass 2 (gemm2):  out = h0 o (V - Y P) + S T     (or - h0 o (Y P) + S T for B_k - B_0)
//
// This file holds the float64 matrix-core form of both passes (float32 and
// float64 storage, and bfloat16 where its own MFMA form in apply_mfma.hip does not
// apply) and the inner solve shared by all forms.
#include <cmath>

#include <algorithm>
#include <type_traits>
#include <vector>

#include "stream_f64.h"

namespace {

// What the sum belongs to, so that a trace tells the two apart.
struct ApplySum;
struct ProjectionSum;

template <typename Use>
__global__ void __launch_bounds__(SUM_THREADS) reduce_partials(int64_t count, int nchunks,
                                                               const double* __restrict__ part,
                                                               double* __restrict__ Z) {
    __shared__ double sh[SUM_DEPTH][SUM_ENTRIES];
    const int64_t e = blockIdx.x * (int64_t)SUM_ENTRIES + threadIdx.x % SUM_ENTRIES;
    const bool live = e < count;
    const double t = ordered_sum(
        0, nchunks, sh, [&](int ch) { return live ? part[(int64_t)ch * count + e] : 0.0; },
        [](double sum, double v, int) { return sum + v; });
    if (threadIdx.x < SUM_ENTRIES && e < count) Z[e] = t;
}

// Where a small solve writes column j of P and T: column-major k x c each, or the packed
// [T ; -P] that the float64 pass 2 reads (with the zero rows that fill its last step), or the
// two bfloat16 halves of [-P ; T] that the bfloat16 pass 2 reads.
struct SolveOut {
    double *P, *T, *M;
    int k, cblocks;
    uint16_t *hi, *lo;   // column j from j * 2 * rows: -P, then T, each k entries and zeros up to rows
    int rows;
    __device__ __forceinline__ void put_halves(int q, int j, double v) const {
        const bf16_t h = float_to_bf16((float)v);
        hi[(int64_t)j * 2 * rows + q] = h.bits;
        lo[(int64_t)j * 2 * rows + q] = float_to_bf16((float)(v - (double)bf16_to_float(h))).bits;
    }
    __device__ __forceinline__ void put(int i, int j, double pv, double tv) const {
        if (M) {
            M[nn_pack_index(i, j, cblocks)] = tv;
            M[nn_pack_index(k + i, j, cblocks)] = -pv;
            if (i == 0)
                for (int q = 2 * k; q % 4; ++q) M[nn_pack_index(q, j, cblocks)] = 0.0;
        } else if (hi) {
            put_halves(i, j, -pv);
            put_halves(rows + i, j, tv);
        } else {
            P[(int64_t)j * k + i] = pv;
            T[(int64_t)j * k + i] = tv;
        }
    }
    // The zeros of the halves of column j, fewer than 32, by as many of the calling threads.
    __device__ __forceinline__ void pad(int i, int j) const {
        const int q = k + i;
        if (!hi || q >= rows) return;
        put_halves(q, j, 0.0);
        put_halves(rows + q, j, 0.0);
    }
};

// One 64-lane wave per probe column j.
//   P = R^-1 Z_s               (column-oriented back substitution)
//   W = (D + YHY) P - Z_y
//   T = R^-T W                 (row-oriented forward substitution)
// Rm is column-major with leading dimension kmax: R(l, i) = Rm[i * kmax + l].
constexpr int SOLVE_MAXK_PER_LANE = BFGS_MAX_PAIRS / 64;

__global__ void __launch_bounds__(64) small_solve(int k, int kmax, int c, const double* __restrict__ Rm,
                                                  const double* __restrict__ YHY, const double* __restrict__ Z,
                                                  SolveOut out, int32_t* __restrict__ status) {
    extern __shared__ double sh[];
    double* b = sh;          // right-hand side, overwritten
    double* x = sh + k;      // P column
    double* w = sh + 2 * k;  // W, then T column
    const int j = blockIdx.x, lane = threadIdx.x;
    const double* zs = Z + (int64_t)j * 2 * k;
    const double* zy = zs + k;
    for (int i = lane; i < k; i += 64) b[i] = zs[i];
    __syncthreads();
    for (int i = k - 1; i >= 0; --i) {
        const double xi = b[i] / Rm[(int64_t)i * kmax + i];
        __syncthreads();
        if (lane == 0) x[i] = xi;
        for (int l = lane; l < i; l += 64) b[l] -= Rm[(int64_t)i * kmax + l] * xi;
        __syncthreads();
    }
    double acc[SOLVE_MAXK_PER_LANE];
#pragma unroll
    for (int u = 0; u < SOLVE_MAXK_PER_LANE; ++u) acc[u] = 0.0;
    for (int m = 0; m < k; ++m) {
        const double xm = x[m];
        const double* col = YHY + (int64_t)m * kmax;
#pragma unroll
        for (int u = 0; u < SOLVE_MAXK_PER_LANE; ++u) {
            const int l = lane + 64 * u;
            if (l < k) acc[u] = fma(col[l], xm, acc[u]);
        }
    }
#pragma unroll
    for (int u = 0; u < SOLVE_MAXK_PER_LANE; ++u) {
        const int l = lane + 64 * u;
        if (l < k) w[l] = acc[u] + Rm[(int64_t)l * kmax + l] * x[l] - zy[l];
    }
    __syncthreads();
    for (int i = 0; i < k; ++i) {
        const double* col = Rm + (int64_t)i * kmax;
        double s = 0.0;
        for (int l = lane; l < i; l += 64) s = fma(col[l], w[l], s);
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
        const double ti = (w[i] - s) / col[i];
        __syncthreads();
        if (lane == 0) w[i] = ti;
        __syncthreads();
    }
    bool bad = false;
    for (int i = lane; i < k; i += 64) {
        const double pv = x[i], tv = w[i];
        out.put(i, j, pv, tv);
        bad |= !isfinite(pv) || !isfinite(tv);
    }
    if (bad) set_status(status, BFGS_ERR_NONFINITE);
}

// Same solve through the stored R^-1, for k <= 256: one workgroup per probe column, one
// thread per pair index.
//   P = R^-1 Z_s;  W = (D + YHY) P - Z_y;  T = R^-T W
// A result is one chain of sums over the pairs, in order, SOLVE_DEPTH matrix entries of it
// fetched while as many are added; the lanes of a wave walk the same pair, so that they come
// as whole lines.  What bounds it is the instructions of one wave and fetching them: so a
// pair is a load, its address (32 bits from the matrix's start, a column further and not past
// the last) and a product, and little else: R^-1 and its transpose hold zeros outside their
// triangles, x is padded with zeros, and the three chains go through one copy of the code.
// One to 71 columns take 3.3 us at k = 5, 6.8 at 61, 9.8 at 100 and 13.7 at 150; with scalar
// addresses, a select at each pair and three copies 4.4, 9.5, 15 and 21.  (More entries in
// flight lose: 32 fetched ahead, 48.)
constexpr int SOLVE_DEPTH = 16;

struct SolveLds {
    alignas(16) double x[256 + SOLVE_DEPTH];
};

// acc + sum of A(i, l) x[l] over l in [lo, hi) in order; A column-major, lo and hi the same in
// a whole wave; x is zero from hi on to the end of the last batch.
__device__ __forceinline__ double solve_chain(double acc, const double* __restrict__ A, int kmax, int i, int lo, int hi,
                                              const double* x) {
    double b0[SOLVE_DEPTH], b1[SOLVE_DEPTH];
    const unsigned step = (unsigned)kmax * 8, last = (unsigned)(hi - 1) * step + (unsigned)i * 8;
    unsigned at = (unsigned)lo * step + (unsigned)i * 8;   // of the next entry to fetch, in bytes; at most 8 MB
    auto fetch = [&](double (&b)[SOLVE_DEPTH]) {           // past hi the last entry again
#pragma unroll
        for (int u = 0; u < SOLVE_DEPTH; ++u) {
            b[u] = *(const double*)((const char*)A + at);
            at = min(at + step, last);
        }
    };
    auto sum = [&](const double (&b)[SOLVE_DEPTH], int l0) {
        double xv[SOLVE_DEPTH];
#pragma unroll
        for (int u = 0; u < SOLVE_DEPTH; ++u) xv[u] = x[l0 + u];
        __builtin_amdgcn_sched_barrier(0);   // all fetched before the first is added
#pragma unroll
        for (int u = 0; u < SOLVE_DEPTH; ++u) acc = fma(b[u], xv[u], acc);
    };
    fetch(b0);
#pragma unroll 1
    for (int l0 = lo; l0 < hi; l0 += 2 * SOLVE_DEPTH) {
        fetch(b1);
        sum(b0, l0);
        if (l0 + SOLVE_DEPTH >= hi) break;
        fetch(b0);
        sum(b1, l0 + SOLVE_DEPTH);
    }
    return acc;
}

__device__ __forceinline__ void small_solve_block(SolveLds& s, int k, int kmax, const double* __restrict__ Rm,
                                                  const double* __restrict__ Rinv, const double* __restrict__ RinvT,
                                                  const double* __restrict__ YHY, const double* __restrict__ Z,
                                                  SolveOut out, int32_t* __restrict__ status, int j) {
    const int i = threadIdx.x;
    const bool live = i < k;
    const int ic = min(i, k - 1);
    const int w0 = __builtin_amdgcn_readfirstlane(i / 64 * 64);   // this wave's rows: w0 .. w1 - 1
    const int w1 = min(k, w0 + 64);
    const double zs = live ? Z[(int64_t)j * 2 * k + i] : 0.0, zy = live ? Z[(int64_t)j * 2 * k + k + i] : 0.0;
    const double dii = Rm[(int64_t)ic * kmax + ic];
    double v = zs, pv = 0.0;
#pragma unroll 1
    for (int step = 0; step < 3; ++step) {
        __syncthreads();
        s.x[i] = live ? v : 0.0;
        __syncthreads();
        const double* A = step == 0 ? Rinv : step == 1 ? YHY : RinvT;
        const int lo = step == 0 ? w0 : 0, hi = step == 2 ? w1 : k;
        const double first = step == 1 ? dii * v - zy : 0.0;
        v = w0 < k ? solve_chain(first, A, kmax, ic, lo, hi, s.x) : 0.0;
        if (step == 0) pv = v;
    }
    out.pad(i, j);
    if (live) {
        out.put(i, j, pv, v);
        if (!isfinite(pv) || !isfinite(v)) set_status(status, BFGS_ERR_NONFINITE);
    }
}

__global__ void __launch_bounds__(256) small_solve_blocks(int k, int kmax, const double* __restrict__ Rm,
                                                          const double* __restrict__ Rinv,
                                                          const double* __restrict__ RinvT,
                                                          const double* __restrict__ YHY,
                                                          const double* __restrict__ Z, SolveOut out,
                                                          int32_t* __restrict__ status) {
    __shared__ SolveLds lds;
    small_solve_block(lds, k, kmax, Rm, Rinv, RinvT, YHY, Z, out, status, blockIdx.x);
}

// The solve of a few columns and pairs: as above, with each sum dealt to FEW_SEGS waves
// (contiguous quarters of the pairs, each padded in x) and added through LDS in a fixed order,
// since with the chip otherwise idle the length of a chain is all that counts: one column at
// k = 61 takes 4.1 us, 5.4 as above.  From 65 pairs, whose rows are two waves, the waves of the
// segments hinder one another: 9.2 us at k = 65 and 10.9 at 100, 5.8 and 8.2 as above.
constexpr int FEW_SEGS = 4, FEW_MAXK = 64;

struct FewLds {
    double red[FEW_SEGS][FEW_MAXK], x[FEW_MAXK + FEW_SEGS * SOLVE_DEPTH];
};

// Column j by a workgroup of FEW_SEGS times k rounded up to 64, or more threads.
__device__ __forceinline__ void small_solve_segments(FewLds& s, int k, int kmax, const double* __restrict__ Rm,
                                                     const double* __restrict__ Rinv,
                                                     const double* __restrict__ RinvT,
                                                     const double* __restrict__ YHY, const double* __restrict__ Z,
                                                     SolveOut out, int32_t* __restrict__ status, int j) {
    auto& red = s.red;
    auto& x = s.x;
    const int rows = (k + 63) / 64 * 64;
    const int seg = __builtin_amdgcn_readfirstlane(threadIdx.x / rows), i = threadIdx.x - seg * rows;
    const int ic = min(i, k - 1);
    const int q = (k + 2 * FEW_SEGS - 1) / (2 * FEW_SEGS) * 2;     // pairs of a segment, even
    const int pitch = (q + SOLVE_DEPTH - 1) / SOLVE_DEPTH * SOLVE_DEPTH;   // in x, zeros between
    const int lo = min(k, seg * q), hi = min(k, lo + q), pos = ic / q * pitch + ic % q;
    const double zy = Z[(int64_t)j * 2 * k + k + ic], dii = Rm[(int64_t)ic * kmax + ic];
    double v = Z[(int64_t)j * 2 * k + ic], pv = 0.0;
    for (int t = threadIdx.x; t < FEW_SEGS * pitch; t += blockDim.x) x[t] = 0.0;
#pragma unroll 1
    for (int step = 0; step < 3; ++step) {
        __syncthreads();
        if (seg == 0 && i < k) x[pos] = v;
        __syncthreads();
        const double* A = step == 0 ? Rinv : step == 1 ? YHY : RinvT;
        if (seg < FEW_SEGS) red[seg][i] = lo < hi ? solve_chain(0.0, A, kmax, ic, lo, hi, x + seg * pitch - lo) : 0.0;
        __syncthreads();
        v = (red[0][i] + red[1][i]) + (red[2][i] + red[3][i]);
        if (step == 0) pv = v;
        if (step == 1) v += fma(dii, pv, -zy);
    }
    if (seg == 0 && i < k) {
        out.put(i, j, pv, v);
        if (!isfinite(pv) || !isfinite(v)) set_status(status, BFGS_ERR_NONFINITE);
    }
}

__global__ void __launch_bounds__(FEW_MAXK * FEW_SEGS) small_solve_few(int k, int kmax, const double* __restrict__ Rm,
                                                                  const double* __restrict__ Rinv,
                                                                  const double* __restrict__ RinvT,
                                                                  const double* __restrict__ YHY,
                                                                  const double* __restrict__ Z, SolveOut out,
                                                                  int32_t* __restrict__ status) {
    __shared__ FewLds lds;
    small_solve_segments(lds, k, kmax, Rm, Rinv, RinvT, YHY, Z, out, status, blockIdx.x);
}

// k = 0: B_0 V (or zero for B_k - B_0); a non-finite input sets the deferred status.
template <typename Th, typename Tv, typename To>
__global__ void scale_by_h0(int64_t n, int c, const Th* __restrict__ h0, const Tv* __restrict__ V,
                            To* __restrict__ out, int diff, int32_t* __restrict__ status) {
    const int64_t total = n * c;
    bool bad = false;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = e % n;
        const double v = to_f64(h0[r]) * to_f64(V[e]);
        bad |= !isfinite(v);
        out[e] = diff ? (To)0 : (To)v;
    }
    if (bad) set_status(status, BFGS_ERR_NONFINITE);
}

// ---------------------------------------------------------------------------
// Float64 matrix-core forms of both passes for float32 and float64 storage
// (tall_f64.h).  Both read W = [S | h0 o Y] (n x 2k), widened to float64 and scaled as it
// is loaded:
//   pass 1:  Z = W^T V                  (= [S^T V ; Y^T (h0 o V)])
//   pass 2:  out = W [T ; -P] + h0 o V  (= h0 o (V - Y P) + S T; no h0 o V for B_k - B_0)
// ---------------------------------------------------------------------------
// Column p of W: S's column p, or Y's column p - k, which takes the row scale.
template <typename Ts>
struct PairCols {
    const Ts *S, *Y;
    int64_t ld;
    int k;
    __device__ __forceinline__ TnCol<Ts> operator()(int p) const {
        const bool y = p >= k;
        return {(y ? Y : S) + (int64_t)(y ? p - k : p) * ld, y};
    }
};

// part[chunk][j * 2k + p] = sum over the chunk's rows of W(r, p) V(r, j); V's columns are
// ldv apart (n for a whole block; the block's row count when the rows come in slices).
template <int TA, int TB, typename Ts, typename Th, typename Tv>
__global__ void __launch_bounds__(64, 2) gemm1_f64mfma(int64_t n, int64_t ld, int k, int c, const Ts* __restrict__ S,
                                                       const Ts* __restrict__ Y, const Th* __restrict__ h0,
                                                       const Tv* __restrict__ V, int64_t ldv,
                                                       double* __restrict__ part, int64_t rows_per_chunk, int nchunks,
                                                       int ptiles, int ctiles) {
    int chunk, pos;
    if (!tn_place(blockIdx.x, ptiles * ctiles, nchunks, chunk, pos)) return;
    tn_tile<TA, TB, true, false, Ts>(n, 2 * k, c, chunk, rows_per_chunk, pos % ptiles, pos / ptiles, ctiles,
                                     PairCols<Ts>{S, Y, ld, k}, h0, V, ldv, part);
}

// Stores the results of rows r .. r + live - 1 of column j, with h0 o V added unless diff.
template <int TA, typename To, typename Tv>
struct ApplyEmit {
    const Tv* V;
    To* out;
    int64_t ldv;
    int diff;
    typedef Run<Tv, TA> Ahead;
    __device__ __forceinline__ Ahead ahead(int j, int64_t r, int live) const {
        Ahead v{};
        if (!diff) {
            const Tv* p = V + (int64_t)j * ldv + r;
            v = live == TA ? load_run<Tv, TA>(p) : load_run_part<Tv, TA>(p, live);
        }
        return v;
    }
    __device__ __forceinline__ void store(int j, int64_t r, const double (&o)[TA], const double (&h)[TA], const Ahead& v,
                                          int live) const {
        To* p = out + (int64_t)j * ldv + r;
        Run<To, TA> w;
#pragma unroll
        for (int f = 0; f < TA; ++f) {
            double s = o[f];
            if (!diff) s += h[f] * to_f64(v.v[f]);
            w.v[f] = (To)s;
        }
        if (live == TA) {
            *(Run<To, TA>*)p = w;
        } else {
#pragma unroll
            for (int f = 0; f < TA; ++f)
                if (f < live) p[f] = w.v[f];
        }
    }
};

// out (column-major n x c, columns ldv apart, as V's) = W [T ; -P] (+ h0 o V unless diff),
// [T ; -P] packed.
template <int TA, int TB, bool SKIP, typename Ts, typename Th, typename To, typename Tv>
__device__ __forceinline__ void gemm2_group(NnLds<TB>& lds, int64_t n, int64_t ld, int k, int c,
                                            const Ts* __restrict__ S, const Ts* __restrict__ Y,
                                            const Th* __restrict__ h0, const Tv* __restrict__ V, int64_t ldv,
                                            const double* __restrict__ M, To* __restrict__ out, int diff, int64_t row0,
                                            int ct, int ctiles) {
    const int cblocks = (c + 15) / 16, cb = ct * cblocks / ctiles, ce = (ct + 1) * cblocks / ctiles;
    // the columns of S and Y are ld (a multiple of 128) rows long: whole runs exist
    nn_group<TA, TB, true, SKIP, Ts>(lds, n, row0, true, 2 * k, c, cblocks, cb, ce - cb, PairCols<Ts>{S, Y, ld, k}, h0,
                                     M, ApplyEmit<TA, To, Tv>{V, out, ldv, diff});
}

template <int TA, int TB, typename Ts, typename Th, typename To, typename Tv>
__global__ void __launch_bounds__(256, 2) gemm2_f64mfma(int64_t n, int64_t ld, int k, int c, const Ts* __restrict__ S,
                                                        const Ts* __restrict__ Y, const Th* __restrict__ h0,
                                                        const Tv* __restrict__ V, int64_t ldv,
                                                        const double* __restrict__ M, To* __restrict__ out, int diff,
                                                        int ctiles) {
    __shared__ NnLds<TB> lds;
    int64_t row0;
    int ct;
    if (!nn_place(blockIdx.x, n, 64 * TA, ctiles, row0, ct)) return;
    gemm2_group<TA, TB, false, Ts, Th, To, Tv>(lds, n, ld, k, c, S, Y, h0, V, ldv, M, out, diff, row0, ct, ctiles);
}

template <typename Ts, typename Th, typename Tv>
void launch_gemm1(hipStream_t st, int64_t n, int64_t ld, int k, int c, const Ts* S, const Ts* Y, const Th* h0,
                  const Tv* V, int64_t ldv, double* part, int64_t rows_per_chunk, int nchunks) {
    constexpr bool wide = sizeof(Tv) == 8;
    const TnShape s = tn_shape(2 * k, c, wide);
    with_tile_width(s.tb, [&](auto tb) {
        constexpr int TB = wide && decltype(tb)::value > TN_WIDE_TB ? TN_WIDE_TB : decltype(tb)::value;
        hipLaunchKernelGGL((gemm1_f64mfma<tile_rows(TB), TB, Ts, Th, Tv>), dim3(tn_grid(s.tiles(), nchunks)),
                           dim3(64), 0, st, n, ld, k, c, S, Y, h0, V, ldv, part, rows_per_chunk, nchunks, s.ptiles,
                           s.ctiles);
    });
}

template <typename Ts, typename Th, typename To, typename Tv>
void launch_gemm2(hipStream_t st, int64_t n, int64_t ld, int k, int c, const Ts* S, const Ts* Y, const Th* h0,
                  const Tv* V, int64_t ldv, const double* M, To* out, bool diff) {
    const NnShape s = nn_shape(c);
    with_tile_width(s.tb, [&](auto tb) {
        constexpr int TB = decltype(tb)::value;
        hipLaunchKernelGGL((gemm2_f64mfma<tile_rows(TB), TB, Ts, Th, To, Tv>), dim3(nn_grid(n, s)), dim3(256), 0, st, n,
                           ld, k, c, S, Y, h0, V, ldv, M, out, diff ? 1 : 0, s.ctiles);
    });
}

// Row chunks of pass 1 over n rows for a history of k pairs and c columns: how many rows
// go into one partial sum.  The chunk length fixes the order of the sums.  For the rSVD's
// range sample (diff) it stays what it was when a tile had 128 x 128 results, about 2048
// of them: the columns of U at numerically zero eigenvalues are rounding noise and would
// turn with any other order.  Otherwise as many chunks as fill the wave slots once, or
// twice where a chunk then still has 1024 rows; counted by XCD (a chunk's tiles share one,
// workgroup g runs on XCD g % 8), so that the last round of waves is a full one: at
// n = 1.785M, k = 200, c = 220, float32, 157 chunks of 26 tiles are 2.03 rounds on five of
// the XCDs and took 7.0 ms, 152 are 1.93 and take 5.9.
struct ChunkPlan {
    int64_t rows_per_chunk;
    int nchunks;
};
ChunkPlan chunk_plan(int64_t n, int k, int c, bool diff, bool wide_v, int most = 1 << 20) {
    int64_t nch;
    if (diff) {
        nch = std::max(1, 2048 / (ceil_div(2 * k, 128) * ceil_div(c, 128)));
    } else {
        const TnShape s = tn_shape(2 * k, c, wide_v);
        const int slots = 32 * 4 * s.waves;   // of one XCD
        nch = 8 * std::max(1, 2 * slots / s.tiles());
        if (n < 1024 * nch) nch = 8 * std::max(1, slots / s.tiles());
        nch = std::min(nch, (n + 63) / 64);
    }
    nch = std::min(std::min<int64_t>(nch, most), (n + 15) / 16);
    const int64_t rows = round_up((n + nch - 1) / nch, 16);
    return {rows, (int)((n + rows - 1) / rows)};
}

// Doubles of the P/T workspace: P and T (k x c each) or the packed [T ; -P].
size_t pt_doubles(int kmax) { return (size_t)(2 * kmax + 2) * BFGS_MAX_COLS; }

int small_solve_launch(bfgsuq_ctx* h, int c, const double* Z, SolveOut out) {
    ProfScope ps(h, "apply_solve");
    const int k = h->k;
    if (k <= 256)
        hipLaunchKernelGGL(small_solve_blocks, dim3(c), dim3((unsigned)round_up(k, 64)), 0, h->stream, k, h->kmax, h->Rm,
                           h->Rinv, h->RinvT, h->YHY, Z, out, h->status);
    else
        hipLaunchKernelGGL(small_solve, dim3(c), dim3(64), 3 * k * sizeof(double), h->stream, k, h->kmax, c, h->Rm,
                           h->YHY, Z, out, h->status);
    return hipGetLastError() == hipSuccess ? BFGS_OK : BFGS_ERR_HIP;
}

// A few columns (c <= STREAM_COLS): both passes on the vector unit (stream_f64.h).
template <typename Ts, typename Th, typename To, typename Tv>
int apply_few(bfgsuq_ctx* h, const Tv* V, int c, To* out, bool diff, const ApplyWs* fixed) {
    const int64_t n = h->n;
    const int k = h->k;
    const Th* h0 = (const Th*)h->h0;
    const Ts *S = (const Ts*)h->S, *Y = (const Ts*)h->Y;
    const size_t chunk_bytes = (size_t)2 * k * c * 8;
    const StreamPlan plan = stream_plan(n, k, fixed ? (int64_t)(fixed->part_bytes / chunk_bytes) : 1 << 20);
    const int groups = plan.groups, nchunks = plan.nchunks;
    const int64_t rows = plan.rows_per_chunk;
    double *part, *Z, *P;
    if (fixed) {
        part = (double*)fixed->part;
        Z = fixed->Z;
        P = fixed->PT;
    } else {
        int rc;
        if ((rc = ensure_ws(h->part, stream_part_bytes(n, h->kmax))) != BFGS_OK) return rc;
        if ((rc = ensure_ws(h->Z, (size_t)2 * h->kmax * BFGS_MAX_COLS * 8)) != BFGS_OK) return rc;
        if ((rc = ensure_ws(h->PT, pt_doubles(h->kmax) * 8)) != BFGS_OK) return rc;
        part = (double*)h->part.ptr;
        Z = (double*)h->Z.ptr;
        P = (double*)h->PT.ptr;
    }
    double* T = P + (size_t)k * c;
    const SolveOut plain{P, T, nullptr, k, 0, nullptr, nullptr, 0};
    {
        ProfScope ps(h, diff ? "hdiff_gemm1" : "apply_gemm1");
        with_few_columns(c, [&](auto cc) {
            hipLaunchKernelGGL((stream_pass1<decltype(cc)::value, Ts, Th, Tv>), dim3(tn_grid(2 * groups, nchunks)),
                               dim3(64), 0, h->stream, n, h->ld, k, c, S, Y, h0, V, nchunks > 1 ? part : Z, rows, nchunks,
                               groups);
        });
    }
    if (nchunks > 1) {
        ProfScope ps(h, "apply_reduce");
        if (int rc = sum_partials(h->stream, (int64_t)2 * k * c, nchunks, part, Z)) return rc;
    }
    if (k <= FEW_MAXK) {
        ProfScope ps(h, "apply_solve");
        hipLaunchKernelGGL(small_solve_few, dim3(c), dim3((unsigned)(FEW_SEGS * round_up(k, 64))), 0, h->stream, k,
                           h->kmax, h->Rm, h->Rinv, h->RinvT, h->YHY, Z, plain, h->status);
    } else if (int rc = small_solve_launch(h, c, Z, plain)) {
        return rc;
    }
    ProfScope ps(h, diff ? "hdiff_gemm2" : "apply_gemm2");
    with_few_columns(c, [&](auto cc) {
        hipLaunchKernelGGL((stream_pass2<decltype(cc)::value, Ts, Th, To, Tv>),
                           dim3((unsigned)ceil_div(n, 64 * stream_rows<Ts>())), dim3(256), 0, h->stream, n, h->ld, k, c,
                           S, Y, h0, V, P, T, out, diff ? 1 : 0);
    });
    return hipGetLastError() == hipSuccess ? BFGS_OK : BFGS_ERR_HIP;
}

// Bytes of the partial sums of a block, for both of its directions (B_k V and (B_k - B_0) V
// are split differently): a caller that takes one after the other, as the variance after
// the inversion's block, would otherwise replace the workspace in between, which waits for
// the device (a batch of 8 such problems: 29.8 ms in its first pass, 11.8 now).
size_t part_bytes(int64_t n, int k, int c, bool wide_v) {
    const int chunks = std::max(chunk_plan(n, k, c, false, wide_v).nchunks, chunk_plan(n, k, c, true, wide_v).nchunks);
    return (size_t)chunks * 2 * k * c * 8;
}

template <typename Ts, typename Th, typename To, typename Tv = Ts>
int apply_generic(bfgsuq_ctx* h, const void* Vv, int c, void* outv, bool diff, const ApplyWs* fixed) {
    const int64_t n = h->n;
    const int k = h->k;
    const Th* h0 = (const Th*)h->h0;
    const Tv* V = (const Tv*)Vv;
    To* out = (To*)outv;
    if (k == 0) {
        int64_t g = std::min<int64_t>(4096, (n * c + 255) / 256);
        hipLaunchKernelGGL((scale_by_h0<Th, Tv, To>), dim3((int)g), dim3(256), 0, h->stream, n, c, h0, V, out,
                           diff ? 1 : 0, h->status);
        return hipGetLastError() == hipSuccess ? BFGS_OK : BFGS_ERR_HIP;
    }
    if (c <= STREAM_COLS) return apply_few<Ts, Th, To, Tv>(h, V, c, out, diff, fixed);
    const int twok = 2 * k;
    const size_t chunk_bytes = (size_t)twok * c * 8;
    int most = 1 << 20;
    if (fixed) {
        most = (int)std::min<size_t>(fixed->part_bytes / chunk_bytes, most);
        if (most < 1) return BFGS_ERR_ARG;
    }
    const ChunkPlan plan = chunk_plan(n, k, c, diff, sizeof(Tv) == 8, most);
    double *part, *Z, *M;
    if (fixed) {
        part = (double*)fixed->part;
        Z = fixed->Z;
        M = fixed->PT;
    } else {
        int rc;
        if ((rc = ensure_ws(h->part, part_bytes(n, k, c, sizeof(Tv) == 8))) != BFGS_OK) return rc;
        if ((rc = ensure_ws(h->Z, (size_t)2 * h->kmax * BFGS_MAX_COLS * 8)) != BFGS_OK) return rc;
        if ((rc = ensure_ws(h->PT, pt_doubles(h->kmax) * 8)) != BFGS_OK) return rc;
        part = (double*)h->part.ptr;
        Z = (double*)h->Z.ptr;
        M = (double*)h->PT.ptr;
    }
    prof_begin(h, diff ? "hdiff_gemm1" : "apply_gemm1");
    launch_gemm1<Ts, Th, Tv>(h->stream, n, h->ld, k, c, (const Ts*)h->S, (const Ts*)h->Y, h0, V, n, part,
                             plan.rows_per_chunk, plan.nchunks);
    prof_end(h);
    prof_begin(h, "apply_reduce");
    if (int rc2 = sum_partials(h->stream, (int64_t)twok * c, plan.nchunks, part, Z)) return rc2;
    prof_end(h);
    const SolveOut packed{nullptr, nullptr, M, k, ceil_div(c, 16), nullptr, nullptr, 0};
    if (int rc2 = small_solve_launch(h, c, Z, packed)) return rc2;
    prof_begin(h, diff ? "hdiff_gemm2" : "apply_gemm2");
    launch_gemm2<Ts, Th, To, Tv>(h->stream, n, h->ld, k, c, (const Ts*)h->S, (const Ts*)h->Y, h0, V, n, M, out, diff);
    prof_end(h);
    return hipGetLastError() == hipSuccess ? BFGS_OK : BFGS_ERR_HIP;
}

// The same two passes for a history kept in host memory (bfgs_create_streamed): each
// pass streams S and Y through the device in row slices and runs its kernel on one
// slice while the next is copied; the pass-1 partials of all slices are summed in one
// fixed order, so the result does not depend on the copy timing.
template <typename Ts, typename Th, typename To, typename Tv = Ts>
int apply_streamed(bfgsuq_ctx* h, const void* Vv, int c, void* outv, bool diff) {
    const int64_t n = h->n;
    const int k = h->k;
    if (k == 0) return apply_generic<Ts, Th, To, Tv>(h, Vv, c, outv, diff, nullptr);   // reads no pair
    const Th* h0 = (const Th*)h->h0;
    const Tv* V = (const Tv*)Vv;
    To* out = (To*)outv;
    const int twok = 2 * k;
    const int64_t sr = h->slice_rows;
    const int ns = (int)((n + sr - 1) / sr);
    const ChunkPlan plan = chunk_plan(sr, k, c, diff, sizeof(Tv) == 8);   // of one slice
    const int64_t rows_per_sub = plan.rows_per_chunk;
    const int nsub = plan.nchunks;
    const int64_t last_rows = n - (int64_t)(ns - 1) * sr;
    const int used = (ns - 1) * nsub + (int)((last_rows + rows_per_sub - 1) / rows_per_sub);
    const size_t chunk_bytes = (size_t)twok * c * 8;
    int rc;
    if ((rc = ensure_ws(h->part, (size_t)ns * nsub * chunk_bytes)) != BFGS_OK) return rc;
    if ((rc = ensure_ws(h->Z, (size_t)2 * h->kmax * BFGS_MAX_COLS * 8)) != BFGS_OK) return rc;
    if ((rc = ensure_ws(h->PT, pt_doubles(h->kmax) * 8)) != BFGS_OK) return rc;
    double* part = (double*)h->part.ptr;
    double* Z = (double*)h->Z.ptr;
    double* M = (double*)h->PT.ptr;
    {
        ProfScope ps(h, diff ? "hdiff_stream_pass1" : "apply_stream_pass1");
        rc = stream_slices(h, k, [&](int i, int64_t r0, int64_t rows, const void* Sst, const void* Yst) {
            const int nsi = (int)((rows + rows_per_sub - 1) / rows_per_sub);
            launch_gemm1<Ts, Th, Tv>(h->stream, rows, h->slice_ld, k, c, (const Ts*)Sst, (const Ts*)Yst, h0 + r0,
                                     V + r0, n, part + (size_t)i * nsub * twok * c, rows_per_sub, nsi);
            return hipGetLastError() == hipSuccess ? BFGS_OK : BFGS_ERR_HIP;
        });
        if (rc != BFGS_OK) return rc;
    }
    const int64_t count = (int64_t)twok * c;
    if ((rc = sum_partials(h->stream, count, used, part, Z)) != BFGS_OK) return rc;
    const SolveOut packed{nullptr, nullptr, M, k, ceil_div(c, 16), nullptr, nullptr, 0};
    if ((rc = small_solve_launch(h, c, Z, packed)) != BFGS_OK) return rc;
    ProfScope ps(h, diff ? "hdiff_stream_pass2" : "apply_stream_pass2");
    rc = stream_slices(h, k, [&](int, int64_t r0, int64_t rows, const void* Sst, const void* Yst) {
        launch_gemm2<Ts, Th, To, Tv>(h->stream, rows, h->slice_ld, k, c, (const Ts*)Sst, (const Ts*)Yst, h0 + r0, V + r0,
                                     n, M, out + r0, diff);
        return hipGetLastError() == hipSuccess ? BFGS_OK : BFGS_ERR_HIP;
    });
    return rc;
}

// ---------------------------------------------------------------------------
// Persistent batched apply (float32 and float64 storage): the first pass of every
// problem, the float64 small steps of every problem and the second pass of every
// problem are one launch each (the solve two where problems of up to FEW_MAXK pairs and few
// columns stand beside others).  A pass's workgroups take (problem, tile) items from
// a work queue (an atomic counter) until it runs dry; the problems are laid out
// longest first (work n k c), so the last items to be taken are small ones.  Each
// item is exactly one workgroup of the per-problem kernels (same tiles, same
// chunking, same fixed-order sums), so the results equal the per-problem path's.
// ---------------------------------------------------------------------------
// A pointer read from memory that is known to be global (loads through it are then global
// loads, not flat ones).
template <typename T>
__device__ __forceinline__ T* global_ptr(const void* p) {
    return (T*)(__attribute__((address_space(1))) T*)(uintptr_t)p;
}

// FEW: some problem has few columns, whose items are those of the streaming passes (a kernel of
// its own, as their registers would spill the tiles').
template <int TB, bool FEW, typename Ts, typename Th, typename Tv>
__global__ void __launch_bounds__(64, 2) batch_pass1(const PersistProblem* __restrict__ pr, int nprob, int total,
                                                     unsigned* __restrict__ head) {
    for (;;) {
        int item = 0;
        if (threadIdx.x == 0) item = (int)atomicAdd(head, 1u);
        item = __builtin_amdgcn_readfirstlane(item);   // a workgroup is one wave
        if (item >= total) break;
        int lo = 0, hi = nprob - 1;   // last problem whose first item is <= item
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (pr[mid].first1 <= item) lo = mid;
            else hi = mid - 1;
        }
        const PersistProblem& q = pr[lo];
        const int local = item - q.first1, per = q.ptiles * q.ctiles1;
        const int chunk = local / per, pos = local % per;
        if (FEW && q.few) {
            with_few_columns(q.c, [&](auto cc) {
                stream_chunk<decltype(cc)::value, Ts, Th, Tv>(
                    q.n, q.ld, q.k, q.c, global_ptr<const Ts>(q.S), global_ptr<const Ts>(q.Y), global_ptr<const Th>(q.h0),
                    global_ptr<const Tv>(q.V), global_ptr<double>(q.nchunks > 1 ? q.part : q.Z), q.rows_per_chunk,
                    q.ptiles / 2, chunk, pos);
            });
            continue;
        }
        tn_tile<2, TB, true, true, Ts>(q.n, 2 * q.k, q.c, chunk, q.rows_per_chunk, pos % q.ptiles, pos / q.ptiles,
                                       q.ctiles1, PairCols<Ts>{global_ptr<const Ts>(q.S), global_ptr<const Ts>(q.Y), q.ld, q.k},
                                       global_ptr<const Th>(q.h0), global_ptr<const Tv>(q.V), q.n, global_ptr<double>(q.part));
    }
}

// Z of every problem: the fixed-order sums of its pass-1 partials, one workgroup per
// (problem, SUM_ENTRIES entries), as reduce_partials forms them.
__global__ void __launch_bounds__(SUM_THREADS) batch_sum(const PersistProblem* __restrict__ pr, int nprob) {
    __shared__ double sh[SUM_DEPTH][SUM_ENTRIES];
    int lo = 0, hi = nprob - 1;   // last problem whose first block is <= this one
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (pr[mid].firstsum <= (int)blockIdx.x) lo = mid;
        else hi = mid - 1;
    }
    const PersistProblem& q = pr[lo];
    const int64_t count = (int64_t)2 * q.k * q.c;
    const int64_t e = (int64_t)((int)blockIdx.x - q.firstsum) * SUM_ENTRIES + threadIdx.x % SUM_ENTRIES;
    const bool live = e < count;
    const double* part = q.part;
    const double t = ordered_sum(
        0, q.nchunks, sh, [&](int ch) { return live ? part[(int64_t)ch * count + e] : 0.0; },
        [](double sum, double v, int) { return sum + v; });
    if (threadIdx.x < SUM_ENTRIES && e < count) q.Z[e] = t;
}

// One workgroup per (problem, column): its small solve, by the kernel of its form.
template <bool SEGMENTS>
__global__ void __launch_bounds__(SEGMENTS ? FEW_MAXK * FEW_SEGS : 256) batch_solve(
    const PersistProblem* __restrict__ pr, int nprob) {
    int j = blockIdx.x, p = 0;
    while (p < nprob && j >= pr[p].c) j -= pr[p++].c;
    if (p >= nprob) return;   // whole workgroup
    const PersistProblem& q = pr[p];
    if (SEGMENTS != (q.few && q.k <= FEW_MAXK)) return;   // whole workgroup
    __shared__ std::conditional_t<SEGMENTS, FewLds, SolveLds> lds;
    double* M = global_ptr<double>(q.M);
    const SolveOut out = q.few ? SolveOut{M, M + (int64_t)q.k * q.c, nullptr, q.k, 0, nullptr, nullptr, 0}
                               : SolveOut{nullptr, nullptr, M, q.k, (q.c + 15) / 16, nullptr, nullptr, 0};
    if constexpr (SEGMENTS)
        small_solve_segments(lds, q.k, q.kmax, global_ptr<double>(q.Rm), global_ptr<double>(q.Rinv),
                             global_ptr<double>(q.RinvT), global_ptr<double>(q.YHY), global_ptr<double>(q.Z), out,
                             q.status, j);
    else
        small_solve_block(lds, q.k, q.kmax, global_ptr<double>(q.Rm), global_ptr<double>(q.Rinv),
                          global_ptr<double>(q.RinvT), global_ptr<double>(q.YHY), global_ptr<double>(q.Z), out,
                          q.status, j);
}

template <bool FEW, typename Ts, typename Th, typename To, typename Tv>
__global__ void __launch_bounds__(256, 2) batch_pass2(const PersistProblem* __restrict__ pr, int nprob, int total,
                                                    unsigned* __restrict__ head) {
    __shared__ int item_sh;
    __shared__ union {
        NnLds<NN_TB> tile;
        StreamLds<1, Ts> s1;
        StreamLds<2, Ts> s2;
        StreamLds<STREAM_COLS, Ts> s4;
    } lds;
    for (;;) {
        if (threadIdx.x == 0) item_sh = (int)atomicAdd(head, 1u);
        __syncthreads();
        const int item = item_sh;
        __syncthreads();
        if (item >= total) break;
        int lo = 0, hi = nprob - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (pr[mid].first2 <= item) lo = mid;
            else hi = mid - 1;
        }
        const PersistProblem& q = pr[lo];
        const int local = item - q.first2;
        if (FEW && q.few) {
            with_few_columns(q.c, [&](auto cc) {
                constexpr int CC = decltype(cc)::value;
                double* M = global_ptr<double>(q.M);
                stream_block<CC, Ts, Th, To, Tv>(
                    (StreamLds<CC, Ts>&)lds, q.n, q.ld, q.k, q.c, global_ptr<const Ts>(q.S), global_ptr<const Ts>(q.Y),
                    global_ptr<const Th>(q.h0), global_ptr<const Tv>(q.V), M, M + (int64_t)q.k * q.c,
                    global_ptr<To>(q.out), 0, local);
            });
            continue;
        }
        gemm2_group<2, NN_TB, true, Ts, Th, To, Tv>(
            lds.tile, q.n, q.ld, q.k, q.c, global_ptr<const Ts>(q.S), global_ptr<const Ts>(q.Y), global_ptr<const Th>(q.h0),
            global_ptr<const Tv>(q.V), q.n, global_ptr<double>(q.M), global_ptr<To>(q.out), 0,
            (int64_t)(local / q.ctiles2) * 128, local % q.ctiles2, q.ctiles2);
    }
}

// The work-queue heads start at zero for every launch (a kernel, so that a captured
// graph resets them on every replay).
__global__ void batch_reset(unsigned* __restrict__ head) {
    if (threadIdx.x < 2) head[threadIdx.x] = 0u;
}

template <typename Ts, typename Th>
int batch_persistent_impl(bfgsuq_ctx* const* hs, int nprob, const void* const* V, const int32_t* ncols,
                          void* const* out, hipStream_t st, PersistSlot* slot, bool upload, int wg_per_cu) {
    constexpr int TB1 = sizeof(Ts) == 8 ? TN_WIDE_TB : NN_TB;
    if (upload) {
        std::vector<int> order(nprob);
        for (int i = 0; i < nprob; ++i) order[i] = i;
        std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
            return (double)hs[a]->n * hs[a]->k * ncols[a] > (double)hs[b]->n * hs[b]->k * ncols[b];
        });
        std::vector<PersistProblem> host(nprob);
        int t1 = 0, tsum = 0, t2 = 0, tsolve = 0;
        bool few = false, segments = false, chains = false;
        for (int r = 0; r < nprob; ++r) {
            const int i = order[r];
            bfgsuq_ctx* h = hs[i];
            const int k = h->k, c = ncols[i], twok = 2 * k;
            if (k < 1 || k > 256) return BFGS_ERR_ARG;
            PersistProblem& q = host[r];
            q.n = h->n;
            q.ld = h->ld;
            q.k = k;
            q.kmax = h->kmax;
            q.c = c;
            q.S = h->S;
            q.Y = h->Y;
            q.h0 = h->h0;
            q.V = V[i];
            q.out = out[i];
            // the per-problem path's form and chunking, so that the partial sums match it
            q.few = c <= STREAM_COLS;
            size_t need;
            if (q.few) {
                const StreamPlan plan = stream_plan(q.n, k);
                q.ptiles = 2 * plan.groups;
                q.ctiles1 = q.ctiles2 = 1;
                q.rows_per_chunk = plan.rows_per_chunk;
                q.nchunks = plan.nchunks;
                need = stream_part_bytes(q.n, h->kmax);
            } else {
                q.ptiles = ceil_div(ceil_div(twok, 16), 2);
                q.ctiles1 = ceil_div(ceil_div(c, 16), TB1);
                q.ctiles2 = ceil_div(ceil_div(c, 16), NN_TB);
                const ChunkPlan plan = chunk_plan(q.n, k, c, false, sizeof(Ts) == 8);
                q.rows_per_chunk = plan.rows_per_chunk;
                q.nchunks = plan.nchunks;
                need = part_bytes(q.n, k, c, sizeof(Ts) == 8);
            }
            few |= q.few != 0;
            (q.few && k <= FEW_MAXK ? segments : chains) = true;
            int rc;
            if ((rc = ensure_ws(h->part, need)) != BFGS_OK) return rc;
            if ((rc = ensure_ws(h->Z, (size_t)2 * h->kmax * BFGS_MAX_COLS * 8)) != BFGS_OK) return rc;
            if ((rc = ensure_ws(h->PT, pt_doubles(h->kmax) * 8)) != BFGS_OK) return rc;
            q.part = (double*)h->part.ptr;
            q.Z = (double*)h->Z.ptr;
            q.M = (double*)h->PT.ptr;
            q.Rm = h->Rm;
            q.Rinv = h->Rinv;
            q.RinvT = h->RinvT;
            q.YHY = h->YHY;
            q.status = h->status;
            q.first1 = t1;
            q.firstsum = tsum;
            q.first2 = t2;
            t1 += q.nchunks * q.ptiles * q.ctiles1;
            if (!q.few || q.nchunks > 1) tsum += ceil_div((int64_t)twok * c, SUM_ENTRIES);
            t2 += ceil_div(q.n, q.few ? 64 * stream_rows<Ts>() : 128) * q.ctiles2;
            tsolve += c;
        }
        if (slot->cap < (size_t)nprob) {
            if (slot->prob) (void)hipFree(slot->prob);
            slot->prob = nullptr;
            slot->cap = 0;
            if (hipMalloc((void**)&slot->prob, (size_t)nprob * sizeof(PersistProblem)) != hipSuccess)
                return BFGS_ERR_ALLOC;
            slot->cap = (size_t)nprob;
        }
        if (!slot->head && hipMalloc((void**)&slot->head, 64) != hipSuccess) {
            slot->head = nullptr;
            return BFGS_ERR_ALLOC;
        }
        // pageable source: the call returns once the data is staged
        BFGS_HIP(hipMemcpyAsync(slot->prob, host.data(), (size_t)nprob * sizeof(PersistProblem),
                                hipMemcpyHostToDevice, st));
        slot->nprob = nprob;
        slot->items1 = t1;
        slot->sum_blocks = tsum;
        slot->items2 = t2;
        slot->solve_blocks = tsolve;
        slot->few = few;
        slot->segments = segments;
        slot->chains = chains;
    }
    if (slot->nprob != nprob || !slot->prob) return BFGS_ERR_STATE;
    int dev = 0, ncu = 256;
    if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    const int g1 = std::max(1, std::min(slot->items1, 4 * ncu * wg_per_cu));   // single waves
    const int g2 = std::max(1, std::min(slot->items2, ncu * wg_per_cu));
    hipLaunchKernelGGL(batch_reset, dim3(1), dim3(64), 0, st, slot->head);
    if (slot->few)
        hipLaunchKernelGGL((batch_pass1<TB1, true, Ts, Th, Ts>), dim3(g1), dim3(64), 0, st, slot->prob, nprob,
                           slot->items1, slot->head);
    else
        hipLaunchKernelGGL((batch_pass1<TB1, false, Ts, Th, Ts>), dim3(g1), dim3(64), 0, st, slot->prob, nprob,
                           slot->items1, slot->head);
    if (slot->sum_blocks)
        hipLaunchKernelGGL(batch_sum, dim3(slot->sum_blocks), dim3(SUM_THREADS), 0, st, slot->prob, nprob);
    if (slot->chains)
        hipLaunchKernelGGL(batch_solve<false>, dim3(slot->solve_blocks), dim3(256), 0, st, slot->prob, nprob);
    if (slot->segments)
        hipLaunchKernelGGL(batch_solve<true>, dim3(slot->solve_blocks), dim3(FEW_MAXK * FEW_SEGS), 0, st, slot->prob,
                           nprob);
    if (slot->few)
        hipLaunchKernelGGL((batch_pass2<true, Ts, Th, Th, Ts>), dim3(g2), dim3(256), 0, st, slot->prob, nprob,
                           slot->items2, slot->head + 1);
    else
        hipLaunchKernelGGL((batch_pass2<false, Ts, Th, Th, Ts>), dim3(g2), dim3(256), 0, st, slot->prob, nprob,
                           slot->items2, slot->head + 1);
    return hipGetLastError() == hipSuccess ? BFGS_OK : BFGS_ERR_HIP;
}

}  // namespace

int batch_apply_persistent(bfgsuq_ctx* const* hs, int nprob, const void* const* V, const int32_t* ncols,
                           void* const* out, hipStream_t st, PersistSlot* slot, bool upload, int wg_per_cu) {
    if (nprob < 1) return BFGS_ERR_ARG;
    const bfgs_dtype s0 = hs[0]->storage;
    for (int i = 0; i < nprob; ++i)
        if (hs[i]->storage != s0 || hs[i]->streamed || hs[i]->k < 1 || hs[i]->k > 256)
            return BFGS_ERR_ARG;
    if (s0 == BFGS_F64) return batch_persistent_impl<double, double>(hs, nprob, V, ncols, out, st, slot, upload, wg_per_cu);
    if (s0 == BFGS_F32) return batch_persistent_impl<float, float>(hs, nprob, V, ncols, out, st, slot, upload, wg_per_cu);
    return BFGS_ERR_ARG;
}

int sum_partials(hipStream_t st, int64_t count, int nchunks, const double* part, double* out, bool projection) {
    hipLaunchKernelGGL(projection ? reduce_partials<ProjectionSum> : reduce_partials<ApplySum>,
                       dim3(ceil_div(count, SUM_ENTRIES)), dim3(SUM_THREADS), 0, st, count, nchunks, part, out);
    return hipGetLastError() == hipSuccess ? BFGS_OK : BFGS_ERR_HIP;
}

int apply_small_solve_halves(bfgsuq_ctx* h, int c, const double* Z, int rows, uint16_t* hi, uint16_t* lo) {
    return small_solve_launch(h, c, Z, SolveOut{nullptr, nullptr, nullptr, h->k, 0, hi, lo, rows});
}

bool apply_takes_tiles(int ncols) { return ncols > STREAM_COLS; }

// B_k V of a few columns from bfloat16 pairs streams them, as other storage does, rather than
// fill a matrix-core tile of 32; the difference form stays on the matrix cores, as the rSVD's
// other blocks are.  Streaming against the tile (the difference form's time, which reads V once
// less), us:
//     k     n        1 column      2            3            4
//    60     9,000    18 | 19      20 | 21      24 | 21      25 | 21
//   100       900    21 | 24      25 | 25      29 | 25      31 | 25
//   100     9,000    24 | 24      27 | 25      33 | 25      34 | 25
//   128    65,536    32 | 36      35 | 37      43 | 37      44 | 37
//   128   200,000    53 | 60      56 | 61      67 | 62      68 | 62
//   128 1,785,000   359 | 359    365 | 376    415 | 383    422 | 388
//   150   200,000    60 | 72      64 | 72      as a tile
//   200    65,536    47 | 50      50 | 50      as a tile
//   200 1,785,000   557 | 529    564 | 548     as a tile
// Three and four columns lose up to 9 us of small blocks that way (the tile as it was before
// took 32 at k = 100, n = 9,000), but the results are the more exact: float64 sums rounded
// once, where the tile's products are bfloat16 pairs in float32.  Beyond 128 pairs a
// workgroup's chain over the pairs in pass 2 costs more than that is worth on small blocks and
// on three columns.
bool apply_takes_mfma(const bfgsuq_ctx* h, int ncols, bool diff) {
    const bool few = !diff && ncols <= STREAM_COLS && (h->k <= 128 || (ncols <= 2 && h->n >= 65536));
    return mfma_apply_supported(h, ncols) && !few;
}

int apply_diff_float_block(bfgsuq_ctx* h, const void* V, bool f64, int32_t ncols, void* out) {
    // (B_k - B_0) V for a block of the type in which the rSVD keeps Q, not a probe block in the
    // storage type (float64 for float32 and float64 storage, float32 for bfloat16), on the
    // float64 matrix cores
    if (h->storage == BFGS_F64 && f64)
        return h->streamed ? apply_streamed<double, double, double, double>(h, V, ncols, out, true)
                           : apply_generic<double, double, double, double>(h, V, ncols, out, true, nullptr);
    if (h->storage == BFGS_F32 && f64)
        return h->streamed ? apply_streamed<float, float, double, double>(h, V, ncols, out, true)
                           : apply_generic<float, float, double, double>(h, V, ncols, out, true, nullptr);
    if (h->storage == BFGS_BF16 && !f64 && !h->streamed)
        return apply_generic<bf16_t, float, float, float>(h, V, ncols, out, true, nullptr);
    return BFGS_ERR_ARG;
}

int apply_block(bfgsuq_ctx* h, const void* V, int32_t ncols, void* out, bool diff, bool out64,
                const ApplyWs* fixed) {
    if (h->streamed) {
        // staged slices need the handle's own buffers: no fixed workspace
        if (fixed) return BFGS_ERR_STATE;
        if (h->storage == BFGS_F64 && !out64) return apply_streamed<double, double, double>(h, V, ncols, out, diff);
        if (h->storage == BFGS_F32)
            return out64 ? apply_streamed<float, float, double>(h, V, ncols, out, diff)
                         : apply_streamed<float, float, float>(h, V, ncols, out, diff);
        return BFGS_ERR_ARG;
    }
    if (out64) {
        if (h->storage != BFGS_F32) return BFGS_ERR_ARG;
        return apply_generic<float, float, double>(h, V, ncols, out, diff, fixed);
    }
    if (apply_takes_mfma(h, ncols, diff)) return mfma_apply(h, V, ncols, out, diff, fixed);
    switch (h->storage) {
        case BFGS_F64: return apply_generic<double, double, double>(h, V, ncols, out, diff, fixed);
        case BFGS_F32: return apply_generic<float, float, float>(h, V, ncols, out, diff, fixed);
        case BFGS_BF16: return apply_generic<bf16_t, float, float>(h, V, ncols, out, diff, fixed);
    }
    return BFGS_ERR_ARG;
}
