// Single-pass randomized SVD of B_k - B_0 (Alg. 3) and the posterior variance
// of eqs. (10) and (14).
//
//   X = probes (c = rank + oversample columns)
//   E = (B_k - B_0) X                                  apply.hip, "difference" form
//   E = Q R                                            Householder TSQR (tsqr.hip)
//   Omega (Q^T X) = Q^T E = R                          LU with partial pivoting, float64
//   Omega <- (Omega + Omega^T) / 2;  Omega = U_s Lambda U_s^T     tridiagonal divide and conquer, float64
//   U = Q U_s[:, :rank],  Sigma = lambda[:rank],  d = h0 + sum_i lambda_i U_i^2
//
// Q^T E equals R exactly for E = Q R, so the R of the factorisation is used
// instead of a second product with E.  Q^T X and Q U_s run on the float64 matrix
// cores, except for bfloat16 storage, where they run on the bfloat16 matrix cores
// with Q and U_s split into bfloat16 terms (rsvd_bf16.hip).
#include <cmath>
#include <type_traits>
#include <utility>

#include "tall_f64.h"

int probes_launch(bfgsuq_ctx* h, uint64_t seed, int32_t c, void* X, hipStream_t stream);

namespace {

// 1 / sqrt(t) for t > 0, denormal t included (hardware estimate refined by two
// Newton steps).
__device__ __forceinline__ double rsqrt_refined(double t) {
    double y = __builtin_amdgcn_rsq(t);
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const double ty = t * y;
        const double e = fma(-ty, y, 1.0);
        y = fma(0.5 * y, e, y);
    }
    return y;
}

// F = R2 R1 for upper-triangular row-major c x c factors.
__global__ void tri_mul(int c, const double* __restrict__ R2, const double* __restrict__ R1, double* __restrict__ F) {
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < c * c; e += gridDim.x * blockDim.x) {
        const int i = e / c, j = e % c;
        double s = 0.0;
        for (int l = i; l <= j; ++l) s = fma(R2[(int64_t)i * c + l], R1[(int64_t)l * c + j], s);
        F[e] = s;
    }
}

// ---------------------------------------------------------------------------
// Small float64 steps, one workgroup of 256 threads.  Matrices live in global
// memory (at most 256 x 256 doubles, cache resident).
// ---------------------------------------------------------------------------
constexpr int SMALL_THREADS = 256;

template <int NTHR = SMALL_THREADS>
__device__ double wg_sum(double v, double* red) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) red[w] = v;
    __syncthreads();
    double s = 0.0;
    for (int i = 0; i < NTHR / 64; ++i) s += red[i];
    __syncthreads();
    return s;
}

// ---------------------------------------------------------------------------
// Float64 matrix-core products with the tall basis (tall_f64.h).
// ---------------------------------------------------------------------------
constexpr int MT_K = 16;          // rows of a step: chunks are a whole number of them

// Columns of an n x c block, none scaled.
template <typename T>
struct BlockCols {
    const T* base;
    int64_t ld;
    __device__ __forceinline__ TnCol<T> operator()(int j) const { return {base + (int64_t)j * ld, false}; }
};

// part[ch] = Q[rows of chunk ch, :]^T X[rows of chunk ch, :]  (cq x cx, column-major:
// part[j * cq + i] = sum_r Q(r, i) X(r, j)), Q column-major n x cq, X n x cx (both
// leading dimension n).  One wave per (chunk, tile), as tall_f64.h describes, and no more
// than two to a SIMD: 256 chunks of 8 tiles are then one even round, where three to a SIMD
// left others with one (120 x 120 of 360,000 rows, float64 Q and float32 X: 233 us,
// 320 with three, 282 in 128 x 128 tiles through LDS).
template <int TA, int TB, typename TQ, typename TX>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2)))
qtx_mfma(int64_t n, int cq, int cx, const TQ* __restrict__ Q, const TX* __restrict__ X, double* __restrict__ part,
         int64_t rows_per_chunk, int nchunks, int ptiles, int ctiles) {
    int chunk, pos;
    if (!tn_place(blockIdx.x, ptiles * ctiles, nchunks, chunk, pos)) return;
    tn_tile<TA, TB, false, false, TQ, double>(n, cq, cx, chunk, rows_per_chunk, pos % ptiles, pos / ptiles, ctiles,
                                              BlockCols<TQ>{Q, n}, nullptr, X, n, part);
}

template <typename TQ, typename TX>
void launch_qtx(hipStream_t st, int64_t n, int cq, int cx, const TQ* Q, const TX* X, double* part,
                int64_t rows_per_chunk, int nchunks) {
    constexpr bool wide = sizeof(TX) == 8;
    const TnShape s = tn_shape(cq, cx, wide);
    with_tile_width(s.tb, [&](auto tb) {
        constexpr int TB = wide && decltype(tb)::value > TN_WIDE_TB ? TN_WIDE_TB : decltype(tb)::value;
        hipLaunchKernelGGL((qtx_mfma<tile_rows(TB), TB, TQ, TX>), dim3(tn_grid(s.tiles(), nchunks)), dim3(64), 0, st, n,
                           cq, cx, Q, X, part, rows_per_chunk, nchunks, s.ptiles, s.ctiles);
    });
}

// U = Q M (n x rank, column-major, TO) from column-major Q (n x c) and packed M (c x rank);
// with SUB (float64 U) U -= Q M instead.
template <int TA, typename TO, bool SUB>
struct BasisEmit {
    TO* U;
    int64_t n;
    typedef Run<TO, TA> Ahead;
    __device__ __forceinline__ Ahead ahead(int j, int64_t r, int live) const {
        Ahead v{};
        if (SUB) {
            const TO* p = U + (int64_t)j * n + r;
            v = live == TA ? load_run<TO, TA>(p) : load_run_part<TO, TA>(p, live);
        }
        return v;
    }
    __device__ __forceinline__ void store(int j, int64_t r, const double (&o)[TA], const double (&)[TA], const Ahead& v,
                                          int live) const {
        TO* p = U + (int64_t)j * n + r;
        Run<TO, TA> w;
#pragma unroll
        for (int f = 0; f < TA; ++f) w.v[f] = SUB ? (TO)(v.v[f] - (TO)o[f]) : (TO)o[f];
        if (live == TA) {
            *(Run<TO, TA>*)p = w;
        } else {
#pragma unroll
            for (int f = 0; f < TA; ++f)
                if (f < live) p[f] = w.v[f];
        }
    }
};

template <int TA, int TB, typename TQ, typename TO, bool SUB>
__global__ void __launch_bounds__(256, 2) basis_mfma(int64_t n, int c, int rank, const TQ* __restrict__ Q,
                                                     const double* __restrict__ M, TO* __restrict__ U, int ctiles) {
    __shared__ NnLds<TB> lds;
    int64_t row0;
    int ct;
    if (!nn_place(blockIdx.x, n, 64 * TA, ctiles, row0, ct)) return;
    const int cblocks = (rank + 15) / 16, cb = ct * cblocks / ctiles, ce = (ct + 1) * cblocks / ctiles;
    nn_group<TA, TB, false, false, TQ, double>(lds, n, row0, false, c, rank, cblocks, cb, ce - cb, BlockCols<TQ>{Q, n},
                                               nullptr, M, BasisEmit<TA, TO, SUB>{U, n});
}

template <bool SUB, typename TQ, typename TO>
void launch_basis(hipStream_t st, int64_t n, int c, int rank, const TQ* Q, const double* M, TO* U) {
    const NnShape s = nn_shape(rank);
    with_tile_width(s.tb, [&](auto tb) {
        constexpr int TB = decltype(tb)::value;
        hipLaunchKernelGGL((basis_mfma<tile_rows(TB), TB, TQ, TO, SUB>), dim3(nn_grid(n, s)), dim3(256), 0, st, n, c,
                           rank, Q, M, U, s.ctiles);
    });
}

// M (nq x nc, column-major) in the fragment order that nn_group reads.
__global__ void pack_nn(int nq, int nc, const double* __restrict__ M, double* __restrict__ packed) {
    const int cblocks = (nc + 15) / 16, rows = (nq + 3) / 4 * 4;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < rows * nc; e += gridDim.x * blockDim.x) {
        const int q = e % rows, j = e / rows;
        packed[nn_pack_index(q, j, cblocks)] = q < nq ? M[(int64_t)j * nq + q] : 0.0;
    }
}

// Omega = F T^-1, symmetrised.  T column-major c x c (T[j*c + i] = T(i, j)).
// F = R, row-major c x c upper triangular.  M = T^T (row-major M[i*c + j] = T(j, i) =
// T[i*c + j], i.e. the same array), B = F^T; M X = B, Omega = X^T.
//
// Three launches, all chains of small steps whose latency is the cost: lu_factor, a blocked
// right-looking LU of M with partial pivoting in one workgroup; lu_solve, both substitutions,
// a workgroup per 16 columns of B held in LDS; omega_symmetric.  (One workgroup for
// all of it, with the rows swapped in memory one by one: 341 us at c = 120 and 911 at 220,
// now 221 and 489.)
// (value, index) of the largest value over a wave, ties to the lower index, in every
// lane (all lanes active).  Quad and 16-lane row steps by DPP, then the rows by the
// permlane swaps; each swap returns the lane's own pair and its partner's, and both
// are offered (the own one changes nothing).  The order does not matter: the
// selection is associative and commutative.
__device__ __forceinline__ void argmax_take(double& best, int& bi, double v, int i) {
    if (v > best || (v == best && i < bi)) {
        best = v;
        bi = i;
    }
}

template <int CTRL>
__device__ __forceinline__ void argmax_dpp(double& best, int& bi) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, best);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xF, 0xF, false);
    const int i2 = __builtin_amdgcn_update_dpp(0, bi, CTRL, 0xF, 0xF, false);
    argmax_take(best, bi, __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo), i2);
}

template <bool ROWS32>
__device__ __forceinline__ void argmax_swap(double& best, int& bi) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, best);
    const unsigned l0 = (unsigned)u, h0 = (unsigned)(u >> 32), i0 = (unsigned)bi;
    const auto lo = ROWS32 ? __builtin_amdgcn_permlane32_swap(l0, l0, false, false)
                           : __builtin_amdgcn_permlane16_swap(l0, l0, false, false);
    const auto hi = ROWS32 ? __builtin_amdgcn_permlane32_swap(h0, h0, false, false)
                           : __builtin_amdgcn_permlane16_swap(h0, h0, false, false);
    const auto ix = ROWS32 ? __builtin_amdgcn_permlane32_swap(i0, i0, false, false)
                           : __builtin_amdgcn_permlane16_swap(i0, i0, false, false);
#pragma unroll
    for (int t = 0; t < 2; ++t)
        argmax_take(best, bi, __builtin_bit_cast(double, ((unsigned long long)hi[t] << 32) | lo[t]), (int)ix[t]);
}

__device__ __forceinline__ void wave_argmax(double& best, int& bi) {
    argmax_dpp<0xB1>(best, bi);    // quad_perm [1, 0, 3, 2]
    argmax_dpp<0x4E>(best, bi);    // quad_perm [2, 3, 0, 1]
    argmax_dpp<0x124>(best, bi);   // row_ror:4
    argmax_dpp<0x128>(best, bi);   // row_ror:8
    argmax_swap<false>(best, bi);  // rows 0 <-> 1, 2 <-> 3
    argmax_swap<true>(best, bi);   // halves
}

// x combined over the wave, in every lane (all lanes active): quad and 16-lane rows by DPP
// (quad permutations, row rotations by 4 and 8), then the four rows by the permlane swaps,
// which return across their two results each lane's own value and that of the same lane
// in the partner row.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

template <typename Op>
__device__ __forceinline__ double swap16_f64(double x, Op op) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)u, (unsigned)u, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(u >> 32), (unsigned)(u >> 32), false, false);
    return op(__builtin_bit_cast(double, ((unsigned long long)hi[0] << 32) | lo[0]),
              __builtin_bit_cast(double, ((unsigned long long)hi[1] << 32) | lo[1]));
}

template <typename Op>
__device__ __forceinline__ double swap32_f64(double x, Op op) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)u, (unsigned)u, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(u >> 32), (unsigned)(u >> 32), false, false);
    return op(__builtin_bit_cast(double, ((unsigned long long)hi[0] << 32) | lo[0]),
              __builtin_bit_cast(double, ((unsigned long long)hi[1] << 32) | lo[1]));
}

template <typename Op>
__device__ __forceinline__ double wave_reduce_d(double x, Op op) {
    x = op(x, dpp_f64<0xB1>(x));    // quad_perm [1, 0, 3, 2]
    x = op(x, dpp_f64<0x4E>(x));    // quad_perm [2, 3, 0, 1]
    x = op(x, dpp_f64<0x124>(x));   // row_ror:4
    x = op(x, dpp_f64<0x128>(x));   // row_ror:8
    return swap32_f64(swap16_f64(x, op), op);
}

__device__ __forceinline__ double wave_sum_d(double x) {
    return wave_reduce_d(x, [](double a, double b) { return a + b; });
}

constexpr int LU_NB = 16;
constexpr int LU_THREADS = 1024;
constexpr int LU_PLD = LU_NB + 1;        // panel row stride (doubles)
constexpr int LU_ULD = 256 + 1;          // row-block stride: M's right columns
constexpr int LU_TILES = 4;              // tiles of the trailing update that a wave has in flight

size_t lu_smem_bytes() { return ((size_t)256 * LU_PLD + (size_t)LU_NB * LU_ULD) * sizeof(double); }

// M = P^T L U in place: panel by panel, the rows of a panel's L as they lie when it is done
// (later panels swap only what is right of them).  piv[i]: the row that step i swapped with
// row i; from[16 panels][256]: the row before the panel's swaps of each row after them,
// both counted from the panel's first.
//
// A panel's rows are held a thread each and stay there: a swap changes only which row a
// thread stands for (pos).  The step's column is always a[0]; the step shifts the row by
// one and puts the finished entry (the multiplier, or U's where the row was a pivot) at its end,
// so that one copy of the code does for all steps.  One barrier a step: every wave offers its
// largest entry and that row.
__global__ void __launch_bounds__(LU_THREADS) lu_factor(int c, double* __restrict__ M, int* __restrict__ piv,
                                                        uint8_t* __restrict__ from, int32_t* __restrict__ status) {
    extern __shared__ double lu_sh[];
    double* P = lu_sh;                              // panel rows kb..c-1 in their places: P[(r - kb) * LU_PLD + j]
    double* Ub = P + 256 * LU_PLD;                  // row block: Ub[i * LU_ULD + column right of the panel]
    __shared__ double cand[2][4][LU_NB], cand_best[2][4];
    __shared__ int cand_row[2][4];
    __shared__ int src[256], pivl[LU_NB];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    bool bad = false;
    for (int kb = 0; kb < c; kb += LU_NB) {
        const int nb = min(LU_NB, c - kb);
        const int rows = c - kb;
        double a[LU_NB];
        int pos = tid;
        bool active = tid < rows;
#pragma unroll
        for (int j = 0; j < LU_NB; ++j) a[j] = active && j < nb ? M[(int64_t)(kb + tid) * c + kb + j] : 0.0;
        for (int j = 0; j < LU_NB; ++j) {
            double u[LU_NB] = {};
            bool pivot = false;
            if (j < nb) {
                const int buf = j & 1;
                if (wave < 4) {
                    // the largest value (NaN and rows that are done: -1), then the rows that
                    // have it: the lowest of several
                    const double v = active && fabs(a[0]) >= 0.0 ? fabs(a[0]) : -1.0;
                    const double best = wave_reduce_d(v, [](double x, double y) { return fmax(x, y); });
                    bool mine = active && v == best;
                    unsigned long long tied = __ballot(mine);
                    if (__popcll(tied) > 1) {
                        int bi = 256;
                        for (; tied; tied &= tied - 1) bi = min(bi, __shfl(pos, __ffsll(tied) - 1, 64));
                        mine = mine && pos == bi;
                    }
                    if (mine) {
                        cand_row[buf][wave] = pos;
#pragma unroll
                        for (int q = 0; q < LU_NB; ++q) cand[buf][wave][q] = a[q];
                    }
                    if (lane == 0) {
                        cand_best[buf][wave] = best;
                        if (best < 0.0) cand_row[buf][wave] = j;
                    }
                }
                __syncthreads();
                if (wave < 4) {
                    double b4[4];
                    int r4[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        b4[q] = cand_best[buf][q];
                        r4[q] = cand_row[buf][q];
                    }
                    double best = b4[0];
                    int p = r4[0], w = 0;
#pragma unroll
                    for (int q = 1; q < 4; ++q) {
                        const bool take = (b4[q] > best) | ((b4[q] == best) & (r4[q] < p));
                        best = take ? b4[q] : best;
                        p = take ? r4[q] : p;
                        w = take ? q : w;
                    }
#pragma unroll
                    for (int q = 0; q < LU_NB; ++q) u[q] = cand[buf][w][q];
#pragma unroll
                    for (int q = 0; q < LU_NB; ++q) u[q] = q + j < LU_NB ? u[q] : 0.0;
                    if (tid == 0) pivl[j] = p;   // (to memory later: a barrier waits for stores)
                    bad |= !(best > 0.0) || !isfinite(best);
                    pivot = active && pos == p;
                    if (pivot) {
                        pos = j;
                        active = false;
                    } else if (pos == j) {
                        pos = p;
                    }
                }
            }
            if (wave < 4) {
                const double d = u[0];
                const double r = a[0] / d;
                const bool update = active && j < nb;
                const double l = update ? (d != 0.0 ? r : 0.0) : a[0];
#pragma unroll
                for (int q = 1; q < LU_NB; ++q) a[q - 1] = update ? fma(-l, u[q], a[q]) : a[q];
                a[LU_NB - 1] = l;
            }
        }
        if (tid < rows) {
#pragma unroll
            for (int j = 0; j < LU_NB; ++j)
                if (j < nb) {
                    P[pos * LU_PLD + j] = a[j];
                    M[(int64_t)(kb + pos) * c + kb + j] = a[j];
                }
            src[pos] = tid;
            from[kb * 16 + pos] = (uint8_t)tid;
        }
        __syncthreads();
        if (tid < nb) piv[kb + tid] = kb + pivl[tid];
        // swaps and forward substitution of the columns right of the panel, one thread each
        // (there are some only where nb = LU_NB)
        const int right = rows - nb;
        if (tid < right) {
            double* col = M + (int64_t)kb * c + kb + nb + tid;
            double top[LU_NB], low[LU_NB];
            int at[LU_NB];
#pragma unroll
            for (int i = 0; i < LU_NB; ++i) at[i] = pivl[i];
#pragma unroll
            for (int i = 0; i < LU_NB; ++i) {
                top[i] = col[(int64_t)src[i] * c];
                low[i] = col[(int64_t)src[at[i]] * c];
            }
#pragma unroll
            for (int i = 0; i < LU_NB; ++i)
                if (at[i] >= LU_NB) col[(int64_t)at[i] * c] = low[i];
#pragma unroll
            for (int i = 0; i < LU_NB; ++i) {
#pragma unroll
                for (int l = 0; l < i; ++l) top[i] = fma(-P[i * LU_PLD + l], top[l], top[i]);
            }
#pragma unroll
            for (int i = 0; i < LU_NB; ++i) {
                col[(int64_t)i * c] = top[i];
                Ub[i * LU_ULD + tid] = top[i];
            }
        }
        __syncthreads();
        // trailing update of M's rows and columns past the panel: C -= L21 U12, a rank-16
        // product on the float64 matrix cores, one wave per 16 x 16 tile of C
        // (A = L21 rows from the panel, B = U12 from the row block; loads from clamped
        // indices, stores only inside C)
        const int nt = (right + 15) / 16, lm = lane & 15, lk = lane >> 4;
        double* C = M + (int64_t)(kb + nb) * c + kb + nb;
        for (int t0 = wave; t0 < nt * nt; t0 += LU_TILES * (LU_THREADS / 64)) {
            v4d acc[LU_TILES];
            int ti[LU_TILES], tj[LU_TILES];
#pragma unroll
            for (int u = 0; u < LU_TILES; ++u) {
                const int tile = min(t0 + u * (LU_THREADS / 64), nt * nt - 1);
                ti[u] = tile / nt * 16;
                tj[u] = tile % nt * 16;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    acc[u][q] = C[(int64_t)min(ti[u] + lk + 4 * q, right - 1) * c + min(tj[u] + lm, right - 1)];
            }
#pragma unroll
            for (int u = 0; u < LU_TILES; ++u) {
                if (t0 + u * (LU_THREADS / 64) >= nt * nt) break;
                const int ar = min(ti[u] + lm, right - 1), ec = min(tj[u] + lm, right - 1);
#pragma unroll
                for (int ks = 0; ks < LU_NB / 4; ++ks) {
                    const int k = 4 * ks + lk;
                    acc[u] = mfma64(-P[(LU_NB + ar) * LU_PLD + k], Ub[k * LU_ULD + ec], acc[u]);
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int r = ti[u] + lk + 4 * q;
                    if (r < right && tj[u] + lm < right) C[(int64_t)r * c + tj[u] + lm] = acc[u][q];
                }
            }
        }
        __syncthreads();
    }
    if (tid == 0 && bad) set_status(status, BFGS_ERR_NUMERIC);
}

// Columns 16 blockIdx.x .. + 15 of X = M^-1 B, B(i, j) = F(j, i), by the factors, pivots and
// row orders of lu_factor; X column-major.  The columns stay in LDS; a panel's factors
// are fetched into registers before the steps that need them.
__global__ void __launch_bounds__(256) lu_solve(int c, const double* __restrict__ M, const int* __restrict__ piv,
                                                const uint8_t* __restrict__ from, const double* __restrict__ F,
                                                double* __restrict__ X) {
    __shared__ double Bs[256][LU_PLD], Ls[LU_NB][LU_PLD];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, lm = lane & 15, lk = lane >> 4;
    const int j0 = blockIdx.x * 16, i16 = tid >> 4, j16 = tid & 15;
    for (int e = tid; e < 16 * c; e += 256) {
        const int j = e / c, i = e % c;
        Bs[i][j] = j0 + j < c ? F[(int64_t)(j0 + j) * c + i] : 0.0;
    }
    if (c + i16 < (c + 15) / 16 * 16) Bs[c + i16][j16] = 0.0;   // the last panel's missing rows
    __syncthreads();
    // rows r0 .. r0 + rows - 1 of B lose A times the 16 rows at kb: A(r, k) = M(r0 + r, kb + k)
    double lf[4][4];
    auto fetch = [&](int r0, int rows, int kb, int nb) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const int r = (wave + 4 * u) * 16 + lm, k = 4 * ks + lk;
                lf[u][ks] = r < rows && k < nb ? -M[(int64_t)(r0 + r) * c + kb + k] : 0.0;
            }
    };
    auto update = [&](int r0, int rows, int kb, int nb) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int t = (wave + 4 * u) * 16;
            if (t >= rows) break;
            v4d acc;
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] = Bs[r0 + min(t + lk + 4 * q, rows - 1)][lm];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const int k = 4 * ks + lk;
                acc = mfma64(lf[u][ks], k < nb ? Bs[kb + k][lm] : 0.0, acc);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (t + lk + 4 * q < rows) Bs[r0 + t + lk + 4 * q][lm] = acc[q];
        }
    };
    auto diagonal = [&](int kb) {   // the panel's own block of the factors
        const int nb = min(LU_NB, c - kb);
        return i16 < nb && j16 < nb ? M[(int64_t)(kb + i16) * c + kb + j16] : 0.0;
    };
    // forward: each panel's swaps, its unit-lower block, the rows below
    double dg = diagonal(0);
    for (int kb = 0; kb < c; kb += LU_NB) {
        const int nb = min(LU_NB, c - kb), below = c - kb - nb;
        fetch(kb + nb, below, kb, nb);
        const int q = i16 < nb ? piv[kb + i16] - kb : 0;
        const double top = Bs[kb + (i16 < nb ? from[kb * 16 + i16] : 0)][j16], low = Bs[kb + from[kb * 16 + q]][j16];
        Ls[i16][j16] = dg;
        __syncthreads();
        if (i16 < nb) Bs[kb + i16][j16] = top;
        if (q >= nb) Bs[kb + q][j16] = low;
        dg = diagonal(kb + LU_NB < c ? kb + LU_NB : kb);
        __syncthreads();
        if (tid < 16) {
            double x[LU_NB];
#pragma unroll
            for (int i = 0; i < LU_NB; ++i) x[i] = Bs[kb + i][tid];
#pragma unroll
            for (int i = 0; i < LU_NB; ++i) {
#pragma unroll
                for (int l = 0; l < i; ++l) x[i] = fma(-Ls[i][l], x[l], x[i]);
            }
#pragma unroll
            for (int i = 0; i < LU_NB; ++i) Bs[kb + i][tid] = x[i];
        }
        __syncthreads();
        update(kb + nb, below, kb, nb);
        __syncthreads();
    }
    // backward: each panel's upper block from the last, the rows above
    for (int kb = (c - 1) / LU_NB * LU_NB; kb >= 0; kb -= LU_NB) {
        const int nb = min(LU_NB, c - kb);
        fetch(0, kb, kb, nb);
        Ls[i16][j16] = dg;
        dg = diagonal(max(kb - LU_NB, 0));
        __syncthreads();
        if (tid < 16) {
            double x[LU_NB];
#pragma unroll
            for (int i = 0; i < LU_NB; ++i) x[i] = Bs[kb + i][tid];
#pragma unroll
            for (int i = LU_NB - 1; i >= 0; --i) {   // (missing rows: 0, their factors too)
#pragma unroll
                for (int l = i + 1; l < LU_NB; ++l) x[i] = fma(-Ls[i][l], x[l], x[i]);
                const double d = Ls[i][i], v = x[i] / d;
                x[i] = d != 0.0 ? v : 0.0;
            }
#pragma unroll
            for (int i = 0; i < LU_NB; ++i) Bs[kb + i][tid] = x[i];
        }
        __syncthreads();
        update(0, kb, kb, nb);
        __syncthreads();
    }
    for (int e = tid; e < 16 * c; e += 256) {
        const int j = e / c, i = e % c;
        if (j0 + j < c) X[(int64_t)(j0 + j) * c + i] = Bs[i][j];
    }
}

// Omega = X^T, symmetrised: Omega(i, j) = (X(j, i) + X(i, j)) / 2
__global__ void __launch_bounds__(256) omega_symmetric(int c, const double* __restrict__ X, double* __restrict__ Omega,
                                                       int32_t* __restrict__ status) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= c * c) return;
    const int i = e / c, j = e % c;
    const double v = 0.5 * (X[(int64_t)i * c + j] + X[(int64_t)j * c + i]);
    Omega[e] = v;
    if (!isfinite(v)) set_status(status, BFGS_ERR_NUMERIC);
}

// Symmetric eigendecomposition of A (row-major c x c, overwritten):
//   sym_tridiag        Householder tridiagonalisation (one workgroup); reflector kk
//                      (unit first entry, acting on rows kk+1..c-1) is stored
//                      contiguously at V[kk * c + r] with tau in taus[kk]
//   householder_accum  Z = H_0 H_1 ... H_{c-3} explicitly, one wave per column
//   tridiag_dc         eigenpairs of the tridiagonal (d, e) by divide and conquer,
//                      eigenvectors of A = Z times those of the tridiagonal
//                      (tridiag_dc.hip)
// Z: column-major c x c eigenvectors (Z[i*c + r] = component r of vector i).
constexpr int TRI_THREADS = 1024;
constexpr int TRI_LDS_MAX = 191;   // trailing matrices up to this size run from LDS (packed lower triangle)
static_assert(TRI_LDS_MAX <= 193, "LDS-phase rows are covered by three 64-lane passes");

__host__ __device__ constexpr size_t tri_lds_bytes() { return (size_t)TRI_LDS_MAX * (TRI_LDS_MAX + 1) / 2 * 8; }

__device__ __forceinline__ int ptri(int i, int l) { return i * (i + 1) / 2 + l; }   // (i, l), l <= i

// Householder tridiagonalisation.  While the trailing matrix is larger than
// TRI_LDS_MAX the steps work on A in global memory (full symmetric storage); the
// remaining steps work on the packed lower triangle of A[b0:, b0:] in LDS, where
// the rank-2 update touches only the lower triangle.
__global__ void __launch_bounds__(TRI_THREADS) sym_tridiag(int c, double* __restrict__ A, double* __restrict__ V,
                                                             double* __restrict__ dg, double* __restrict__ eg,
                                                             double* __restrict__ taus) {
    extern __shared__ double Tl[];   // packed lower triangle of A[b0:, b0:]
    __shared__ double red[2 * (TRI_THREADS / 64)];
    __shared__ double vsh[256];
    __shared__ double wsh[256];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int NW = TRI_THREADS / 64;
    const int b0 = c > TRI_LDS_MAX ? c - TRI_LDS_MAX : 0;
    for (int kk = 0; kk < b0 && kk + 2 < c; ++kk) {
        const int m = c - kk - 1;   // length of x = A(kk+1:, kk)
        double part = 0.0;
        for (int i = 1 + tid; i < m; i += TRI_THREADS) {
            const double x = A[(int64_t)(kk + 1 + i) * c + kk];
            part = fma(x, x, part);
        }
        const double xn2 = wg_sum<TRI_THREADS>(part, red);
        const double alpha = A[(int64_t)(kk + 1) * c + kk];
        double tau = 0.0, beta = alpha, scale = 0.0;
        if (xn2 > 0.0) {
            beta = -copysign(sqrt(fma(alpha, alpha, xn2)), alpha);
            tau = (beta - alpha) / beta;
            scale = 1.0 / (alpha - beta);
        }
        for (int i = tid; i < m; i += TRI_THREADS) {
            const double v = (i == 0) ? 1.0 : A[(int64_t)(kk + 1 + i) * c + kk] * scale;
            vsh[i] = v;
            V[(int64_t)kk * c + kk + 1 + i] = v;
        }
        __syncthreads();
        if (tid == 0) {
            taus[kk] = tau;
            dg[kk] = A[(int64_t)kk * c + kk];
            eg[kk] = beta;
        }
        if (tau != 0.0) {
            // p = tau * A22 v;  w = p - (tau/2)(p^T v) v;  A22 -= v w^T + w v^T
            // one wave per row, lanes across the row (coalesced), then a wave sum
            // two rows per pass, all loads of a pass first (m <= 255: four per lane and row)
            for (int i0 = wave; i0 < m; i0 += 2 * NW) {
                double sr[2] = {0.0, 0.0};
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const int i = i0 + r * NW;
                    const double* row = A + (int64_t)(kk + 1 + i) * c + (kk + 1);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int l = lane + 64 * u;
                        if (i < m && l < m) sr[r] = fma(row[l], vsh[l], sr[r]);
                    }
                }
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const int i = i0 + r * NW;
                    if (i >= m) break;   // uniform
                    const double p = wave_sum_d(sr[r]);
                    if (lane == 0) wsh[i] = tau * p;
                }
            }
            __syncthreads();
            double pp = 0.0;
            for (int i = tid; i < m; i += TRI_THREADS) pp = fma(wsh[i], vsh[i], pp);
            const double K = 0.5 * tau * wg_sum<TRI_THREADS>(pp, red);
            for (int i = tid; i < m; i += TRI_THREADS) wsh[i] -= K * vsh[i];
            __syncthreads();
            for (int i0 = wave; i0 < m; i0 += 2 * NW) {
                double x[2][4];
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const int i = i0 + r * NW;
                    const double* row = A + (int64_t)(kk + 1 + i) * c + (kk + 1);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int l = lane + 64 * u;
                        x[r][u] = (i < m && l < m) ? row[l] : 0.0;
                    }
                }
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const int i = i0 + r * NW;
                    if (i >= m) break;   // uniform
                    double* row = A + (int64_t)(kk + 1 + i) * c + (kk + 1);
                    const double vi = vsh[i], wi = wsh[i];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int l = lane + 64 * u;
                        if (l < m) row[l] = x[r][u] - (vi * wsh[l] + wi * vsh[l]);
                    }
                }
            }
        }
        __syncthreads();
    }
    // the trailing (c - b0) x (c - b0) matrix moves to LDS
    const int s0 = c - b0;
    for (int e = tid; e < s0 * (s0 + 1) / 2; e += TRI_THREADS) {
        int i = (int)((sqrt(8.0 * e + 1.0) - 1.0) * 0.5);
        while (ptri(i + 1, 0) <= e) ++i;
        while (ptri(i, 0) > e) --i;
        const int l = e - ptri(i, 0);
        Tl[e] = A[(int64_t)(b0 + i) * c + b0 + l];
    }
    __syncthreads();
    // Three barriers per step: (v written) (p and the partials of p^T v written)
    // (A22 updated and the partials of the next column's norm written).  w = p - K v
    // is formed on the fly in the update, whose lane 0 of each row also sums the
    // squares of the next column below its subdiagonal.
    double* red2 = red + NW;
    double xn2 = 0.0;
    if (b0 + 2 < c) {
        const int m = c - b0 - 1;
        double part = 0.0;
        for (int i = 1 + tid; i < m; i += TRI_THREADS) {
            const double x = Tl[ptri(1 + i, 0)];
            part = fma(x, x, part);
        }
        xn2 = wg_sum<TRI_THREADS>(part, red);
    }
    for (int kk = b0; kk + 2 < c; ++kk) {
        const int o = kk - b0;      // local index of the column being eliminated
        const int m = c - kk - 1;
        const double alpha = Tl[ptri(o + 1, o)];
        double tau = 0.0, beta = alpha, scale = 0.0;
        if (xn2 > 0.0) {
            beta = -copysign(sqrt(fma(alpha, alpha, xn2)), alpha);
            tau = (beta - alpha) / beta;
            scale = 1.0 / (alpha - beta);
        }
        for (int i = tid; i < m; i += TRI_THREADS) {
            const double v = (i == 0) ? 1.0 : Tl[ptri(o + 1 + i, o)] * scale;
            vsh[i] = v;
            V[(int64_t)kk * c + kk + 1 + i] = v;
        }
        if (tid == 0) {
            taus[kk] = tau;
            dg[kk] = Tl[ptri(o, o)];
            eg[kk] = beta;
        }
        __syncthreads();
        const int q0 = o + 1;
        if (tau != 0.0) {
            // p_i = tau sum_l A22(i, l) v_l: row i up to the diagonal, then column i below
            // it; each wave also sums p_i v_i over its rows
            double pv = 0.0, vl[3];
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                const int l = lane + 64 * u;
                vl[u] = l < m ? vsh[l] : 0.0;
            }
            for (int i0 = wave; i0 < m; i0 += 2 * NW) {
                double sr[2] = {0.0, 0.0};
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const int i = i0 + r * NW, gi = q0 + i, rbase = ptri(gi, q0);
#pragma unroll
                    for (int u = 0; u < 3; ++u) {
                        const int l = lane + 64 * u;
                        const double aval = (i < m && l < m) ? (l <= i ? Tl[rbase + l] : Tl[ptri(q0 + l, gi)]) : 0.0;
                        sr[r] = fma(aval, vl[u], sr[r]);
                    }
                }
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const int i = i0 + r * NW;
                    if (i >= m) break;   // uniform
                    const double p = tau * wave_sum_d(sr[r]);
                    if (lane == 0) wsh[i] = p;
                    pv = fma(p, vsh[i], pv);
                }
            }
            if (lane == 0) red[wave] = pv;
            __syncthreads();
            double ps = 0.0;
            for (int w = 0; w < NW; ++w) ps += red[w];
            const double K = 0.5 * tau * ps;
            // lower triangle of A22 -= v w^T + w v^T with w = p - K v; two rows per pass,
            // every load of a pass issued before its stores (rows do not overlap, which
            // the compiler cannot see)
            double nrm = 0.0;
            for (int i0 = wave; i0 < m; i0 += 2 * NW) {
                double x[2][3], vl[3], wl[3];
#pragma unroll
                for (int u = 0; u < 3; ++u) {
                    const int l = lane + 64 * u;
                    vl[u] = l < m ? vsh[l] : 0.0;
                    wl[u] = l < m ? fma(-K, vl[u], wsh[l]) : 0.0;
                }
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const int i = i0 + r * NW;
                    const double* row = Tl + ptri(q0 + i, q0);
#pragma unroll
                    for (int u = 0; u < 3; ++u) {
                        const int l = lane + 64 * u;
                        x[r][u] = (i < m && l <= i) ? row[l] : 0.0;
                    }
                }
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const int i = i0 + r * NW;
                    if (i >= m) break;   // uniform
                    double* row = Tl + ptri(q0 + i, q0);
                    const double vi = vsh[i], wi = fma(-K, vi, wsh[i]);
#pragma unroll
                    for (int u = 0; u < 3; ++u) {
                        const int l = lane + 64 * u;
                        if (l <= i) {
                            const double y = x[r][u] - (vi * wl[u] + wi * vl[u]);
                            row[l] = y;
                            if (l == 0 && i >= 2) nrm = fma(y, y, nrm);
                        }
                    }
                }
            }
            if (lane == 0) red2[wave] = nrm;
        } else {
            // A22 unchanged: the next column's norm directly
            double nrm = 0.0;
            for (int i = 2 + wave; i < m; i += NW)
                if (lane == 0) {
                    const double x = Tl[ptri(q0 + i, q0)];
                    nrm = fma(x, x, nrm);
                }
            if (lane == 0) red2[wave] = nrm;
        }
        __syncthreads();
        xn2 = 0.0;
        for (int w = 0; w < NW; ++w) xn2 += red2[w];
    }
    if (tid == 0) {
        if (c >= 2) {
            dg[c - 2] = Tl[ptri(c - 2 - b0, c - 2 - b0)];
            eg[c - 2] = Tl[ptri(c - 1 - b0, c - 2 - b0)];
            taus[c - 2] = 0.0;
        }
        dg[c - 1] = Tl[ptri(c - 1 - b0, c - 1 - b0)];
        eg[c - 1] = 0.0;
    }
}

// Column col of Z = H_0 H_1 ... H_{c-3} e_col: the reflectors are applied to e_col
// from the last to the first.  One wave per column; lane holds rows lane + 64 q.
__global__ void __launch_bounds__(256) householder_accum(int c, const double* __restrict__ V,
                                                         const double* __restrict__ taus, double* __restrict__ Z) {
    const int lane = threadIdx.x & 63;
    const int col = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (col >= c) return;   // uniform per wave
    double z[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) z[q] = (lane + 64 * q == col) ? 1.0 : 0.0;
    // the chain is two dozen instructions a reflector; reflectors are fetched AHEAD steps
    // before they are applied (fetched on demand, each waited for memory: 115 us at c = 220)
    constexpr int AHEAD = 4;
    double v[AHEAD][4], tau[AHEAD];
    auto fetch = [&](double (&x)[4], double& t, int kk) {
        const int k1 = max(kk, 0);
        t = taus[k1];
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = V[(int64_t)k1 * c + min(lane + 64 * q, c - 1)];
    };
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) fetch(v[u], tau[u], c - 3 - u);
    for (int k0 = c - 3; k0 >= 0; k0 -= AHEAD) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const int kk = k0 - u;
            if (kk < 0) break;
            const double t = tau[u];
            double x[4], s = 0.0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = lane + 64 * q;
                x[q] = (r > kk && r < c) ? v[u][q] : 0.0;
                s = fma(x[q], z[q], s);
            }
            fetch(v[u], tau[u], kk - AHEAD);
            s = t * wave_sum_d(s);
            if (t == 0.0) continue;   // uniform: the reflector is the identity
#pragma unroll
            for (int q = 0; q < 4; ++q) z[q] = fma(-s, x[q], z[q]);
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int r = lane + 64 * q;
        if (r < c) Z[(int64_t)col * c + r] = z[q];
    }
}

// Order eigenpairs by |lambda| descending (ties: lambda descending, then index),
// make each eigenvector's largest-magnitude entry positive (lowest index on ties),
// write lam_out (c) and Us (column-major c x c, sorted), and, where packed is given, the
// first `rank` columns in the fragment order that nn_group reads.  One wave per
// eigenvector (one workgroup for all of them took 117 us at c = 220).
__global__ void __launch_bounds__(64) order_sign(int c, int rank, const double* __restrict__ d,
                                                 const double* __restrict__ Z, double* __restrict__ lam_out,
                                                 double* __restrict__ Us, double* __restrict__ packed) {
    const int i = blockIdx.x, lane = threadIdx.x;
    const double li = d[i], ai = fabs(li);
    int before = 0;
    for (int j = lane; j < c; j += 64) {
        if (j == i) continue;
        const double lj = d[j], aj = fabs(lj);
        before += (aj > ai) || (aj == ai && lj > li) || (aj == ai && lj == li && j < i) ? 1 : 0;
    }
    for (int off = 32; off > 0; off >>= 1) before += __shfl_xor(before, off, 64);
    const int o = before;
    const double* zc = Z + (int64_t)i * c;
    double z[4], best = -1.0;
    int arg = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int r = lane + 64 * q;
        z[q] = r < c ? zc[r] : 0.0;
        const double v = fabs(z[q]);
        if (r < c && v > best) {
            best = v;
            arg = r;
        }
    }
    wave_argmax(best, arg);
    const double sg = zc[arg] < 0.0 ? -1.0 : 1.0;
    if (lane == 0) lam_out[o] = li;
    const int cblocks = (rank + 15) / 16;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int r = lane + 64 * q;
        if (r < c) Us[(int64_t)o * c + r] = sg * z[q];
        if (packed && o < rank && r < (c + 3) / 4 * 4) packed[nn_pack_index(r, o, cblocks)] = r < c ? sg * z[q] : 0.0;
    }
}

template <typename TO, typename Th>
__global__ void posterior_diag_kernel(int64_t n, int rank, const TO* __restrict__ U, const double* __restrict__ lam,
                                      const Th* __restrict__ h0, TO* __restrict__ dout, int32_t* __restrict__ status,
                                      int whitened) {
    // whitened basis (B_k = B_0 + B_0^1/2 U Lambda U^T B_0^1/2): d = h0 + h0 sum_i lam_i U_i^2
    bool bad = false;
    for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x) {
        const double hr = to_f64(h0[r]);
        double s = 0.0;
        int i = 0;
        for (; i + 8 <= rank; i += 8) {   // eight in flight, added in order
            TO u[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) u[q] = U[(int64_t)(i + q) * n + r];
#pragma unroll
            for (int q = 0; q < 8; ++q) s = fma(lam[i + q], to_f64(u[q]) * to_f64(u[q]), s);
        }
        for (; i < rank; ++i) {
            const double u = to_f64(U[(int64_t)i * n + r]);
            s = fma(lam[i], u * u, s);
        }
        const TO d = (TO)(whitened ? fma(hr, s, hr) : hr + s);
        bad |= !isfinite(to_f64(d));
        dout[r] = d;
    }
    if (bad) set_status(status, BFGS_ERR_NONFINITE);   // includes overflow of the stored type
}

template <typename TO, typename Th>
__global__ void zero_rsvd(int64_t n, int rank, TO* __restrict__ U, double* __restrict__ Sigma, const Th* __restrict__ h0,
                          TO* __restrict__ dout) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n * rank; e += (int64_t)gridDim.x * blockDim.x)
        U[e] = (TO)0;
    for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x)
        dout[r] = (TO)to_f64(h0[r]);
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < rank; i += blockDim.x) Sigma[i] = 0.0;
}

// ---------------------------------------------------------------------------
// Column-blocked QR of a float64 E (n x c) when c is too wide for a float64 slot:
// E = [E1 E2] with E1 the first c1 columns; E1 = Q1 R11 (TSQR, two passes); E2 is
// projected off Q1 twice (block Gram-Schmidt with reorthogonalisation), R12 the sum
// of the two projections; the remainder = Q2 R22 (TSQR, two passes).  Then
// E = [Q1 Q2] [R11 R12; 0 R22].  Every block has c1, c - c1 <= 128 columns, whose
// slots are float64.
// ---------------------------------------------------------------------------
__global__ void add_into(int64_t count, const double* __restrict__ src, double* __restrict__ dst) {
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (e < count) dst[e] += src[e];
}

// R12 (column-major c1 x c2) += P (column-major c1 x c2) R22 (row-major c2 x c2, upper).
__global__ void add_p_times_r(int c1, int c2, const double* __restrict__ P, const double* __restrict__ R22,
                              double* __restrict__ R12) {
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < c1 * c2; e += gridDim.x * blockDim.x) {
        const int i = e % c1, j = e / c1;
        double s = 0.0;
        for (int l = 0; l <= j; ++l) s = fma(P[(int64_t)l * c1 + i], R22[(int64_t)l * c2 + j], s);
        R12[e] += s;
    }
}

// R (row-major c x c) = [R11 R12; 0 R22]: R11 row-major c1 x c1, R12 column-major c1 x c2,
// R22 row-major c2 x c2.
__global__ void assemble_r(int c, int c1, const double* __restrict__ R11, const double* __restrict__ R12,
                           const double* __restrict__ R22, double* __restrict__ R) {
    const int c2 = c - c1;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < c * c; e += gridDim.x * blockDim.x) {
        const int i = e / c, j = e % c;
        double v = 0.0;
        if (i < c1 && j < c1) v = R11[(int64_t)i * c1 + j];
        else if (i < c1) v = R12[(int64_t)(j - c1) * c1 + i];
        else if (j >= c1) v = R22[(int64_t)(i - c1) * c2 + (j - c1)];
        R[e] = v;
    }
}

// Two TSQR passes over one column block: src (n x cb) -> tmp -> dst; R (row-major cb x cb)
// = R2 R1 into Rout.
int tsqr_twice(bfgsuq_ctx* h, int cb, const double* src, double* tmp, double* dst, double* R1keep, double* Rout) {
    double* R = nullptr;
    int rc;
    if ((rc = tsqr_run(h, cb, src, tmp, &R)) != BFGS_OK) return rc;
    if (hipMemcpyAsync(R1keep, R, (size_t)cb * cb * 8, hipMemcpyDeviceToDevice, h->stream) != hipSuccess)
        return BFGS_ERR_HIP;
    if ((rc = tsqr_run(h, cb, tmp, dst, &R)) != BFGS_OK) return rc;
    hipLaunchKernelGGL(tri_mul, dim3(ceil_div((int64_t)cb * cb, 256)), dim3(256), 0, h->stream, cb, R, R1keep, Rout);
    return hipGetLastError() == hipSuccess ? BFGS_OK : BFGS_ERR_HIP;
}

int qr_two_blocks(bfgsuq_ctx* h, int c, double* E, double* Q, int nchunks, int64_t rows_per_chunk, double* part,
                  double* Rb, double* Rout) {
    const int64_t n = h->n;
    const int c1 = (int)std::min<int64_t>(128, round_up((c + 1) / 2, 16));
    const int c2 = c - c1;
    if (c2 < 1 || c2 > 128) return BFGS_ERR_ARG;
    int rc;
    if ((rc = ensure_ws(h->W, (size_t)n * c1 * 8)) != BFGS_OK) return rc;
    double* W = (double*)h->W.ptr;
    const size_t cc = (size_t)c * c;
    double* R11 = Rb;
    double* R12 = Rb + cc;
    double* R22 = Rb + 2 * cc;
    double* Rk = Rb + 3 * cc;   // first-pass R of a block, then one projection
    double* E2 = E + (int64_t)c1 * n;
    double* Q2 = Q + (int64_t)c1 * n;
    if ((rc = tsqr_twice(h, c1, E, W, Q, Rk, R11)) != BFGS_OK) return rc;
    const int64_t cnt = (int64_t)c1 * c2;
    for (int pass = 0; pass < 2; ++pass) {
        launch_qtx(h->stream, n, c1, c2, (const double*)Q, (const double*)E2, part, rows_per_chunk, nchunks);
        double* dst = pass == 0 ? R12 : Rk;
        if ((rc = sum_partials(h->stream, cnt, nchunks, part, dst, true)) != BFGS_OK) return rc;
        hipLaunchKernelGGL(pack_nn, dim3(64), dim3(256), 0, h->stream, c1, c2, dst, part);   // the partials are summed
        launch_basis<true>(h->stream, n, c1, c2, (const double*)Q, part, E2);
        if (pass == 1) hipLaunchKernelGGL(add_into, dim3(ceil_div(cnt, 256)), dim3(256), 0, h->stream, cnt, Rk, R12);
    }
    if ((rc = tsqr_twice(h, c2, E2, W, Q2, Rk, R22)) != BFGS_OK) return rc;
    // Where E2 lies in span(Q1) its remainder is rounding noise, which is not orthogonal
    // to Q1, and neither are the columns of Q2 it yields: project Q2 off Q1 once more and
    // refactor it.  Q2 = Q1 P + Q2', Q2' = Q2'' R'', so E2 = Q1 (R12 + P R22) + Q2'' (R'' R22).
    double* P = Rk;
    double* Rn = Rb + 4 * cc;
    double* Rn1 = Rb + 5 * cc;
    launch_qtx(h->stream, n, c1, c2, (const double*)Q, (const double*)Q2, part, rows_per_chunk, nchunks);
    if ((rc = sum_partials(h->stream, cnt, nchunks, part, P, true)) != BFGS_OK) return rc;
    hipLaunchKernelGGL(pack_nn, dim3(64), dim3(256), 0, h->stream, c1, c2, P, part);
    launch_basis<true>(h->stream, n, c1, c2, (const double*)Q, part, Q2);
    hipLaunchKernelGGL(add_p_times_r, dim3(ceil_div(cnt, 256)), dim3(256), 0, h->stream, c1, c2, P, R22, R12);
    if ((rc = tsqr_twice(h, c2, Q2, W, Q2, Rn1, Rn)) != BFGS_OK) return rc;
    hipLaunchKernelGGL(tri_mul, dim3(ceil_div((int64_t)c2 * c2, 256)), dim3(256), 0, h->stream, c2, Rn, R22, Rn1);
    R22 = Rn1;
    hipLaunchKernelGGL(assemble_r, dim3(ceil_div((int64_t)cc, 256)), dim3(256), 0, h->stream, c, c1, R11, R12, R22,
                       Rout);
    return hipGetLastError() == hipSuccess ? BFGS_OK : BFGS_ERR_HIP;
}

// Row scaling by h0^(p/2), p = +1 or -1 (the whitening of the preconditioned variant):
// in place, or into a copy.
template <typename T, typename Th>
__global__ void scale_rows_kernel(int64_t n, int c, const Th* __restrict__ h0, int p, const T* __restrict__ in,
                                  T* __restrict__ out) {
    const int64_t total = n * c;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const double hr = to_f64(h0[e % n]);
        const double w = p > 0 ? sqrt(hr) : 1.0 / sqrt(hr);
        out[e] = (T)(w * to_f64(in[e]));
    }
}

template <typename T>
void scale_rows_copy(bfgsuq_ctx* h, int c, const T* in, T* out, int p) {
    const int g = (int)std::min<int64_t>(8192, (h->n * c + 255) / 256);
    if (h->storage == BFGS_F64)
        hipLaunchKernelGGL((scale_rows_kernel<T, double>), dim3(g), dim3(256), 0, h->stream, h->n, c,
                           (const double*)h->h0, p, in, out);
    else
        hipLaunchKernelGGL((scale_rows_kernel<T, float>), dim3(g), dim3(256), 0, h->stream, h->n, c,
                           (const float*)h->h0, p, in, out);
}

template <typename T>
void scale_rows_launch(bfgsuq_ctx* h, int c, T* x, int p) {
    scale_rows_copy<T>(h, c, x, x, p);
}

// Omega = (M + M^T) / 2, column-major c x c.
__global__ void symmetrise(int c, const double* __restrict__ M, double* __restrict__ Om) {
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < c * c; e += gridDim.x * blockDim.x) {
        const int i = e % c, j = e / c;
        Om[e] = 0.5 * (M[(int64_t)j * c + i] + M[(int64_t)i * c + j]);
    }
}

// ---------------------------------------------------------------------------
// Host driver
// ---------------------------------------------------------------------------
template <typename TS, typename TO, typename Th>
int rsvd_impl(bfgsuq_ctx* h, int rank, int oversample, uint64_t seed, TO* U, double* Sigma, uint32_t flags) {
    const bool precond = (flags & BFGS_RSVD_PRECOND) != 0;
    const bool two_pass = (flags & BFGS_RSVD_TWO_PASS) != 0;
    const int64_t n = h->n;
    const int c = rank + oversample;
    int rc;
    if ((rc = ensure_ws(h->diag, (size_t)n * sizeof(TO))) != BFGS_OK) return rc;
    TO* dout = (TO*)h->diag.ptr;
    if (h->k == 0) {
        hipLaunchKernelGGL((zero_rsvd<TO, Th>), dim3(1024), dim3(256), 0, h->stream, n, rank, U, Sigma,
                           (const Th*)h->h0, dout);
        if (hipGetLastError() != hipSuccess) return BFGS_ERR_HIP;
        h->have_rsvd = true;
        h->last_rank = rank;
        return BFGS_OK;
    }
    if ((rc = ensure_ws(h->X, (size_t)n * c * sizeof(TS))) != BFGS_OK) return rc;
    // E = (B_k - B_0) X: float64 for float32 storage, whose Sigma would otherwise carry the
    // float32 rounding of E amplified by the Omega solve (about 6e-7 relative to Sigma_0
    // on the 1700 x 350 x 3 grid with k = 200, c = 220, against a 1e-6 budget)
    // and so is Q: rounding Q to float32 perturbs E = Q R by the same relative amount,
    // and with Q^T X built from the rounded Q the Omega solve amplifies it by cond(Q^T X)
    constexpr bool e64 = std::is_same<TS, float>::value;
    using TE = typename std::conditional<e64, double, TO>::type;
    using TQ = TE;
    if ((rc = ensure_ws(h->E, (size_t)n * c * sizeof(TE))) != BFGS_OK) return rc;
    // bfloat16 storage: Q chain-blocked (each TSQR chain's rows one contiguous block),
    // which the projection and the basis read without a translation miss per column;
    // the whitened and two-pass forms pass Q to column-major kernels and keep it so
    constexpr bool bf16_path = std::is_same<TS, bf16_t>::value;
    const bool qblk = bf16_path && !precond && !two_pass;
    const int64_t qb_rows = qblk ? tsqr_chain_rows(h) : 0;
    const int64_t q_rows = qblk ? ceil_div(n, qb_rows) * qb_rows : n;
    if ((rc = ensure_ws(h->Q, (size_t)q_rows * c * sizeof(TQ))) != BFGS_OK) return rc;
    // small: part(nchunks*c*c) + T, M, B, Omega, Z (5 c*c) + d, e, taus, rot, lam (5 c) + piv, from
    // Q^T X row chunks: about one per CU, each chunk a multiple of the staging depth
    int nchunks = (int)std::min<int64_t>(256, std::max<int64_t>(1, (n + 63) / 64));
    const int64_t rows_per_chunk = round_up((n + nchunks - 1) / nchunks, MT_K);
    nchunks = (int)((n + rows_per_chunk - 1) / rows_per_chunk);
    // a blocked Q is projected one chain block per chunk
    const int qx_chunks = qblk ? (int)ceil_div(n, qb_rows) : nchunks;
    const int part_chunks = std::max(nchunks, qx_chunks);
    const size_t cc = (size_t)c * c;
    if ((rc = ensure_ws(h->small, ((size_t)part_chunks * cc + 14 * cc + nn_pack_doubles(c, rank) + 6 * (size_t)c) * 8 +
                                      (size_t)c * 4 + 16 * 256)) !=
        BFGS_OK)
        return rc;
    // tridiagonal eigensolver workspace, then Z = Q_H Y (c x c)
    const size_t ush_bytes = bf16_path ? basis_bf16_workspace(c, rank) : 0;
    const size_t ush_off = round_up((int64_t)(tridiag_dc_workspace(c) + cc * sizeof(double)), 256);
    if ((rc = ensure_ws(h->lam, ush_off + ush_bytes)) != BFGS_OK) return rc;
    double* dcwork = (double*)h->lam.ptr;
    double* Zt = dcwork + tridiag_dc_workspace(c) / sizeof(double);
    uint16_t* ush = (uint16_t*)((char*)h->lam.ptr + ush_off);   // 16-byte fragment loads
    double* part = (double*)h->small.ptr;
    double* Tm = part + (size_t)part_chunks * cc;
    double* Bm = Tm + cc;
    double* Om = Bm + cc;
    double* Zm = Om + cc;
    double* Usm = Zm + cc;
    double* dv = Usm + cc;
    double* ev = dv + c;
    double* tv = ev + c;
    double* rot = tv + c;
    double* lam = rot + 2 * (size_t)c;
    double* R1c = lam + c;
    double* Fm = R1c + cc;
    double* Rb = Fm + cc;   // 6 c x c: the column-blocked QR's pieces
    double* Mpk = Rb + 6 * cc;   // the basis' small operand, packed
    int* piv = (int*)(Mpk + nn_pack_doubles(c, rank));
    uint8_t* from = (uint8_t*)(piv + c);   // 16 panels of 256 rows
    TS* X = (TS*)h->X.ptr;
    TE* E = (TE*)h->E.ptr;
    TQ* Q = (TQ*)h->Q.ptr;

    {
        ProfScope ps(h, "probes");
        if ((rc = probes_launch(h, seed, c, X, h->stream)) != BFGS_OK) return rc;
    }
    if ((rc = apply_block(h, X, c, E, true, e64)) != BFGS_OK) return rc;
    // whitened operator B_0^-1/2 (B_k - B_0) B_0^-1/2: its sketch of X_w = B_0^1/2 X is
    // B_0^-1/2 E
    if (precond) scale_rows_launch(h, c, E, -1);
    double* R = nullptr;
    if constexpr (std::is_same<TE, double>::value) {
        if (tsqr_f64_slot(c)) {
            // E kept in float64 (float64 or float32 storage) is exactly rank deficient at
            // its noise level, and the zero-started slot then keeps part of Q.  A second
            // pass over the (well conditioned) Q restores orthonormality: E = Q2 (R2 R1).
            if ((rc = tsqr_run(h, c, E, Q, &R)) != BFGS_OK) return rc;
            if (hipMemcpyAsync(R1c, R, cc * 8, hipMemcpyDeviceToDevice, h->stream) != hipSuccess) return BFGS_ERR_HIP;
            TQ* Q2 = reinterpret_cast<TQ*>(E);   // E is free now and as large as Q
            if ((rc = tsqr_run(h, c, Q, Q2, &R)) != BFGS_OK) return rc;
            hipLaunchKernelGGL(tri_mul, dim3(ceil_div((int64_t)cc, 256)), dim3(256), 0, h->stream, c, R, R1c, Fm);
            Q = Q2;
            R = Fm;
        } else {
            // wider than a float64 slot fits in LDS: two column blocks, each with a float64
            // slot (a float32 slot would round R at every fold)
            if ((rc = qr_two_blocks(h, c, E, Q, nchunks, rows_per_chunk, part, Rb, Fm)) != BFGS_OK) return rc;
            R = Fm;
        }
    } else {
        if constexpr (bf16_path) {
            if ((rc = tsqr_run(h, c, E, Q, &R, qblk)) != BFGS_OK) return rc;
        } else {
            if ((rc = tsqr_run(h, c, E, Q, &R)) != BFGS_OK) return rc;
        }
    }
    // the E / Q buffer that Q does not occupy is free now
    TE* Efree = (void*)Q == h->E.ptr ? (TE*)h->Q.ptr : E;
    if (two_pass) {
        // Halko et al.'s two-pass form: apply the operator to Q itself, Omega = Q^T (A Q)
        ProfScope ps(h, "two_pass_AQ");
        const TQ* V2 = Q;
        if (precond) {
            if ((rc = ensure_ws(h->W, (size_t)n * c * sizeof(TQ))) != BFGS_OK) return rc;
            TQ* Qs = (TQ*)h->W.ptr;
            scale_rows_copy(h, c, Q, Qs, -1);
            V2 = Qs;
        }
        if ((rc = apply_diff_float_block(h, V2, sizeof(TQ) == 8, c, Efree)) != BFGS_OK) return rc;
        if (precond) scale_rows_launch(h, c, Efree, -1);
        launch_qtx(h->stream, n, c, c, (const TQ*)Q, (const TE*)Efree, part, rows_per_chunk, nchunks);
        if ((rc = sum_partials(h->stream, (int64_t)cc, nchunks, part, Tm, true)) != BFGS_OK) return rc;
        hipLaunchKernelGGL(symmetrise, dim3(ceil_div((int64_t)cc, 256)), dim3(256), 0, h->stream, c, Tm, Om);
    } else {
        ProfScope ps(h, "proj_QtX");
        const TQ* Qp = Q;
        if (precond) {
            // T = Q^T X_w = (B_0^1/2 Q)^T X
            if ((rc = ensure_ws(h->W, (size_t)n * c * sizeof(TQ))) != BFGS_OK) return rc;
            TQ* Qs = (TQ*)h->W.ptr;
            scale_rows_copy(h, c, Q, Qs, +1);
            Qp = Qs;
        }
        if constexpr (bf16_path) {
            if ((rc = qtx_bf16_launch(h->stream, n, c, Qp, X, part, qx_chunks, qblk ? qb_rows : rows_per_chunk,
                                      qb_rows)) != BFGS_OK)
                return rc;
        } else {
            launch_qtx(h->stream, n, c, c, Qp, (const TS*)X, part, rows_per_chunk, nchunks);
        }
        if ((rc = sum_partials(h->stream, (int64_t)cc, bf16_path ? qx_chunks : nchunks, part, Tm, true)) != BFGS_OK)
            return rc;
    }
    if (!two_pass) {
        ProfScope ps(h, "omega_lu");
        static bool attr = false;
        if (!attr) {
            if (hipFuncSetAttribute((const void*)lu_factor, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)lu_smem_bytes()) != hipSuccess)
                return BFGS_ERR_HIP;
            attr = true;
        }
        hipLaunchKernelGGL(lu_factor, dim3(1), dim3(LU_THREADS), lu_smem_bytes(), h->stream, c, Tm, piv, from, h->status);
        hipLaunchKernelGGL(lu_solve, dim3(ceil_div(c, 16)), dim3(256), 0, h->stream, c, Tm, piv, from, R, Bm);
        hipLaunchKernelGGL(omega_symmetric, dim3(ceil_div((int64_t)cc, 256)), dim3(256), 0, h->stream, c, Bm, Om,
                           h->status);
    }
    prof_begin(h, "sym_eig");
    // Bm (X) is free after omega_symmetric: it holds the reflectors
    {
        static bool attr = false;
        if (!attr) {
            if (hipFuncSetAttribute((const void*)sym_tridiag, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)tri_lds_bytes()) != hipSuccess)
                return BFGS_ERR_HIP;
            attr = true;
        }
        hipLaunchKernelGGL(sym_tridiag, dim3(1), dim3(TRI_THREADS), tri_lds_bytes(), h->stream, c, Om, Bm, dv, ev, tv);
    }
    hipLaunchKernelGGL(householder_accum, dim3(ceil_div(c, 4)), dim3(256), 0, h->stream, c, Bm, tv, Zm);
    double* wv = nullptr;
    if ((rc = tridiag_dc(h->stream, c, dv, ev, Zm, dcwork, &wv, Zt, h->status)) != BFGS_OK) return rc;
    hipLaunchKernelGGL(order_sign, dim3(c), dim3(64), 0, h->stream, c, rank, wv, Zt, lam, Usm,
                       bf16_path ? nullptr : Mpk);
    if (hipMemcpyAsync(Sigma, lam, (size_t)rank * 8, hipMemcpyDeviceToDevice, h->stream) != hipSuccess)
        return BFGS_ERR_HIP;
    prof_end(h);
    prof_begin(h, "basis_diag");
    if constexpr (bf16_path) {
        // the posterior diagonal is formed in the same pass
        if ((rc = basis_bf16_launch(h->stream, n, c, rank, Q, Usm, ush, lam, (const float*)h->h0, U, dout,
                                    h->status, precond, qb_rows)) != BFGS_OK)
            return rc;
    } else {
        launch_basis<false>(h->stream, n, c, rank, (const TQ*)Q, (const double*)Mpk, U);
        const int g = (int)std::min<int64_t>(4096, (n + 255) / 256);
        hipLaunchKernelGGL((posterior_diag_kernel<TO, Th>), dim3(g), dim3(256), 0, h->stream, n, rank, U, lam,
                           (const Th*)h->h0, dout, h->status, precond ? 1 : 0);
    }
    prof_end(h);
    if (hipGetLastError() != hipSuccess) return BFGS_ERR_HIP;
    h->have_rsvd = true;
    h->last_rank = rank;
    return BFGS_OK;
}

}  // namespace

int rsvd_run(bfgsuq_ctx* h, int32_t rank, int32_t oversample, uint64_t seed, void* U, double* Sigma, uint32_t flags) {
    switch (h->storage) {
        case BFGS_F64: return rsvd_impl<double, double, double>(h, rank, oversample, seed, (double*)U, Sigma, flags);
        case BFGS_F32: return rsvd_impl<float, float, float>(h, rank, oversample, seed, (float*)U, Sigma, flags);
        case BFGS_BF16: return rsvd_impl<bf16_t, float, float>(h, rank, oversample, seed, (float*)U, Sigma, flags);
    }
    return BFGS_ERR_ARG;
}
