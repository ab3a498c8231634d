// Both passes of the float64 apply for a few columns (c <= STREAM_COLS), on the vector
// unit.  They read S and Y once each and do 2 c float64 multiply-adds per entry, so memory
// bounds them; the matrix-core tiles of tall_f64.h would multiply 16 columns.  Measured at
// n = 360,000, k = 100, one float32 column (0.29 GB of pairs a pass): 46 and
// 47 us (6.2 TB/s), 75 and 69 us with the tiles.
#pragma once

#include <algorithm>

#include "tall_f64.h"

constexpr int STREAM_COLS = 4;
constexpr int STREAM_PAIRS = 8;   // pairs a wave of pass 1 takes at a time

// Calls f(std::integral_constant<int, CC>) for up to STREAM_COLS columns (1, 2 or 4 of them
// computed).
template <typename F>
__host__ __device__ __forceinline__ void with_few_columns(int c, F&& f) {
    if (c == 1) f(std::integral_constant<int, 1>());
    else if (c == 2) f(std::integral_constant<int, 2>());
    else f(std::integral_constant<int, STREAM_COLS>());
}

// Row chunks of pass 1: as many as keep 16 waves a CU busy, of at least 1024 rows, so that the
// sum of the partials stays short; a single chunk writes Z itself.
struct StreamPlan {
    int groups, nchunks;
    int64_t rows_per_chunk;
};
inline StreamPlan stream_plan(int64_t n, int k, int64_t most = 1 << 20) {
    const int groups = ceil_div(k, STREAM_PAIRS);
    int64_t nch = std::min<int64_t>(8 * std::max(1, 512 / (2 * groups)), (n + 1023) / 1024);
    nch = std::min(nch, most);
    const int64_t rows = round_up((n + nch - 1) / nch, 256);
    return {groups, (int)((n + rows - 1) / rows), rows};
}
// Bytes of the partial sums, enough for any number of pairs and columns here: at most 1 MB
// (8 * 256 / groups chunks of 16 groups sums), so that a handle that gains pairs between its
// calls, as an optimizer's does, never replaces them (which would wait for the device).  None
// where n is one chunk for any number of pairs.
inline size_t stream_part_bytes(int64_t n, int kmax) {
    if (n <= 1024) return 0;
    return (size_t)std::min<int64_t>(8 * 256 * 16, (n + 1023) / 1024 * 2 * kmax) * STREAM_COLS * 8;
}

// Consecutive rows a lane loads at a time: 16 bytes of the pairs' type.
template <typename T>
constexpr int stream_rows() {
    return sizeof(T) == 8 ? 2 : 4;
}

// Sums of E values over the wave's lanes (E a power of two up to 64): lane l is left with
// that of value l / (64 / E).  Each step halves the values a lane still carries, so 32
// sums cost 32 exchanges (192 one at a time, 7 of pass 1's 13 us where it has nothing to read).
template <int LEFT, int OFF, int E>
__device__ __forceinline__ double stream_wave_sums(double (&a)[E]) {
    if constexpr (OFF == 0) {
        return a[0];
    } else if constexpr (LEFT > 1) {
        const bool up = threadIdx.x & OFF;
#pragma unroll
        for (int i = 0; i < LEFT / 2; ++i) {
            const double mine = up ? a[i + LEFT / 2] : a[i], other = up ? a[i] : a[i + LEFT / 2];
            a[i] = mine + __shfl_xor(other, OFF, 64);
        }
        return stream_wave_sums<LEFT / 2, OFF / 2>(a);
    } else {
        a[0] += __shfl_xor(a[0], OFF, 64);
        return stream_wave_sums<1, OFF / 2>(a);
    }
}

// Pass 1: part[chunk][j * 2k + p] = sum over the chunk's rows of W(r, p) V(r, j).  A
// workgroup is one wave: STREAM_PAIRS columns of S or of Y over one chunk, the sums kept in
// registers, V (and h0 for Y) read again by each group of pairs, from L2.
template <int CC, typename Ts, typename Th, typename Tv>
__device__ __forceinline__ void stream_chunk(int64_t n, int64_t ld, int k, int c, const Ts* __restrict__ S,
                                             const Ts* __restrict__ Y, const Th* __restrict__ h0,
                                             const Tv* __restrict__ V, double* __restrict__ part,
                                             int64_t rows_per_chunk, int groups, int chunk, int pos) {
    constexpr int VR = stream_rows<Ts>();
    const bool y = pos >= groups;
    const int p0 = (y ? pos - groups : pos) * STREAM_PAIRS;
    const int lane = threadIdx.x;
    const int64_t rb = (int64_t)chunk * rows_per_chunk, re = min(n, rb + rows_per_chunk);
    const Ts* W = y ? Y : S;
    double acc[STREAM_PAIRS * CC] = {};
    for (int64_t r0 = rb; r0 < re; r0 += 64 * VR) {
        const int64_t r = r0 + VR * lane;
        const int live = (int)max((int64_t)0, min((int64_t)VR, re - r));
        Run<Ts, VR> w[STREAM_PAIRS];
        Run<Tv, VR> v[CC];
        Run<Th, VR> h;
        if (r0 + 64 * VR <= re) {
#pragma unroll
            for (int u = 0; u < STREAM_PAIRS; ++u) w[u] = load_run<Ts, VR>(W + (int64_t)min(p0 + u, k - 1) * ld + r);
#pragma unroll
            for (int j = 0; j < CC; ++j) v[j] = load_run<Tv, VR>(V + (int64_t)min(j, c - 1) * n + r);
            if (y) h = load_run<Th, VR>(h0 + r);
        } else {
            const int64_t rl = live > 0 ? r : rb;   // a row that exists
#pragma unroll
            for (int u = 0; u < STREAM_PAIRS; ++u)
                w[u] = load_run_part<Ts, VR>(W + (int64_t)min(p0 + u, k - 1) * ld + rl, live);
#pragma unroll
            for (int j = 0; j < CC; ++j) v[j] = load_run_part<Tv, VR>(V + (int64_t)min(j, c - 1) * n + rl, live);
            if (y) h = load_run_part<Th, VR>(h0 + rl, live);
        }
#pragma unroll
        for (int e = 0; e < VR; ++e) {
            double x[CC];
#pragma unroll
            for (int j = 0; j < CC; ++j) {
                x[j] = to_f64(v[j].v[e]);
                if (y) x[j] *= to_f64(h.v[e]);
            }
#pragma unroll
            for (int u = 0; u < STREAM_PAIRS; ++u) {
                const double we = to_f64(w[u].v[e]);
#pragma unroll
                for (int j = 0; j < CC; ++j) acc[u * CC + j] = fma(we, x[j], acc[u * CC + j]);
            }
        }
    }
    double* dst = part + (int64_t)chunk * 2 * k * c + (y ? k : 0);
    constexpr int LANES = 64 / (STREAM_PAIRS * CC);   // to a sum
    const double s = stream_wave_sums<STREAM_PAIRS * CC, 32>(acc);
    const int u = lane / LANES / CC, j = lane / LANES % CC;
    if (lane % LANES == 0 && p0 + u < k && j < c) dst[(int64_t)j * 2 * k + p0 + u] = s;
}

template <int CC, typename Ts, typename Th, typename Tv>
__global__ void __launch_bounds__(64, CC > 2 ? 2 : 4) stream_pass1(int64_t n, int64_t ld, int k, int c, const Ts* __restrict__ S,
                                                      const Ts* __restrict__ Y, const Th* __restrict__ h0,
                                                      const Tv* __restrict__ V, double* __restrict__ part,
                                                      int64_t rows_per_chunk, int nchunks, int groups) {
    int chunk, pos;
    if (tn_place(blockIdx.x, 2 * groups, nchunks, chunk, pos))
        stream_chunk<CC, Ts, Th, Tv>(n, ld, k, c, S, Y, h0, V, part, rows_per_chunk, groups, chunk, pos);
}

// Pass 2: out = h0 o (V - Y P) + S T (without h0 o V for B_k - B_0); P, T column-major k x c.
// A workgroup's four waves share its rows: two take a half of S's columns each, two a
// half of Y's, and their sums meet in LDS.
template <int CC, typename Ts>
struct StreamLds {
    double sums[4][CC][64 * stream_rows<Ts>()];
};

template <int CC, typename Ts, typename Th, typename To, typename Tv>
__device__ __forceinline__ void stream_block(StreamLds<CC, Ts>& lds, int64_t n, int64_t ld, int k, int c,
                                             const Ts* __restrict__ S, const Ts* __restrict__ Y,
                                             const Th* __restrict__ h0, const Tv* __restrict__ V,
                                             const double* __restrict__ P, const double* __restrict__ T,
                                             To* __restrict__ out, int diff, int block) {
    constexpr int VR = stream_rows<Ts>(), ROWS = 64 * VR, DEPTH = 8;
    auto& sums = lds.sums;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t row0 = (int64_t)block * ROWS;
    {
        const Ts* W = (wave < 2 ? S : Y) + row0 + VR * lane;   // columns are ld (a multiple of 128) rows long
        const double* M = wave < 2 ? T : P;
        const int q0 = wave % 2 ? k / 2 : 0, q1 = wave % 2 ? k : k / 2;
        const bool there = row0 + VR * lane < n;               // then the whole run is within ld
        double acc[VR][CC] = {};
        for (int q = q0; q < q1; q += DEPTH) {
            Run<Ts, VR> w[DEPTH];
#pragma unroll
            for (int u = 0; u < DEPTH; ++u)
                w[u] = there ? load_run<Ts, VR>(W + (int64_t)min(q + u, q1 - 1) * ld) : Run<Ts, VR>{};
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) {
                if (q + u >= q1) break;
#pragma unroll
                for (int j = 0; j < CC; ++j) {
                    const double m = M[(int64_t)min(j, c - 1) * k + q + u];
#pragma unroll
                    for (int e = 0; e < VR; ++e) acc[e][j] = fma(to_f64(w[u].v[e]), m, acc[e][j]);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < CC; ++j)
#pragma unroll
            for (int e = 0; e < VR; ++e) sums[wave][j][VR * lane + e] = acc[e][j];
    }
    __syncthreads();
    for (int t = threadIdx.x; t < CC * ROWS; t += 256) {
        const int j = t / ROWS, i = t % ROWS;
        const int64_t r = row0 + i;
        if (j >= c || r >= n) continue;
        const double h = to_f64(h0[r]), v = diff ? 0.0 : to_f64(V[(int64_t)j * n + r]);
        out[(int64_t)j * n + r] = (To)fma(h, v - (sums[2][j][i] + sums[3][j][i]), sums[0][j][i] + sums[1][j][i]);
    }
}

template <int CC, typename Ts, typename Th, typename To, typename Tv>
__global__ void __launch_bounds__(256) stream_pass2(int64_t n, int64_t ld, int k, int c, const Ts* __restrict__ S,
                                                    const Ts* __restrict__ Y, const Th* __restrict__ h0,
                                                    const Tv* __restrict__ V, const double* __restrict__ P,
                                                    const double* __restrict__ T, To* __restrict__ out, int diff) {
    __shared__ StreamLds<CC, Ts> lds;
    stream_block<CC, Ts, Th, To, Tv>(lds, n, ld, k, c, S, Y, h0, V, P, T, out, diff, blockIdx.x);
}
