// Tall-skinny products on the float64 matrix cores (v_mfma_f64_16x16x4f64), shared by
// the float32/float64 apply and the rSVD:
//   tn:  D(p, j)   = sum_r W(r, p) V(r, j)     contraction over the n rows
//   nn:  out(r, j) = sum_q W(r, q) M(q, j)     contraction over the pairs or basis columns
// W, V and out are column-major; values are widened to float64 as they are loaded.
//
// Fragment layout of one 16 x 16 x 4 product: lane l holds A(l % 16, l / 16),
// B(l / 16, l % 16), and C(l / 16 + 4 r, l % 16) in accumulator element r.  In both
// products A carries the column block (V, M), B the wide operand (W), so that a lane's
// results share one pair (tn) or one row (nn).
//
// What bounds them: the matrix cores (one product takes 64 cycles of a SIMD), as long as
// their operands arrive in time.  So a wave loads its share of W (and of V) straight from
// global memory into fragments, the next 16 rows or 16 pairs in flight, and L1 and L2 serve
// the repeats; a tile is TA x TB blocks of 16, not a padded 128 x 128.  Measured at
// n = 1.785M, k = 200, c = 220, float32: pass 1 5.9 ms
// (54 TFLOP/s of 72 that a float64 library product reaches), pass 2 5.4 ms (59 TFLOP/s);
// the 128 x 128 tiles staged through LDS between barriers took 8.1 and 10.3 ms.
#pragma once

#include <type_traits>

#include "common.h"

typedef double v4d __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v4d mfma64(double a, double b, v4d c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// N consecutive values at any element-aligned address (columns of a block start at
// multiples of n, so 16-byte alignment cannot be had; the hardware does not need it).
template <typename T, int N>
struct alignas(sizeof(T)) Run {
    T v[N];
};
template <>
struct Run<float, 4> {
    typedef float vec __attribute__((ext_vector_type(4), aligned(4)));
    union {
        vec x;
        float v[4];
    };
};
template <>
struct Run<float, 2> {
    typedef float vec __attribute__((ext_vector_type(2), aligned(4)));
    union {
        vec x;
        float v[2];
    };
};
template <>
struct Run<double, 2> {
    typedef double vec __attribute__((ext_vector_type(2), aligned(8)));
    union {
        vec x;
        double v[2];
    };
};
template <>
struct Run<double, 4> {
    typedef double vec __attribute__((ext_vector_type(4), aligned(8)));
    union {
        vec x;
        double v[4];
    };
};

template <typename T, int N>
__device__ __forceinline__ Run<T, N> load_run(const T* p) {
    return *(const Run<T, N>*)p;
}
// The same with only the first `live` values read (zero beyond).
template <typename T, int N>
__device__ __forceinline__ Run<T, N> load_run_part(const T* p, int live) {
    Run<T, N> r;
#pragma unroll
    for (int e = 0; e < N; ++e) r.v[e] = e < live ? p[e] : T{};
    return r;
}

// 4 x 4 transpose between a lane's four values and the wave's four 16-lane groups: group
// g's value s goes to group s as value g, so four consecutive rows per group become, step
// by step, one row per group.
__device__ __forceinline__ void transpose_groups(uint32_t (&x)[4]) {
    const auto a = __builtin_amdgcn_permlane16_swap(x[0], x[1], false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(x[2], x[3], false, false);
    const auto c = __builtin_amdgcn_permlane32_swap(a[0], b[0], false, false);
    const auto d = __builtin_amdgcn_permlane32_swap(a[1], b[1], false, false);
    x[0] = c[0];
    x[1] = d[0];
    x[2] = c[1];
    x[3] = d[1];
}

// In the storage type; values are widened as the products take them.
__device__ __forceinline__ void rows_to_steps(Run<float, 4>& q) {
    uint32_t x[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) x[s] = __builtin_bit_cast(uint32_t, q.v[s]);
    transpose_groups(x);
#pragma unroll
    for (int s = 0; s < 4; ++s) q.v[s] = __builtin_bit_cast(float, x[s]);
}
__device__ __forceinline__ void rows_to_steps(Run<bf16_t, 4>& q) {
    uint32_t x[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) x[s] = q.v[s].bits;
    transpose_groups(x);
#pragma unroll
    for (int s = 0; s < 4; ++s) q.v[s].bits = (uint16_t)x[s];
}
__device__ __forceinline__ void rows_to_steps(Run<double, 4>& q) {
    uint32_t lo[4], hi[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const uint64_t u = __builtin_bit_cast(uint64_t, (double)q.v[s]);
        lo[s] = (uint32_t)u;
        hi[s] = (uint32_t)(u >> 32);
    }
    transpose_groups(lo);
    transpose_groups(hi);
#pragma unroll
    for (int s = 0; s < 4; ++s) q.v[s] = __builtin_bit_cast(double, ((uint64_t)hi[s] << 32) | lo[s]);
}

// ---------------------------------------------------------------------------
// tn.  One wave: rows rb .. re (rb a multiple of 16) of up to TA blocks of W's columns
// from block pb (nta of them) and TB blocks of V's columns from block cb (ntb of them).
// The sum over rows runs in order, four rows to a product.  wcol(p) is W's column p and
// whether it takes the row scale h0 (SCALE); columns past the end are read as the last
// one and not stored.  SKIP leaves out the products of blocks that a short tile lacks (a
// branch around each); without it they are computed and not stored, which is cheaper
// when TB is the tile's own width.
//   part[j * np + p] = D(p, j)
// ---------------------------------------------------------------------------
template <typename Tw>
struct TnCol {
    const Tw* ptr;
    bool scaled;
};

template <int TA, int TB, bool SCALE, bool SKIP, typename Tw, typename Th, typename Tv, typename WCol>
__device__ __forceinline__ void tn_wave(int64_t n, int64_t rb, int64_t re, int np, int c, int pb, int nta, int cb,
                                        int ntb, WCol wcol, const Th* __restrict__ h0, const Tv* __restrict__ V,
                                        int64_t ldv, double* __restrict__ part) {
    const int lane = threadIdx.x & 63, m = lane % 16, g = lane / 16;
    const Tw* wp[TA];
    bool ws[TA];
    const Tv* vp[TB];
#pragma unroll
    for (int a = 0; a < TA; ++a) {
        const TnCol<Tw> w = wcol(min((pb + min(a, nta - 1)) * 16 + m, np - 1));
        wp[a] = w.ptr + rb + 4 * g;
        ws[a] = w.scaled;
    }
#pragma unroll
    for (int b = 0; b < TB; ++b)
        vp[b] = V + (int64_t)min((cb + min(b, ntb - 1)) * 16 + m, c - 1) * ldv + rb + 4 * g;
    const Th* hp = SCALE ? h0 + rb + 4 * g : nullptr;
    v4d acc[TA][TB];
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b) acc[a][b] = v4d{0, 0, 0, 0};
    Run<Tw, 4> wq[TA];
    Run<Tv, 4> vq[TB];
    Run<Th, 4> hq;
    auto load = [&](int64_t r0) {
        if (r0 + 16 <= n) {
#pragma unroll
            for (int a = 0; a < TA; ++a)
                if (!SKIP || a < nta) wq[a] = load_run<Tw, 4>(wp[a]);
#pragma unroll
            for (int b = 0; b < TB; ++b)
                if (!SKIP || b < ntb) vq[b] = load_run<Tv, 4>(vp[b]);
            if (SCALE) hq = load_run<Th, 4>(hp);
        } else {
            const int live = (int)(n - r0) - 4 * g;   // rows of this lane that exist (may be <= 0)
#pragma unroll
            for (int a = 0; a < TA; ++a)
                if (!SKIP || a < nta) wq[a] = load_run_part<Tw, 4>(wp[a], live);
#pragma unroll
            for (int b = 0; b < TB; ++b)
                if (!SKIP || b < ntb) vq[b] = load_run_part<Tv, 4>(vp[b], live);
            if (SCALE) hq = load_run_part<Th, 4>(hp, live);
        }
#pragma unroll
        for (int a = 0; a < TA; ++a) wp[a] += 16;
#pragma unroll
        for (int b = 0; b < TB; ++b) vp[b] += 16;
        if (SCALE) hp += 16;
    };
    if (rb < re) load(rb);
    for (int64_t r0 = rb; r0 < re; r0 += 16) {
        Run<Tw, 4> w[TA];
        Run<Tv, 4> v[TB];
        Run<Th, 4> h;
#pragma unroll
        for (int a = 0; a < TA; ++a)
            if (!SKIP || a < nta) rows_to_steps(w[a] = wq[a]);
#pragma unroll
        for (int b = 0; b < TB; ++b)
            if (!SKIP || b < ntb) rows_to_steps(v[b] = vq[b]);
        if (SCALE) rows_to_steps(h = hq);
        if (r0 + 16 < re) load(r0 + 16);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            double ws4[TA];
#pragma unroll
            for (int a = 0; a < TA; ++a) {
                ws4[a] = to_f64(w[a].v[s]);
                if (SCALE) ws4[a] *= ws[a] ? to_f64(h.v[s]) : 1.0;
            }
#pragma unroll
            for (int b = 0; b < TB; ++b)
                if (!SKIP || b < ntb) {
                    const double vb = to_f64(v[b].v[s]);
#pragma unroll
                    for (int a = 0; a < TA; ++a)
                        if (!SKIP || a < nta) acc[a][b] = mfma64(vb, ws4[a], acc[a][b]);
                }
        }
    }
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b)
            if (a < nta && b < ntb) {
                const int p = (pb + a) * 16 + m;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int j = (cb + b) * 16 + g + 4 * r;
                    if (p < np && j < c) part[(int64_t)j * np + p] = acc[a][b][r];
                }
            }
}

// How the column blocks and the W blocks of a tn product are dealt to waves.  A wave's
// tile is at most 14 blocks (112 accumulator registers, two waves to a SIMD): 2 x TB up to
// 2 x 7, and 4 x TB for one and two column blocks, where reading W dominates and a wave
// wants more of it in flight.  A float64 V takes twice the registers and stops at 2 x 4.
constexpr int NN_TB = 7, TN_WIDE_TB = 4;   // most column blocks of a tile
__host__ __device__ constexpr int tile_rows(int tb) { return tb <= 2 ? 4 : 2; }

struct TnShape {
    int ta, tb;      // blocks per wave tile (template arguments)
    int ptiles;      // wave tiles along W's columns
    int ctiles;      // tiles along V's columns
    int waves;       // waves of this tile a SIMD holds (by its registers)
    int tiles() const { return ptiles * ctiles; }
};

inline TnShape tn_shape(int np, int c, bool wide_v) {
    const int pblocks = ceil_div(np, 16), cblocks = ceil_div(c, 16);
    TnShape s;
    s.ctiles = ceil_div(cblocks, wide_v ? TN_WIDE_TB : NN_TB);
    s.tb = ceil_div(cblocks, s.ctiles);
    s.ta = tile_rows(s.tb);
    s.ptiles = ceil_div(pblocks, s.ta);
    s.waves = s.tb >= 5 ? 2 : (s.tb % 2 ? 4 : 3) - (wide_v ? 1 : 0);
    return s;
}

// A workgroup is one wave (waves share nothing, and tiles of one wave fill the SIMDs
// evenly: with four to a workgroup a fifth of the chip idled at 13 tiles): row chunk
// `chunk`, W tile `pt`, V tile `ct`.
template <int TA, int TB, bool SCALE, bool SKIP, typename Tw, typename Th, typename Tv, typename WCol>
__device__ __forceinline__ void tn_tile(int64_t n, int np, int c, int chunk, int64_t rows_per_chunk, int pt, int ct,
                                        int ctiles, WCol wcol, const Th* __restrict__ h0, const Tv* __restrict__ V,
                                        int64_t ldv, double* __restrict__ part) {
    const int pblocks = (np + 15) / 16, cblocks = (c + 15) / 16, pb = pt * TA;
    const int cb = ct * cblocks / ctiles, ce = (ct + 1) * cblocks / ctiles;
    const int64_t rb = (int64_t)chunk * rows_per_chunk;
    const int64_t re = min(n, rb + rows_per_chunk);
    tn_wave<TA, TB, SCALE, SKIP, Tw>(n, rb, re, np, c, pb, min(TA, pblocks - pb), cb, ce - cb, wcol, h0, V, ldv,
                                     part + (int64_t)chunk * np * c);
}

// Workgroup id -> (chunk, position in the chunk).  Workgroup g runs on XCD g % 8; the
// tiles of a chunk sit side by side on one XCD, which reads their rows from HBM once.
__device__ __forceinline__ bool tn_place(int id, int tiles, int nchunks, int& chunk, int& pos) {
    const int local = id / 8;
    chunk = id % 8 + 8 * (local / tiles);
    pos = local % tiles;
    return chunk < nchunks;
}
inline int tn_grid(int tiles, int nchunks) { return 8 * ceil_div(nchunks, 8) * tiles; }

// ---------------------------------------------------------------------------
// nn.  M comes packed in fragment order (A of step s, column block b: 64 consecutive
// values): M(q, j) at ((q / 4) * cblocks + j / 16) * 64 + (q % 4) * 16 + j % 16, rows
// nq .. 4 ceil(nq / 4) - 1 zero.
// ---------------------------------------------------------------------------
__host__ __device__ inline int64_t nn_pack_index(int q, int j, int cblocks) {
    return ((int64_t)(q / 4) * cblocks + j / 16) * 64 + (q % 4) * 16 + j % 16;
}
inline size_t nn_pack_doubles(int nq, int c) { return (size_t)ceil_div(nq, 4) * ceil_div(c, 16) * 64; }

// One workgroup of four waves, 16 TA rows each from row0 (row TA (l % 16) + f of a wave's
// rows in fragment f, so loads and stores are runs of TA rows), ntb column blocks from cb.
// M goes through LDS, NN_STEPS steps at a time, because loads return in order: fetched
// with the products that need it, it would wait for every older load of W.  wcol(q) as
// for tn (its row scale is h0); W's runs are loaded whole where `full` (rows past n exist).
// The results go out block by block: emit.ahead(j, r, live) reads what storing rows r ..
// r + live - 1 of column j needs, a block before emit.store(j, r, o, h, read, live) does it
// (h: the row scales; read on demand, the epilogue was a chain of memory round trips).
constexpr int NN_STEPS = 4;
template <int TB>
struct NnLds {
    double m[2][NN_STEPS][TB][64];
};

template <int TA, int TB, bool SCALE, bool SKIP, typename Tw, typename Th, typename WCol, typename Emit>
__device__ __forceinline__ void nn_group(NnLds<TB>& lds, int64_t n, int64_t row0, bool full, int nq, int c, int cblocks,
                                         int cb, int ntb, WCol wcol, const Th* __restrict__ h0,
                                         const double* __restrict__ M, Emit emit) {
    const int lane = threadIdx.x & 63, m = lane % 16, g = lane / 16;
    const int64_t r = row0 + 16 * TA * (int64_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) + TA * m;
    const int live = (int)max((int64_t)0, min((int64_t)TA, n - r));
    const int64_t rl = live > 0 ? r : n - 1;     // a row that exists
    const int steps = (nq + 3) / 4, batches = (steps + NN_STEPS - 1) / NN_STEPS;
    const bool whole = full ? live > 0 : live == TA;
    double h[TA];
    if (SCALE) {
#pragma unroll
        for (int f = 0; f < TA; ++f) h[f] = f < live ? to_f64(h0[r + f]) : 0.0;
    }
    v4d acc[TA][TB];
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b) acc[a][b] = v4d{0, 0, 0, 0};
    // a batch of M: NN_STEPS x TB fragments of 64, NN_STEPS x TB / 4 values to a thread
    // (thread t: step t / 64, lane t % 64); steps past the end are zero
    double mreg[TB];
    auto fetch_m = [&](int batch) {
        const int s = batch * NN_STEPS + (int)(threadIdx.x >> 6);
        const double* src = M + ((int64_t)min(s, steps - 1) * cblocks + cb) * 64 + lane;
#pragma unroll
        for (int b = 0; b < TB; ++b) mreg[b] = s < steps ? src[(int64_t)min(b, ntb - 1) * 64] : 0.0;
    };
    auto store_m = [&](int buf) {
#pragma unroll
        for (int b = 0; b < TB; ++b) lds.m[buf][threadIdx.x >> 6][b][lane] = mreg[b];
    };
    Run<Tw, TA> wq[NN_STEPS];
    bool ws[NN_STEPS];
    auto load_w = [&](int s, Run<Tw, TA>& w, bool& scaled) {
        const TnCol<Tw> col = wcol(min(4 * s + g, nq - 1));
        w = whole ? load_run<Tw, TA>(col.ptr + r) : load_run_part<Tw, TA>(col.ptr + rl, live);
        scaled = col.scaled;
    };
    fetch_m(0);
#pragma unroll
    for (int d = 0; d < NN_STEPS; ++d) load_w(min(d, steps - 1), wq[d], ws[d]);
    store_m(0);
    __syncthreads();
    for (int t = 0; t < batches; ++t) {
        fetch_m(t + 1);
#pragma unroll
        for (int d = 0; d < NN_STEPS; ++d) {
            const int s = t * NN_STEPS + d;
            double w[TA];
#pragma unroll
            for (int f = 0; f < TA; ++f) {
                w[f] = to_f64(wq[d].v[f]);
                if (SCALE) w[f] *= ws[d] ? h[f] : 1.0;
            }
            load_w(min(s + NN_STEPS, steps - 1), wq[d], ws[d]);
            if (s < steps) {
#pragma unroll
                for (int b = 0; b < TB; ++b)
                    if (!SKIP || b < ntb) {
                        const double mv = lds.m[t & 1][d][b][lane];
#pragma unroll
                        for (int f = 0; f < TA; ++f) acc[f][b] = mfma64(mv, w[f], acc[f][b]);
                    }
            }
        }
        // the other buffer was last read a batch ago, before the barrier that ended it
        store_m((t + 1) & 1);
        __syncthreads();
    }
    if (live <= 0) return;
    typename Emit::Ahead ahead[2][4];
    auto read = [&](int b) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int j = (cb + b) * 16 + g + 4 * e;
            if (b < ntb && j < c) ahead[b & 1][e] = emit.ahead(j, r, live);
        }
    };
    read(0);
#pragma unroll
    for (int b = 0; b < TB; ++b) {
        if (b + 1 < TB) read(b + 1);
        __builtin_amdgcn_sched_barrier(0);   // the next block's reads before this one's stores
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int j = (cb + b) * 16 + g + 4 * e;
            double o[TA];
#pragma unroll
            for (int f = 0; f < TA; ++f) o[f] = acc[f][b][e];
            if (b < ntb && j < c) emit.store(j, r, o, h, ahead[b & 1][e], live);
        }
    }
}

struct NnShape {
    int ta, tb, ctiles;
    __host__ __device__ int rows() const { return 64 * ta; }   // rows of a workgroup (four waves)
};

// Four rows to a lane while the accumulators leave room (16-byte runs), two beyond.
inline NnShape nn_shape(int c) {
    const int cblocks = ceil_div(c, 16);
    NnShape s;
    s.ctiles = ceil_div(cblocks, NN_TB);
    const int tb = ceil_div(cblocks, s.ctiles);
    s.tb = tb;
    s.ta = tile_rows(tb);
    return s;
}
// The column tiles of a row block sit side by side on one XCD (workgroup g on XCD g % 8).
inline int nn_grid(int64_t n, const NnShape& s) { return 8 * ceil_div(ceil_div(n, s.rows()), 8) * s.ctiles; }
__device__ __forceinline__ bool nn_place(int id, int64_t n, int rows, int ctiles, int64_t& row0, int& ct) {
    const int local = id / 8;
    const int64_t blk = id % 8 + 8 * (int64_t)(local / ctiles);
    ct = local % ctiles;
    row0 = blk * rows;
    return row0 < n;
}

// Calls f(std::integral_constant<int, TB>) for the tile width tb (1 .. 7).
template <typename F>
void with_tile_width(int tb, F&& f) {
    switch (tb) {
        case 1: f(std::integral_constant<int, 1>()); break;
        case 2: f(std::integral_constant<int, 2>()); break;
        case 3: f(std::integral_constant<int, 3>()); break;
        case 4: f(std::integral_constant<int, 4>()); break;
        case 5: f(std::integral_constant<int, 5>()); break;
        case 6: f(std::integral_constant<int, 6>()); break;
        default: f(std::integral_constant<int, 7>()); break;
    }
}
