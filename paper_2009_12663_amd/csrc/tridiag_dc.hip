// Eigenpairs of the symmetric tridiagonal T (diagonal d, off-diagonal e, e[i] =
// T(i, i+1)) from the Householder reduction of Omega, for Alg. 3's small symmetric
// eigenproblem (Omega = U_s Lambda U_s^T), by divide and conquer (Cuppen 1981):
//
//   T = diag(T_A - b e_last e_last^T, T_B - b e_1 e_1^T) + b u u^T,  u = e_last + e_1,
//
// so with T_A = Q_A D_A Q_A^T and T_B = Q_B D_B Q_B^T the merged problem is
// diag(D_A, D_B) + rho z z^T with rho = 2 b and z = [Q_A's last row, Q_B's first row]
// / sqrt 2.  Its eigenvalues are the roots of the secular equation
// f(x) = 1 + rho sum_i z_i^2 / (d_i - x), one between consecutive poles and one above
// the last (rho > 0; a negative rho is handled by negating D).  Steps of a merge:
//   * sort the poles; deflate components with |rho z_i| <= tol, and close poles by a
//     Givens rotation that moves one pole's weight onto its neighbour;
//   * each root by safeguarded Newton steps on tau f(tau) inside a bracket that every
//     evaluation's sign narrows (falling back to the bracket's midpoint), measured from
//     the nearer pole (x = d_o + tau), so that differences x - d_i keep their relative
//     accuracy;
//   * z recomputed from the roots (Loewner's formula; Gu and Eisenstat 1994), which
//     makes the eigenvectors z_i / (d_i - x_j) numerically orthogonal;
//   * the merged basis: the sorted, rotated columns of diag(Q_A, Q_B) times those
//     eigenvectors.
// The merges run bottom-up over power-of-two blocks (leaf i starts at d_i - e_{i-1}
// - e_i, since every adjacent pair is split at some level), one workgroup per merge,
// all merges of a level in one launch.  Z = Q_H Y then gives the eigenvectors of Omega.
#include <algorithm>
#include <cmath>

#include "common.h"

namespace {

constexpr double EPS = 2.220446049250313e-16;   // 2^-52
constexpr int DC_MAX = 256;
constexpr int DC_THREADS = 1024;   // at most: a merge of blocks of h takes 8 h, four to a pole

// The value that lane q of this lane's quad holds (q a constant).
template <int Q>
__device__ __forceinline__ double quad_get(double x) {
    constexpr int CTRL = Q * 0x55;   // quad_perm [Q, Q, Q, Q]
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

// What the merges of a workgroup share, by the column's place in the workgroup.
struct MergeLds {
    double Dv[DC_MAX], zv[DC_MAX], ds[DC_MAX], zs[DC_MAX];
    double dn[DC_MAX], z2n[DC_MAX], zn[DC_MAX], taun[DC_MAX], zh[DC_MAX], lamn[DC_MAX];
    double rot_c[DC_MAX], rot_s[DC_MAX];
    int pcol[DC_MAX], ndx[DC_MAX], slot_of[DC_MAX], orgn[DC_MAX], rot_a[DC_MAX], rot_b[DC_MAX], nrot[DC_MAX];
    // a bit a pole: of weight (not deflated by it), turning with the pole before it, kept
    uint32_t weighty[DC_MAX / 32], turns[DC_MAX / 32], kept[DC_MAX / 32];
};

// First set bit of [from, end), or end.
__device__ __forceinline__ int next_bit(const uint32_t* w, int from, int end) {
    while (from < end) {
        const uint32_t m = w[from >> 5] >> (from & 31);
        if (m) return min(end, from + __ffs(m) - 1);
        from = (from | 31) + 1;
    }
    return end;
}

// Last set bit of [first, before), or -1.
__device__ __forceinline__ int prev_bit(const uint32_t* w, int first, int before) {
    while (before > first) {
        const uint32_t m = w[(before - 1) >> 5] << (31 - ((before - 1) & 31));
        if (m) {
            const int at = before - 1 - __clz(m);
            return at >= first ? at : -1;
        }
        before = (before - 1) & ~31;
    }
    return -1;
}

// Set bits of [first, before).
__device__ __forceinline__ int count_bits(const uint32_t* w, int first, int before) {
    int n = 0;
    while (first < before) {
        const int stop = min(before, (first | 31) + 1), len = stop - first;
        n += __popc((w[first >> 5] >> (first & 31)) & (len == 32 ? ~0u : (1u << len) - 1u));
        first = stop;
    }
    return n;
}

// One merge of blocks [s, s + h) and [s + h, s + h + hb) by 8 h threads (t of them; 4 to a
// pole), whose part of the shared arrays begins at `off`; the workgroup's merges of a level
// run side by side and meet the same barriers (one with nothing to merge has n = 0).
// Qin/lam_in hold the blocks' eigenvectors (block-diagonal, column-major c x c) and
// eigenvalues; lam_out receives the merged ones, R and U (c x c scratch, block regions) the
// rotated basis and the eigenvectors in it, whose product is the merged basis.
// Returns the number K of poles kept.
// The time is that of chains: divisions, and at the last level the root whose Newton steps
// are most (52 at 120 poles).  A pole's or root's sums and products are shared by a quad of
// lanes: each forms every fourth term, and the terms are added or multiplied in index
// order, as by one lane.  The scan for close poles walks only those that turn.
__device__ __forceinline__ int merge_block(MergeLds& m, int c, int h, int s, int off, int n, int ha, int t,
                                           const double* __restrict__ e, const double* __restrict__ lam_in,
                                           const double* __restrict__ Qin, double* __restrict__ lam_out,
                                           double* __restrict__ R, double* __restrict__ U) {
    const int step = 8 * h, quad = t >> 2, q = t & 3, end = off + n;
    const double beta = n > 0 ? e[s + ha - 1] : 0.0;
    const bool neg = beta < 0.0;
    const double rho = 2.0 * fabs(beta);
    const double r2 = 0.7071067811865476;   // 1 / sqrt 2
    double *Dv = m.Dv + off, *zv = m.zv + off, *ds = m.ds + off, *zs = m.zs + off, *dn = m.dn + off;
    double *z2n = m.z2n + off, *zn = m.zn + off, *taun = m.taun + off, *zh = m.zh + off, *lamn = m.lamn + off;
    int *pcol = m.pcol + off, *ndx = m.ndx + off, *slot_of = m.slot_of + off, *orgn = m.orgn + off;
    // poles and weights (negated when beta < 0, so that rho > 0)
    for (int p = t; p < n; p += step) {
        const double dv = lam_in[s + p];
        Dv[p] = neg ? -dv : dv;
        zv[p] = r2 * (p < ha ? Qin[(int64_t)(s + p) * c + s + ha - 1] : Qin[(int64_t)(s + p) * c + s + ha]);
    }
    for (int w = threadIdx.x; w < DC_MAX / 32; w += (int)blockDim.x) m.weighty[w] = m.turns[w] = 0;
    __syncthreads();
    // sort by rank (ties by index).  The order is total even for NaN (after every
    // number, among themselves by index), so the ranks are a permutation and every
    // pcol entry is written: a non-finite input gives wrong values, never an index
    // out of range.
    double tol = 0.0;
    if (quad < n) {
        const double dt = Dv[quad];
        const bool nt = isnan(dt);
        int rk = 0;
        double dmax = rho;
        for (int u = q; u < n; u += 4) {
            const double du = Dv[u];
            const bool before = isnan(du) ? (nt && u < quad) : (nt || du < dt || (du == dt && u < quad));
            rk += before ? 1 : 0;
            dmax = fmax(dmax, fabs(du));
        }
        rk += __shfl_xor(rk, 1, 4);
        rk += __shfl_xor(rk, 2, 4);
        dmax = fmax(fmax(quad_get<0>(dmax), quad_get<1>(dmax)), fmax(quad_get<2>(dmax), quad_get<3>(dmax)));
        tol = 8.0 * EPS * dmax;
        const double z = zv[quad];
        if (q == 0) {
            ds[rk] = dt;
            zs[rk] = z;
            pcol[rk] = quad;
            if (!(fabs(rho * z) <= tol)) atomicOr(&m.weighty[(off + rk) >> 5], 1u << ((off + rk) & 31));
        }
    }
    __syncthreads();
    // Deflation of close neighbours among the poles of weight: the pairs that would turn are
    // found by all threads, and one lane walks from turn to turn (a turn changes the pair
    // after it, which is tested anew).
    auto turn_of = [&](int a, int b, double& tau, double& cc, double& sn) {
        const double zl = zs[a], zi = zs[b];
        tau = sqrt(fma(zl, zl, zi * zi));
        cc = zi / tau;
        sn = -zl / tau;
        return fabs((ds[b] - ds[a]) * cc * sn) <= tol;
    };
    for (int w = threadIdx.x; w < DC_MAX / 32; w += (int)blockDim.x) m.kept[w] = m.weighty[w];
    if (t < n && (m.weighty[(off + t) >> 5] >> ((off + t) & 31) & 1)) {
        const int last = prev_bit(m.weighty, off, off + t);
        double tau, cc, sn;
        if (last >= 0 && turn_of(last - off, t, tau, cc, sn)) atomicOr(&m.turns[(off + t) >> 5], 1u << ((off + t) & 31));
    }
    __syncthreads();
    if (t == 0) {
        int nrot = 0;
        int p = next_bit(m.turns, off, end);
        while (p < end) {
            int last = prev_bit(m.weighty, off, p);
            double tau, cc, sn;
            turn_of(last - off, p - off, tau, cc, sn);
            do {
                zs[p - off] = tau;
                zs[last - off] = 0.0;
                const double dl = ds[last - off], di = ds[p - off];
                ds[last - off] = dl * cc * cc + di * sn * sn;
                ds[p - off] = dl * sn * sn + di * cc * cc;
                atomicAnd(&m.kept[last >> 5], ~(1u << (last & 31)));
                m.rot_a[off + nrot] = last - off;
                m.rot_b[off + nrot] = p - off;
                m.rot_c[off + nrot] = cc;
                m.rot_s[off + nrot] = sn;
                ++nrot;
                last = p;
                p = next_bit(m.weighty, p + 1, end);
            } while (p < end && turn_of(last - off, p - off, tau, cc, sn));
            if (p < end) p = next_bit(m.turns, p + 1, end);
        }
        m.nrot[off] = nrot;
    }
    __syncthreads();
    const int K = count_bits(m.kept, off, end), nrot = n > 0 ? m.nrot[off] : 0;
    if (t < n) {
        const bool kept = m.kept[(off + t) >> 5] >> ((off + t) & 31) & 1;
        const int j = count_bits(m.kept, off, off + t);
        slot_of[t] = kept ? j : -1;
        if (kept) {
            const double zj = zs[t];
            ndx[j] = t;
            dn[j] = ds[t];
            zn[j] = zj;
            z2n[j] = zj * zj;
        }
    }
    __syncthreads();
    // secular roots: quad j finds root j from its nearer pole (bracket, then Newton); lane q
    // of the quad forms the terms i = 4 l + q
    if (quad < K) {
        const int j = quad, K4 = K & ~3;
        int o;
        double a, b;
        if (j < K - 1) {
            const double mid = 0.5 * (dn[j] + dn[j + 1]);
            double f = 1.0;
#pragma unroll 2
            for (int i = 0; i < K; i += 4) {
                const int iq = min(i + q, K - 1);
                const double v = rho * z2n[iq] / (dn[iq] - mid);
                f += quad_get<0>(v);
                if (i + 1 < K) f += quad_get<1>(v);
                if (i + 2 < K) f += quad_get<2>(v);
                if (i + 3 < K) f += quad_get<3>(v);
            }
            if (f > 0.0) {
                o = j;
                a = 0.0;
                b = mid - dn[j];
            } else {
                o = j + 1;
                a = mid - dn[j + 1];
                b = 0.0;
            }
        } else {
            double z2sum = 0.0;
            for (int i = 0; i < K; ++i) z2sum += z2n[i];
            o = K - 1;
            a = 0.0;
            b = rho * z2sum;
        }
        // Newton on h(x) = x f(x), which has the same root but no pole at the origin
        // (that term of x f is the constant -rho z_o^2; the other pole is at least twice
        // as far as the root).  The iterate stays inside the bracket [a, b] that each
        // evaluation's sign of f narrows (f increases in x); a step that leaves it is
        // replaced by the bracket's midpoint.  Every lane of the quad takes the same steps.
        const double dorg = dn[o];
        double x = 0.5 * (a + b);
        for (int it = 0; it < 256; ++it) {
            // lane q: the sums over i = 4 l + q below K4; lane 0 also the rest, in order
            double fq = 0.0, gq = 0.0;
#pragma unroll 4
            for (int i = q; i < K4; i += 4) {
                const double qi = 1.0 / ((dn[i] - dorg) - x), w = z2n[i] * qi;
                fq += w;
                gq = fma(w, qi, gq);
            }
            if (q == 0)
                for (int i = K4; i < K; ++i) {
                    const double qi = 1.0 / ((dn[i] - dorg) - x), w = z2n[i] * qi;
                    fq += w;
                    gq = fma(w, qi, gq);
                }
            const double fs = (quad_get<0>(fq) + quad_get<1>(fq)) + (quad_get<2>(fq) + quad_get<3>(fq));
            const double gs = (quad_get<0>(gq) + quad_get<1>(gq)) + (quad_get<2>(gq) + quad_get<3>(gq));
            const double f = fma(rho, fs, 1.0);
            const double fp = rho * gs;
            if (f == 0.0) break;
            if (f > 0.0) b = x;
            else a = x;
            const double dx = x * f / fma(x, fp, f);
            double xn = x - dx;
            if (fabs(dx) <= 2.0 * EPS * fabs(x)) {
                x = xn;
                break;
            }
            if (!(xn > a && xn < b)) xn = 0.5 * (a + b);
            x = xn;
            if (b - a <= 2.0 * EPS * fmax(fabs(a), fabs(b))) break;
        }
        if (q == 0) {
            orgn[j] = o;
            taun[j] = x;
            lamn[j] = dorg + x;
        }
    }
    __syncthreads();
    // Loewner: zh_i^2 = prod_j (x_j - d_i) / prod_{j != i} (d_j - d_i) / rho; the quad's
    // lanes form four quotients at a time, multiplied in order
    if (quad < K) {
        const int i = quad;
        const double di = dn[i];
        double p = (dn[orgn[K - 1]] - di) + taun[K - 1];
#pragma unroll 2
        for (int j0 = 0; j0 < K - 1; j0 += 4) {
            const int j = min(j0 + q, K - 2);
            const double lj = (dn[orgn[j]] - di) + taun[j];
            const double dd = j >= i ? dn[j + 1] - di : dn[j] - di;
            const double v = lj / dd;
            p *= quad_get<0>(v);
            if (j0 + 1 < K - 1) p *= quad_get<1>(v);
            if (j0 + 2 < K - 1) p *= quad_get<2>(v);
            if (j0 + 3 < K - 1) p *= quad_get<3>(v);
        }
        p /= rho;
        if (q == 0) zh[i] = copysign(sqrt(fmax(p, 0.0)), zn[i]);
    }
    __syncthreads();
    // U (K x K, column j = normalised zh / (d - x_j)) in the block region of U
    if (quad < K) {
        double* Uj = U + (int64_t)(s + quad) * c + s;
        const double dj = dn[orgn[quad]], tj = taun[quad];
        double ss = 0.0;
#pragma unroll 2
        for (int i = 0; i < K; i += 4) {
            const int iq = min(i + q, K - 1);
            const double v = zh[iq] / ((dn[iq] - dj) - tj);
            if (i + q < K) Uj[iq] = v;
            const double v0 = quad_get<0>(v), v1 = quad_get<1>(v), v2 = quad_get<2>(v), v3 = quad_get<3>(v);
            ss = fma(v0, v0, ss);
            if (i + 1 < K) ss = fma(v1, v1, ss);
            if (i + 2 < K) ss = fma(v2, v2, ss);
            if (i + 3 < K) ss = fma(v3, v3, ss);
        }
        const double inv = 1.0 / sqrt(ss);
        for (int i = q; i < K; i += 32) {   // the lane's own entries, eight in flight
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = Uj[min(i + 4 * u, K - 1)];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (i + 4 * u < K) Uj[i + 4 * u] = v[u] * inv;
        }
    }
    // rotated basis R: row r, sorted column p = column pcol[p] of diag(Q_A, Q_B) (only the
    // diagonal blocks of Qin are current; the rest is zero), then the deflation rotations in
    // order (one thread per row).  Row r's operands are columns that no earlier rotation has
    // written, but for a pair's first one where it is the second of the pair before.
    const int r = t & (2 * h - 1);
    double* Rr = R + (int64_t)s * c + s + r;   // Rr[p * c] = R(r, p)
    if (r < n) {
        const double* Qr = Qin + (int64_t)s * c + s + r;
        for (int p0 = t / (2 * h); p0 < n; p0 += 32) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = Qr[(int64_t)pcol[min(p0 + 4 * u, n - 1)] * c];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int p = p0 + 4 * u;
                if (p < n) Rr[(int64_t)p * c] = (pcol[p] < ha) == (r < ha) ? v[u] : 0.0;
            }
        }
    }
    __syncthreads();
    if (t < n && nrot > 0) {
        const int* ra = m.rot_a + off;
        const int* rb = m.rot_b + off;
        double carried = 0.0;
        for (int u0 = 0; u0 < nrot; u0 += 4) {
            double xa4[4], xb4[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int w = min(u0 + u, nrot - 1);
                xa4[u] = Rr[(int64_t)ra[w] * c];
                xb4[u] = Rr[(int64_t)rb[w] * c];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int w = u0 + u;
                if (w >= nrot) break;
                const int pa = ra[w], pb = rb[w];
                const double cc = m.rot_c[off + w], sn = m.rot_s[off + w];
                const double xa = w > 0 && pa == rb[w - 1] ? carried : xa4[u], xb = xb4[u];
                Rr[(int64_t)pa * c] = cc * xa + sn * xb;
                carried = -sn * xa + cc * xb;
                Rr[(int64_t)pb * c] = carried;
            }
        }
    }
    if (t < n) {
        const int j = slot_of[t];
        const double v = j < 0 ? ds[t] : lamn[j];
        lam_out[s + t] = neg ? -v : v;
    }
    return K;
}

// Merges of one level, a workgroup each; the merged basis (R[:, ndx] U, deflated columns as
// rotated) is formed by dc_merge_gemm.
__global__ void __launch_bounds__(DC_THREADS) dc_merge(int c, int h, const double* __restrict__ e,
                                                       const double* __restrict__ lam_in, const double* __restrict__ Qin,
                                                       double* __restrict__ lam_out, double* __restrict__ Qout,
                                                       double* __restrict__ R, double* __restrict__ U,
                                                       int* __restrict__ Kg, int* __restrict__ ndx_g,
                                                       int* __restrict__ slot_g) {
    __shared__ MergeLds m;
    const int t = threadIdx.x;
    const int s = blockIdx.x * 2 * h;
    if (s >= c) return;                                   // whole workgroup
    const int ha = min(h, c - s);
    const int hb = min(h, c - s - ha);
    const int n = ha + hb;
    if (hb == 0) {
        // nothing to merge: copy the block (dc_merge_gemm skips it)
        if (t == 0) Kg[blockIdx.x] = -1;
        for (int u = t; u < n * n; u += (int)blockDim.x) {
            const int col = s + u / n, row = s + u % n;
            Qout[(int64_t)col * c + row] = Qin[(int64_t)col * c + row];
        }
        for (int u = t; u < n; u += (int)blockDim.x) lam_out[s + u] = lam_in[s + u];
        return;
    }
    const int K = merge_block(m, c, h, s, 0, n, ha, t, e, lam_in, Qin, lam_out, R, U);
    if (t == 0) Kg[blockIdx.x] = K;
    if (t < n) {
        slot_g[s + t] = m.slot_of[t];
        ndx_g[s + t] = t < K ? m.ndx[t] : 0;
    }
}

// The leaves (lam_i = d_i - e_{i-1} - e_i, Q = I) and the levels up to blocks of DC_FIRST
// columns in one launch: a workgroup takes a block through all of them, its merges side
// by side, and forms each merged basis.  Ten launches of 5 to 25 us, mostly fetching the
// same code anew, took 110 us at c = 50, this one 79.  In: d, e; out: lam, Q (in the first
// of each pair after an even number of levels, else in the second; only the diagonal
// blocks are written).
constexpr int DC_FIRST = 32;

__global__ void __launch_bounds__(4 * DC_FIRST) dc_first(int c, const double* __restrict__ d,
                                                         const double* __restrict__ e, double* lam_a, double* Qa,
                                                         double* lam_b, double* Qb, double* R, double* U,
                                                         int32_t* __restrict__ status) {
    __shared__ MergeLds m;
    const int c0 = blockIdx.x * DC_FIRST;
    for (int x = threadIdx.x; x < DC_FIRST * DC_FIRST; x += 4 * DC_FIRST) {
        const int col = c0 + x / DC_FIRST, row = c0 + x % DC_FIRST;
        if (col >= c || row >= c) continue;
        Qa[(int64_t)col * c + row] = col == row ? 1.0 : 0.0;
        if (row == c0) {
            const double el = col > 0 ? e[col - 1] : 0.0, er = col + 1 < c ? e[col] : 0.0;
            lam_a[col] = d[col] - el - er;
            if (!isfinite(d[col]) || !isfinite(el) || !isfinite(er)) set_status(status, BFGS_ERR_NUMERIC);
        }
    }
    __syncthreads();
    for (int h = 1; h < DC_FIRST && h < c; h *= 2) {
        const int t = threadIdx.x & (8 * h - 1), off = threadIdx.x / (8 * h) * (2 * h);
        const int s = blockIdx.x * DC_FIRST + off;
        const int ha = max(0, min(h, c - s)), hb = max(0, min(h, c - s - ha)), n = hb > 0 ? ha + hb : 0;
        const int K = merge_block(m, c, h, s, off, n, ha, t, e, lam_a, Qa, lam_b, R, U);
        __syncthreads();
        const int r = t & (2 * h - 1);
        if (hb == 0) {   // nothing to merge: copied
            for (int p = t / (2 * h); p < ha && r < ha; p += 4) Qb[(int64_t)(s + p) * c + s + r] = Qa[(int64_t)(s + p) * c + s + r];
            if (t < ha) lam_b[s + t] = lam_a[s + t];
        }
        for (int p = t / (2 * h); p < n && r < n; p += 4) {
            const int j = m.slot_of[off + p];
            double acc = 0.0;
            if (j < 0) {
                acc = R[(int64_t)(s + p) * c + s + r];
            } else {
                for (int k0 = 0; k0 < K; k0 += 8) {
                    double a[8], b[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int k = min(k0 + u, K - 1);
                        a[u] = R[(int64_t)(s + m.ndx[off + k]) * c + s + r];
                        b[u] = U[(int64_t)(s + j) * c + s + k];
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (k0 + u < K) acc = fma(a[u], b[u], acc);
                }
            }
            Qb[(int64_t)(s + p) * c + s + r] = acc;
        }
        __syncthreads();
        double* x = Qa;
        Qa = Qb;
        Qb = x;
        x = lam_a;
        lam_a = lam_b;
        lam_b = x;
    }
}

// Merged basis of each merge of the level: column p of the block is R[:, p] when p was
// deflated, else R[:, ndx] U[:, slot(p)].  Grid (merges, tiles of 64 x 64 outputs);
// thread = 4 x 4 outputs; the reduction is staged 16 deep in LDS.
constexpr int MG_T = 64, MG_K = 16;

__global__ void __launch_bounds__(256) dc_merge_gemm(int c, int h, const double* __restrict__ R,
                                                     const double* __restrict__ U, const int* __restrict__ Kg,
                                                     const int* __restrict__ ndx_g, const int* __restrict__ slot_g,
                                                     double* __restrict__ Qout) {
    __shared__ double As[MG_K][MG_T + 1];   // As[k][r] = R(r, ndx[k])
    __shared__ double Bs[MG_K][MG_T + 1];   // Bs[k][p] = U(k, slot(p))
    const int b = blockIdx.x, K = Kg[b];
    if (K < 0) return;                      // whole workgroup: block copied by dc_merge
    const int s = b * 2 * h, n = min(2 * h, c - s);
    const int tpd = (2 * h + MG_T - 1) / MG_T;
    const int r0 = (blockIdx.y / tpd) * MG_T, p0 = (blockIdx.y % tpd) * MG_T;
    if (r0 >= n || p0 >= n) return;         // whole workgroup
    const int tid = threadIdx.x, tr = tid / 16, tp = tid % 16;
    double acc[4][4] = {};
    for (int k0 = 0; k0 < K; k0 += MG_K) {
        for (int e = tid; e < MG_K * MG_T; e += 256) {
            const int kk = e / MG_T, rr = e % MG_T, k = k0 + kk;
            As[kk][rr] = (k < K && r0 + rr < n) ? R[(int64_t)(s + ndx_g[s + k]) * c + s + r0 + rr] : 0.0;
            const int pp = e % MG_T, kb = e / MG_T, kq = k0 + kb;
            int j = p0 + pp < n ? slot_g[s + p0 + pp] : -1;
            Bs[kb][pp] = (kq < K && j >= 0) ? U[(int64_t)(s + j) * c + s + kq] : 0.0;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < MG_K; ++kk) {
            double a[4], bb[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                a[u] = As[kk][tr * 4 + u];
                bb[u] = Bs[kk][tp * 4 + u];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[u][v] = fma(a[u], bb[v], acc[u][v]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int p = p0 + tp * 4 + v;
        if (p >= n) continue;
        const bool defl = slot_g[s + p] < 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int r = r0 + tr * 4 + u;
            if (r < n) Qout[(int64_t)(s + p) * c + s + r] = defl ? R[(int64_t)(s + p) * c + s + r] : acc[u][v];
        }
    }
}

// C = A B, all c x c column-major; block (ceil(c / 64), c): lane -> row, y -> column.
__global__ void __launch_bounds__(64) dc_gemm_nn(int c, const double* __restrict__ A, const double* __restrict__ B,
                                                 double* __restrict__ C) {
    const int r = blockIdx.x * 64 + threadIdx.x, col = blockIdx.y;
    if (r >= c) return;
    const double* bc = B + (int64_t)col * c;
    double acc = 0.0;
    int k = 0;
    for (; k + 16 <= c; k += 16) {   // sixteen in flight, added in order
        double a[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) a[u] = A[(int64_t)(k + u) * c + r];
#pragma unroll
        for (int u = 0; u < 16; ++u) acc = fma(a[u], bc[k + u], acc);
    }
    for (; k < c; ++k) acc = fma(A[(int64_t)k * c + r], bc[k], acc);
    C[(int64_t)col * c + r] = acc;
}

}  // namespace

size_t tridiag_dc_workspace(int c) { return ((size_t)4 * c * c + 2 * (size_t)c) * sizeof(double) + (size_t)4 * c * sizeof(int); }

int tridiag_dc(hipStream_t st, int c, const double* d, const double* e, const double* Qh, double* work, double** w_out,
               double* Z, int32_t* status) {
    if (c < 1 || c > DC_MAX) return BFGS_ERR_ARG;
    const size_t cc = (size_t)c * c;
    double* Qa = work;
    double* Qb = Qa + cc;
    double* R = Qb + cc;
    double* U = R + cc;
    double* la = U + cc;
    double* lb = la + c;
    int* Kg = (int*)(lb + c);
    int* ndx_g = Kg + c;
    int* slot_g = ndx_g + c;
    hipLaunchKernelGGL(dc_first, dim3(ceil_div(c, DC_FIRST)), dim3(4 * DC_FIRST), 0, st, c, d, e, la, Qa, lb, Qb, R, U,
                       status);
    int h = 1;
    for (; h < DC_FIRST && h < c; h *= 2) {
        std::swap(Qa, Qb);
        std::swap(la, lb);
    }
    for (; h < c; h *= 2) {
        const int nb = ceil_div(c, 2 * h);
        const int tpd = ceil_div(2 * h, MG_T);
        hipLaunchKernelGGL(dc_merge, dim3(nb), dim3(8 * h), 0, st, c, h, e, la, Qa, lb, Qb, R, U, Kg, ndx_g, slot_g);
        hipLaunchKernelGGL(dc_merge_gemm, dim3(nb, tpd * tpd), dim3(256), 0, st, c, h, R, U, Kg, ndx_g, slot_g, Qb);
        std::swap(Qa, Qb);
        std::swap(la, lb);
    }
    hipLaunchKernelGGL(dc_gemm_nn, dim3(ceil_div(c, 64), c), dim3(64), 0, st, c, Qh, Qa, Z);
    *w_out = la;
    return hipGetLastError() == hipSuccess ? BFGS_OK : BFGS_ERR_HIP;
}
