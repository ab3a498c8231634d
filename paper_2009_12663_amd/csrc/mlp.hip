// Learned diagonal initial inverse Hessian: an 8 -> 64 -> 64 -> 1 GELU network
// predicting log h0 per (grid point, parameter) -- the learned counterpart of the
// paper's wavefield-based diagonal preconditioners (eqs. 4-8), with gamma I as
// the fallback when no network is used.
//
// Parameters (4801, flattened): W1 (64 x 8), b1 (64), W2 (64 x 64), b2 (64), w3 (64), b3.
// Float32 master copy, bfloat16 compute copy; every product accumulates in float32.
//
// Kernels: a wave takes 32 samples at a time through the matrix cores, one sample per lane
// pair.  The accumulator layout of a 32 x 32 product puts units 8 a + 4 (lane / 32) + b in
// register 4 a + b, and a contraction over units may take them in any order, so a layer's
// activations are the next product's B operand as they stand; the weights wait in LDS in
// the order the products read them.  The forward pass runs its products with a weight
// matrix as bfloat16 products (v_mfma_f32_32x32x16_bf16): the weights are bfloat16 exactly,
// and an activation is the exact sum of three bfloat16 terms.  (Float32 products share the
// vector unit's multipliers: with them it took the sum of its products' and its GELUs'
// time.)  Its error against float64 is 1.0e-7, 1.8e-7 before.  The gradient keeps float32
// products (v_mfma_f32_32x32x2f32): the bfloat16 ones leave an error of one sign in every
// sample, which the sum over the samples does not average away (4.5e-8 against
// 3.5e-8, both with the GELU as it was then).
// Its outer products contract over the samples and go through LDS once.  Per-wave gradient
// partials are summed in a fixed order in float64 (deterministic), followed by Adam on the
// float32 master weights.
//
// What bounds them: the vector unit, with the GELUs, the splitting and, in the gradient,
// the products.  Before, with one wave per sample and a lane per unit: 1,690 us for the
// forward pass of 1.785M samples, now 118 (208 with float32 products); 421 us for the
// gradient of 65,536 samples, of which 252 were its reduction, now 39 (33 and 7).
#include <cmath>
#include <new>

#include "common.h"

namespace {

constexpr int NP = 4801;
constexpr int OFF_W1 = 0, OFF_B1 = 512, OFF_W2 = 576, OFF_B2 = 4672, OFF_W3 = 4736, OFF_B3 = 4800;
constexpr int MLP_BLOCKS = 256;   // 4 waves each -> 1024 waves
constexpr int MLP_WAVES = MLP_BLOCKS * 4;

__device__ __forceinline__ float bfv(const uint16_t* w, int i) {
    bf16_t h;
    h.bits = w[i];
    return bf16_to_float(h);
}

// Twice the upper tail of the normal distribution, 2 Q(u) = 2 (1 - Phi(u)), 0 <= u <= 8, as
// 2^-(u p(u)); about a third of erff's instructions.  p, of degree 8, has the least largest
// absolute error of 2 Q on [0, 6] (2.2e-9), found as a linear program, that of its
// derivative at the exact 2 Q; the coefficients are rounded to float32 from the constant on,
// the rest fitted anew after each (2.4e-9 with these; rounded all at once, 1.3e-8, and since
// that is the same for every sample the sum over the samples kept it: 1.9e-8 of a gradient).
// Beyond 6 the error is under 1e-9.  Beyond 8 the callers take 2 Q(8) = 2e-14.  The
// coefficients here are those of u / 2, the fitted ones times powers of two.
// In float32 2 Q is within 7e-8 (rms 0.9e-8 over [-6, 6]), 1 + erff within 1.5e-7 (3.4e-8);
// the GELU within 2.5e-7 (5.9e-8), with erff 4.5e-7 (7.9e-8).
__device__ __forceinline__ float normal_tail2(float v) {   // of u = 2 v
    float p = -0.0002665532229002565f;
    p = fmaf(p, v, 0.0024759056977927685f);
    p = fmaf(p, v, -0.00968013796955347f);
    p = fmaf(p, v, 0.018327578902244568f);
    p = fmaf(p, v, -0.000594229088164866f);
    p = fmaf(p, v, -0.11083942651748657f);
    p = fmaf(p, v, 0.4194616377353668f);
    p = fmaf(p, v, 1.836888074874878f);
    p = fmaf(p, v, 2.302208423614502f);
    return __builtin_amdgcn_exp2f(-(p * v));
}
// x Phi(x) = max(x, 0) - |x| Q(|x|), from v = x / 2: v + |v| is exact, keeps a NaN, and does
// not overflow where x + |x| would.
__device__ __forceinline__ float gelu_f(float x) {
    const float h = 0.5f * x, v = fminf(fabsf(h), 4.0f);
    return fmaf(-v, normal_tail2(v), h + fabsf(h));
}
// gelu(x) and its derivative Phi(x) + x phi(x)
__device__ __forceinline__ float gelu_with_grad(float x, float& grad) {
    const float h = 0.5f * x, v = fminf(fabsf(h), 4.0f), q = normal_tail2(v);
    const float cdf = x >= 0.0f ? fmaf(-0.5f, q, 1.0f) : 0.5f * q;
    const float e = __builtin_amdgcn_exp2f(x * x * -0.72134752044448170f);   // exp(-x^2 / 2)
    grad = fmaf(x * 0.39894228040143268f, e, cdf);
    return fmaf(-v, q, h + fabsf(h));
}

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // at any float's address
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 mfma_bf16(uint4 a, uint4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                   0, 0);
}

// x = hi + mid + lo exactly, each with at most eight significant bits (truncation): term t
// of eight values, packed.  Of an infinite x, hi is x and the others are zero, not the NaN that
// x - hi is: `infinite` says that the wave may hold one (nothing else needs to look).
struct Split8 {
    uint4 term[3];
};
__device__ __forceinline__ uint32_t high_halves(uint32_t a, uint32_t b) {   // bfloat16 a, then b
    return __builtin_amdgcn_perm(b, a, 0x07060302u);
}
__device__ __forceinline__ Split8 split8(const float (&x)[8], bool infinite) {
    uint32_t t[3][8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const uint32_t u = __builtin_bit_cast(uint32_t, x[e]);
        const float r1 = x[e] - __builtin_bit_cast(float, u & 0xffff0000u);
        const uint32_t v = __builtin_bit_cast(uint32_t, r1);
        const float r2 = r1 - __builtin_bit_cast(float, v & 0xffff0000u);
        t[0][e] = u;
        t[1][e] = v;
        t[2][e] = __builtin_bit_cast(uint32_t, r2);
    }
    if (infinite) {
        asm volatile("" ::: "memory");   // a branch, not a select for every value
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (isinf(x[e])) t[1][e] = t[2][e] = 0u;
    }
    Split8 s;
#pragma unroll
    for (int q = 0; q < 3; ++q)
        s.term[q] = make_uint4(high_halves(t[q][0], t[q][1]), high_halves(t[q][2], t[q][3]),
                               high_halves(t[q][4], t[q][5]), high_halves(t[q][6], t[q][7]));
    return s;
}

// Weights as the products read them (A operand: lane l holds output unit l % 32 of the
// tile and eight inputs).  w1: features 0 .. 7 in both halves.  w2: step (tk, p) takes input
// units 32 tk + 16 p + 4 half + 0 .. 3 and those plus 8, what registers 8 p .. 8 p + 7 hold.
struct MlpWeights {
    uint4 w1[2][32];           // [unit tile][unit]
    uint4 w2[2][2][2][64];     // [output tile][tk][p][lane]
    float4 b1[16], b2[16], w3[16];
    float b3;
};

// The same for the gradient's float32 products, four steps to a float4.
struct MlpGradWeights {
    float4 w1[2][64];          // [unit tile][lane]: features 4 half + 0 .. 3
    float4 w2[2][2][4][64];    // [output tile][input tile][a][lane]: inputs 32 tile + 8 a + 4 half + 0 .. 3
    float4 w2t[2][2][4][64];   // the same of W2 transposed
    float4 b1[16], b2[16], w3[16];
    float b3;
};

template <typename W>
__device__ __forceinline__ void stage_vectors(W& w, const uint16_t* __restrict__ wbf) {
    const int t = threadIdx.x;
    if (t < 64) ((float*)w.b1)[t] = bfv(wbf, OFF_B1 + t);
    else if (t < 128) ((float*)w.b2)[t - 64] = bfv(wbf, OFF_B2 + t - 64);
    else if (t < 192) ((float*)w.w3)[t - 128] = bfv(wbf, OFF_W3 + t - 128);
    else if (t == 192) w.b3 = bfv(wbf, OFF_B3);
}

__device__ __forceinline__ void stage_weights(MlpWeights& w, const uint16_t* __restrict__ wbf) {
    for (int e = threadIdx.x; e < 2 * 2 * 2 * 64 * 2; e += 256) {   // four inputs each
        const int hi = e % 2, l = e / 2 % 64, p = e / 128 % 2, tk = e / 256 % 2, ti = e / 512;
        ((uint2*)w.w2)[e] = *(const uint2*)(wbf + OFF_W2 + (32 * ti + l % 32) * 64 + 32 * tk + 16 * p + 8 * hi +
                                            4 * (l / 32));
    }
    if (threadIdx.x < 64) ((uint4*)w.w1)[threadIdx.x] = *(const uint4*)(wbf + OFF_W1 + threadIdx.x * 8);
    stage_vectors(w, wbf);
}

__device__ __forceinline__ float4 widen4(const uint16_t* src) {   // 8-byte aligned
    const uint2 v = *(const uint2*)src;
    return make_float4(__builtin_bit_cast(float, v.x << 16), __builtin_bit_cast(float, v.x & 0xffff0000u),
                       __builtin_bit_cast(float, v.y << 16), __builtin_bit_cast(float, v.y & 0xffff0000u));
}

__device__ __forceinline__ void stage_weights(MlpGradWeights& w, const uint16_t* __restrict__ wbf) {
    for (int e = threadIdx.x; e < 2 * 2 * 4 * 64; e += 256) {
        const int l = e % 64, a = e / 64 % 4, tk = e / 256 % 2, ti = e / 512;
        ((float4*)w.w2)[e] = widen4(wbf + OFF_W2 + (32 * ti + l % 32) * 64 + 32 * tk + 8 * a + 4 * (l / 32));
    }
    for (int e = threadIdx.x; e < 64 * 16; e += 256) {   // input unit u of W2^T, output units 4 o .. 4 o + 3
        const int u = e / 16, o = e % 16;
        const float4 v = widen4(wbf + OFF_W2 + u * 64 + 4 * o);
        const int tk = u / 32, a = u / 8 % 4, half = u / 4 % 2, ti = o / 8;
        float* dst = (float*)&w.w2t[ti][tk][a][32 * half + 4 * o % 32] + u % 4;
        dst[0] = v.x;
        dst[4] = v.y;
        dst[8] = v.z;
        dst[12] = v.w;
    }
    if (threadIdx.x < 128) {
        const int l = threadIdx.x % 64, ti = threadIdx.x / 64;
        w.w1[ti][l] = widen4(wbf + OFF_W1 + (32 * ti + l % 32) * 8 + 4 * (l / 32));
    }
    stage_vectors(w, wbf);
}

// Register r of tile t belongs to unit 32 t + 8 (r / 4) + 4 half + r % 4.
__device__ __forceinline__ f32x16 units_of(const float4* v, int t, int half) {
    f32x16 x;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const float4 q = v[8 * t + 2 * a + half];
        x[4 * a] = q.x;
        x[4 * a + 1] = q.y;
        x[4 * a + 2] = q.z;
        x[4 * a + 3] = q.w;
    }
    return x;
}

// z = W1 x + b1 for the sample's eight features: one product takes hi (half 0) and mid
// (half 1), another lo and zeros.
__device__ __forceinline__ void layer1(const MlpWeights& w, int lane, const float (&x)[8], f32x16 (&z)[2]) {
    const int half = lane >> 5;
    uint32_t most = 0u;
#pragma unroll
    for (int e = 0; e < 8; ++e) most = max(most, __builtin_bit_cast(uint32_t, x[e]) << 1);
    const Split8 s = split8(x, __any(most >= 0xff000000u));
    uint4 first, second;
    first.x = half ? s.term[1].x : s.term[0].x;
    first.y = half ? s.term[1].y : s.term[0].y;
    first.z = half ? s.term[1].z : s.term[0].z;
    first.w = half ? s.term[1].w : s.term[0].w;
    second.x = half ? 0u : s.term[2].x;
    second.y = half ? 0u : s.term[2].y;
    second.z = half ? 0u : s.term[2].z;
    second.w = half ? 0u : s.term[2].w;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const uint4 a = w.w1[t][lane & 31];
        z[t] = mfma_bf16(a, second, units_of(w.b1, t, half));
        z[t] = mfma_bf16(a, first, z[t]);
    }
}

// out[ti] += sum over input units of M(., unit) in(unit); the smaller terms first
__device__ __forceinline__ void layer64(const uint4 (&m)[2][2][2][64], int lane, const f32x16 (&in)[2],
                                        f32x16 (&out)[2]) {
    Split8 s[2][2];
    int most = 0;   // of the bits: infinities (the GELU's are positive) and NaN are the largest
#pragma unroll
    for (int tk = 0; tk < 2; ++tk)
#pragma unroll
        for (int r = 0; r < 16; ++r) most = max(most, __builtin_bit_cast(int, in[tk][r]));
    const bool infinite = __any(most >= 0x7f800000);
#pragma unroll
    for (int tk = 0; tk < 2; ++tk)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = in[tk][8 * p + e];
            s[tk][p] = split8(v, infinite);
        }
#pragma unroll
    for (int q = 2; q >= 0; --q)
#pragma unroll
        for (int tk = 0; tk < 2; ++tk)
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int ti = 0; ti < 2; ++ti) out[ti] = mfma_bf16(m[ti][tk][p][lane], s[tk][p].term[q], out[ti]);
}

// The same with float32 products; x: the lane's four features.
__device__ __forceinline__ void layer1(const MlpGradWeights& w, int lane, const f32x4u x, f32x16 (&z)[2]) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const float4 a = w.w1[t][lane];
        z[t] = mfma_f32(a.x, x[0], units_of(w.b1, t, lane >> 5));
        z[t] = mfma_f32(a.y, x[1], z[t]);
        z[t] = mfma_f32(a.z, x[2], z[t]);
        z[t] = mfma_f32(a.w, x[3], z[t]);
    }
}
__device__ __forceinline__ void layer64(const float4 (&m)[2][2][4][64], int lane, const f32x16 (&in)[2],
                                        f32x16 (&out)[2]) {
#pragma unroll
    for (int tk = 0; tk < 2; ++tk)
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int ti = 0; ti < 2; ++ti) {
                const float4 q = m[ti][tk][a][lane];
                out[ti] = mfma_f32(q.x, in[tk][4 * a], out[ti]);
                out[ti] = mfma_f32(q.y, in[tk][4 * a + 1], out[ti]);
                out[ti] = mfma_f32(q.z, in[tk][4 * a + 2], out[ti]);
                out[ti] = mfma_f32(q.w, in[tk][4 * a + 3], out[ti]);
            }
}

// A sample's features.
__device__ __forceinline__ void load_features(const float* __restrict__ X, int64_t s, float (&x)[8]) {
    const f32x4u a = *(const f32x4u*)(X + s * 8), b = *(const f32x4u*)(X + s * 8 + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        x[e] = a[e];
        x[4 + e] = b[e];
    }
}

// The lane index, re-formed where a loop's body takes its weights from LDS: the loads would
// otherwise be hoisted out of the loop and spill.
__device__ __forceinline__ int fresh_lane() {
    int l = threadIdx.x & 63;
    asm volatile("" : "+v"(l));
    return l;
}

// Sum of v over the two halves of the wave, in both.
__device__ __forceinline__ float both_halves(float v) { return v + __shfl_xor(v, 32, 64); }

template <bool EXP>
__global__ void __launch_bounds__(256, 3) mlp_forward_kernel(const uint16_t* __restrict__ wbf,
                                                             const float* __restrict__ X, int64_t N,
                                                             float* __restrict__ out) {
    __shared__ MlpWeights w;
    stage_weights(w, wbf);
    __syncthreads();
    const int col = threadIdx.x & 31;
    const int64_t stride = (int64_t)gridDim.x * 4 * 32;
    int64_t s = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 32 + col;
    float x[8];
    load_features(X, min(s, N - 1), x);
    for (; s - col < N; s += stride) {
        const int lane = fresh_lane(), half = lane >> 5;
        f32x16 h[2], z[2];
        layer1(w, lane, x, h);
        load_features(X, min(s + stride, N - 1), x);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int r = 0; r < 16; ++r) h[t][r] = gelu_f(h[t][r]);
            z[t] = units_of(w.b2, t, half);
        }
        layer64(w.w2, lane, h, z);
        float o[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const f32x16 w3 = units_of(w.w3, t, half);
#pragma unroll
            for (int r = 0; r < 16; ++r) o[r % 4] = fmaf(w3[r], gelu_f(z[t][r]), o[r % 4]);
        }
        const float v = both_halves((o[0] + o[1]) + (o[2] + o[3])) + w.b3;
        if (half == 0 && s < N) out[s] = EXP ? expf(v) : v;
    }
}

// Per-wave scratch: 64 units x 32 samples of two arrays and the 8 features, rows padded so
// that reads of 16 consecutive samples by 32 units do not collide.
constexpr int MLP_PITCH = 36;
struct MlpScratch {
    alignas(16) float d[64 * MLP_PITCH];   // dz2, then dz1
    alignas(16) float h[64 * MLP_PITCH];   // h1
    alignas(16) float x[8 * MLP_PITCH];
};
struct MlpGradLds {
    MlpGradWeights w;
    MlpScratch scratch[4];
};

// Row `row` of a scratch array: the 16 samples of this lane's half (the products take
// sample 16 half + t at step t).
__device__ __forceinline__ void read_samples(const float* rows, int row, int half, float (&v)[16]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float4 u = *(const float4*)(rows + row * MLP_PITCH + 16 * half + 4 * q);
        v[4 * q] = u.x;
        v[4 * q + 1] = u.y;
        v[4 * q + 2] = u.z;
        v[4 * q + 3] = u.w;
    }
}

// Sums v (one value per sample and unit register) over the samples: lane u returns unit u's.
__device__ __forceinline__ float sum_samples(float* rows, int lane, const f32x16 (&v)[2]) {
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            rows[(32 * t + 8 * (r / 4) + 4 * (lane >> 5) + r % 4) * MLP_PITCH + (lane & 31)] = v[t][r];
    __builtin_amdgcn_wave_barrier();
    float s0 = 0.f, s1 = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const float4 u = *(const float4*)(rows + lane * MLP_PITCH + 4 * q);
        s0 += u.x + u.y;
        s1 += u.z + u.w;
    }
    __builtin_amdgcn_wave_barrier();
    return s0 + s1;
}

// `scale` times half the gradient of the sum of squared residuals over the wave's samples:
// partial[wave] = the NP gradients, then the sum of squared residuals.  The scale is the power
// of two in 2 / N, so that the sums stay in range where the gradient does; the rest comes in
// float64 with the sum of the partials (all of 2 / N rounded to float32 was an error common to
// all: 4.8e-8 at N = 1,000).  A wave takes `per` samples at a time, 32 but for the smallest batches
// (mlp_grad_impl): it sums them in float32, and with few of them nothing averages that.
// Relative error of the gradient at N = 64, 1,000, 8,000 and 65,536 (medians and root mean
// squares over random networks): 7.6e-8, 3.6e-8, 2.7e-8 and 2.4e-8; of the former kernel, one
// sample per wave at a time, 7.4e-8, 5.6e-8, 4.5e-8 and 2.8e-8.
__global__ void __launch_bounds__(256, 1) mlp_grad_kernel(const uint16_t* __restrict__ wbf, const float* __restrict__ X,
                                                          const float* __restrict__ target, int64_t N, int per,
                                                          float scale, float* __restrict__ partial) {
    extern __shared__ unsigned char mlp_sh[];
    MlpGradLds& lds = *(MlpGradLds*)mlp_sh;
    const MlpGradWeights& w = lds.w;
    stage_weights(lds.w, wbf);
    __syncthreads();
    const int lane0 = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane0 & 31;
    MlpScratch& sc = lds.scratch[wave];
    f32x16 g2[2][2], g1[2], gw3[2], gb2[2], gb1[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) g2[0][t][r] = g2[1][t][r] = g1[t][r] = gw3[t][r] = gb2[t][r] = gb1[t][r] = 0.f;
    float gb3 = 0.f, lsum = 0.f;
    const int64_t gw = (int64_t)blockIdx.x * 4 + wave, stride = (int64_t)gridDim.x * 4 * per;
    for (int64_t s = gw * per + col; s - col < N; s += stride) {
        const int lane = fresh_lane(), half = lane >> 5;
        const bool valid = col < per && s < N;
        const f32x4u x = *(const f32x4u*)(X + min(s, N - 1) * 8 + 4 * half);
        const float tgt = target[min(s, N - 1)];
        f32x16 h[2], z[2], d1[2], d2[2];   // d1, d2: the derivatives of both GELUs, then dz1, dz2
        layer1(w, lane, x, h);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int t = 0; t < 4; ++t) sc.x[(4 * half + t) * MLP_PITCH + col] = x[t];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float g;
                h[t][r] = gelu_with_grad(h[t][r], g);
                d1[t][r] = g;
                sc.h[(32 * t + 8 * (r / 4) + 4 * half + r % 4) * MLP_PITCH + col] = h[t][r];
            }
            z[t] = units_of(w.b2, t, half);
        }
        layer64(w.w2, lane, h, z);
        float o[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const f32x16 w3 = units_of(w.w3, t, half);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float g;
                z[t][r] = gelu_with_grad(z[t][r], g);   // h2
                d2[t][r] = w3[r] * g;
                o[r % 4] = fmaf(w3[r], z[t][r], o[r % 4]);
            }
        }
        const float res = valid ? both_halves((o[0] + o[1]) + (o[2] + o[3])) + w.b3 - tgt : 0.f;
        const float dout = res * scale;
        lsum = fmaf(res, res, lsum);
        gb3 += dout;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                gw3[t][r] = fmaf(dout, z[t][r], gw3[t][r]);
                d2[t][r] *= dout;                        // dz2
                gb2[t][r] += d2[t][r];
                sc.d[(32 * t + 8 * (r / 4) + 4 * half + r % 4) * MLP_PITCH + col] = d2[t][r];
            }
        __builtin_amdgcn_wave_barrier();
        // dW2 += dz2 h1^T over the samples
        {
            float da[2][16], hb[2][16];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                read_samples(sc.d, 32 * t + col, half, da[t]);
                read_samples(sc.h, 32 * t + col, half, hb[t]);
            }
#pragma unroll
            for (int q = 0; q < 16; ++q)
#pragma unroll
                for (int ti = 0; ti < 2; ++ti)
#pragma unroll
                    for (int tj = 0; tj < 2; ++tj) g2[ti][tj] = mfma_f32(da[ti][q], hb[tj][q], g2[ti][tj]);
        }
        // dh1 = W2^T dz2, dz1 = dh1 gelu'(z1)
        f32x16 dh[2];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) dh[t][r] = 0.f;
        layer64(w.w2t, lane, d2, dh);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                d1[t][r] *= dh[t][r];
                gb1[t][r] += d1[t][r];
                sc.d[(32 * t + 8 * (r / 4) + 4 * half + r % 4) * MLP_PITCH + col] = d1[t][r];
            }
        __builtin_amdgcn_wave_barrier();
        // dW1 += dz1 x^T over the samples (8 columns of the tile)
        {
            float da[2][16], xb[16];
            read_samples(sc.x, col % 8, half, xb);
#pragma unroll
            for (int t = 0; t < 2; ++t) read_samples(sc.d, 32 * t + col, half, da[t]);
#pragma unroll
            for (int q = 0; q < 16; ++q)
#pragma unroll
                for (int t = 0; t < 2; ++t) g1[t] = mfma_f32(da[t][q], xb[q], g1[t]);
        }
        __builtin_amdgcn_wave_barrier();
    }
    const int lane = lane0, half = lane >> 5;
    float* P = partial + gw * (NP + 1);
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int u = 32 * ti + 8 * (r / 4) + 4 * half + r % 4;
            if (col < 8) P[OFF_W1 + u * 8 + col] = g1[ti][r];
            P[OFF_W2 + u * 64 + col] = g2[ti][0][r];
            P[OFF_W2 + u * 64 + 32 + col] = g2[ti][1][r];
        }
    P[OFF_B1 + lane] = sum_samples(sc.d, lane, gb1);
    P[OFF_B2 + lane] = sum_samples(sc.d, lane, gb2);
    P[OFF_W3 + lane] = sum_samples(sc.d, lane, gw3);
    for (int off = 16; off > 0; off >>= 1) {   // both halves hold the same samples
        gb3 += __shfl_xor(gb3, off, 64);
        lsum += __shfl_xor(lsum, off, 64);
    }
    if (lane == 0) {
        P[OFF_B3] = gb3;
        P[NP] = lsum;
    }
}

// grad[p] = sum over waves (float64, in a fixed order: 32 interleaved sums, then those in
// order); optional Adam step on the master weights.  A workgroup is 32 parameters x 32
// sums (one thread per parameter took 252 us: its 1024 loads queued behind one another).
constexpr int RED_ENTRIES = 32, RED_SEGS = 32;
__global__ void __launch_bounds__(RED_ENTRIES* RED_SEGS) mlp_reduce_adam(
    const float* __restrict__ partial, int nwaves, float* __restrict__ grad, float* __restrict__ loss,
    float* __restrict__ master, float* __restrict__ m1, float* __restrict__ m2, uint16_t* __restrict__ wbf, int step,
    float lr, double inv_n, double factor, int update) {
    __shared__ double sh[RED_SEGS][RED_ENTRIES + 1];
    const int px = threadIdx.x % RED_ENTRIES, seg = threadIdx.x / RED_ENTRIES;
    const int p = blockIdx.x * RED_ENTRIES + px;
    double g = 0.0;
    if (p <= NP)
#pragma unroll 8
        for (int w = seg; w < nwaves; w += RED_SEGS) g += (double)partial[(int64_t)w * (NP + 1) + p];
    sh[seg][px] = g;
    __syncthreads();
    if (seg != 0 || p > NP) return;
    g = 0.0;
#pragma unroll
    for (int i = 0; i < RED_SEGS; ++i) g += sh[i][px];
    if (p == NP) {
        if (loss) loss[0] = (float)(g * inv_n);
        return;
    }
    const float gf = (float)(g * factor);
    if (grad) grad[p] = gf;
    if (!update) return;
    const float beta1 = 0.9f, beta2 = 0.999f, eps = 1e-8f;
    const float a = beta1 * m1[p] + (1.f - beta1) * gf;
    const float b = beta2 * m2[p] + (1.f - beta2) * gf * gf;
    m1[p] = a;
    m2[p] = b;
    const float mhat = a / (1.f - powf(beta1, (float)step));
    const float vhat = b / (1.f - powf(beta2, (float)step));
    const float w = master[p] - lr * mhat / (sqrtf(vhat) + eps);
    master[p] = w;
    wbf[p] = float_to_bf16(w).bits;
}

__global__ void mlp_copy_params(const float* __restrict__ src, float* __restrict__ master, float* __restrict__ m1,
                                float* __restrict__ m2, uint16_t* __restrict__ wbf) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= NP) return;
    const float w = src[p];
    master[p] = w;
    m1[p] = 0.f;
    m2[p] = 0.f;
    wbf[p] = float_to_bf16(w).bits;
}

// Features of point i = (param p, iz, ix) of a field-major model vector.
__global__ void mlp_features_kernel(int64_t nx, int64_t nz, const float* __restrict__ logD,
                                    const float* __restrict__ gabs, float sigma_scale, float* __restrict__ X) {
    const int64_t m = nx * nz, n = 3 * m;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t p = i / m, r = i % m;
        const int64_t iz = r / nx;
        const int64_t q = (p + 1) % 3, u = (p + 2) % 3;
        float* f = X + i * 8;
        f[0] = logD[i];
        f[1] = logD[q * m + r];
        f[2] = logD[u * m + r];
        f[3] = gabs[i];
        f[4] = gabs[q * m + r];
        f[5] = gabs[u * m + r];
        f[6] = nz > 1 ? (float)iz / (float)(nz - 1) : 0.f;
        f[7] = sigma_scale;
    }
}

}  // namespace

struct bfgsuq_mlp {
    hipStream_t stream = nullptr;
    float* master = nullptr;
    float* m1 = nullptr;
    float* m2 = nullptr;
    uint16_t* wbf = nullptr;
    float* partial = nullptr;
    int step = 0;
};

extern "C" {

int bfgs_mlp_destroy(bfgs_mlp_t m) {
    if (!m) return BFGS_OK;
    (void)hipStreamSynchronize(m->stream);
    void* ptrs[] = {m->master, m->m1, m->m2, m->wbf, m->partial};
    for (void* p : ptrs)
        if (p) (void)hipFree(p);
    delete m;
    return BFGS_OK;
}

int bfgs_mlp_create(void* stream, bfgs_mlp_t* out) {
    if (!out) return BFGS_ERR_ARG;
    *out = nullptr;
    bfgsuq_mlp* m = new (std::nothrow) bfgsuq_mlp();
    if (!m) return BFGS_ERR_ALLOC;
    m->stream = (hipStream_t)stream;
    if (hipMalloc(&m->master, NP * 4) != hipSuccess || hipMalloc(&m->m1, NP * 4) != hipSuccess ||
        hipMalloc(&m->m2, NP * 4) != hipSuccess || hipMalloc(&m->wbf, NP * 2) != hipSuccess ||
        hipMalloc(&m->partial, (size_t)MLP_WAVES * (NP + 1) * 4) != hipSuccess) {
        bfgs_mlp_destroy(m);
        return BFGS_ERR_ALLOC;
    }
    if (hipMemsetAsync(m->master, 0, NP * 4, m->stream) != hipSuccess ||
        hipMemsetAsync(m->m1, 0, NP * 4, m->stream) != hipSuccess ||
        hipMemsetAsync(m->m2, 0, NP * 4, m->stream) != hipSuccess ||
        hipMemsetAsync(m->wbf, 0, NP * 2, m->stream) != hipSuccess || hipStreamSynchronize(m->stream) != hipSuccess) {
        bfgs_mlp_destroy(m);
        return BFGS_ERR_HIP;
    }
    *out = m;
    return BFGS_OK;
}

int bfgs_mlp_set_params(bfgs_mlp_t m, const float* params) {
    if (!m || !params) return BFGS_ERR_ARG;
    hipLaunchKernelGGL(mlp_copy_params, dim3((NP + 255) / 256), dim3(256), 0, m->stream, params, m->master, m->m1,
                       m->m2, m->wbf);
    m->step = 0;
    return hipGetLastError() == hipSuccess ? BFGS_OK : BFGS_ERR_HIP;
}

int bfgs_mlp_get_params(bfgs_mlp_t m, float* params) {
    if (!m || !params) return BFGS_ERR_ARG;
    BFGS_HIP(hipMemcpyAsync(params, m->master, NP * 4, hipMemcpyDeviceToDevice, m->stream));
    return BFGS_OK;
}

int bfgs_mlp_features(int64_t nx, int64_t nz, const float* logD, const float* gabs, float sigma_scale, float* X,
                      void* stream) {
    if (nx < 1 || nz < 1 || !logD || !gabs || !X) return BFGS_ERR_ARG;
    const int64_t n = 3 * nx * nz;
    const int grid = (int)std::min<int64_t>(4096, (n + 255) / 256);
    hipLaunchKernelGGL(mlp_features_kernel, dim3(grid), dim3(256), 0, (hipStream_t)stream, nx, nz, logD, gabs,
                       sigma_scale, X);
    return hipGetLastError() == hipSuccess ? BFGS_OK : BFGS_ERR_HIP;
}

int bfgs_mlp_forward(bfgs_mlp_t m, const float* X, int64_t N, float* out, int32_t exp_out) {
    if (!m || !X || !out || N < 1) return BFGS_ERR_ARG;
    const int grid = (int)std::min<int64_t>(3 * MLP_BLOCKS, (N + 127) / 128);   // three waves to a SIMD, 32 samples each
    if (exp_out)
        hipLaunchKernelGGL(mlp_forward_kernel<true>, dim3(grid), dim3(256), 0, m->stream, m->wbf, X, N, out);
    else
        hipLaunchKernelGGL(mlp_forward_kernel<false>, dim3(grid), dim3(256), 0, m->stream, m->wbf, X, N, out);
    return hipGetLastError() == hipSuccess ? BFGS_OK : BFGS_ERR_HIP;
}

static int mlp_grad_impl(bfgs_mlp_t m, const float* X, const float* target, int64_t N, float* grad, float* loss,
                         float lr, int update) {
    static const hipError_t lds_ok = hipFuncSetAttribute(
        (const void*)mlp_grad_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(MlpGradLds));
    if (lds_ok != hipSuccess) return BFGS_ERR_HIP;
    // one wave to a SIMD, 32 samples each; up to 512 samples are dealt to 128 waves (at N = 64
    // the error is 7.6e-8 with one sample to a wave, 9.2e-8 with 32; from 500 on 32 to a wave
    // are as accurate as the former kernel, and 128 partials would take 2 of 20 us more)
    const int per = N <= 512 ? (int)((N + 127) / 128) : 32;
    const int grid = (int)std::min<int64_t>(MLP_BLOCKS, (N + 4 * per - 1) / (4 * per));
    const double two_over_n = 2.0 / (double)N, scale = std::ldexp(1.0, std::ilogb(two_over_n));
    hipLaunchKernelGGL(mlp_grad_kernel, dim3(grid), dim3(256), sizeof(MlpGradLds), m->stream, m->wbf, X, target, N,
                       per, (float)scale, m->partial);
    if (update) ++m->step;
    hipLaunchKernelGGL(mlp_reduce_adam, dim3(ceil_div(NP + 1, RED_ENTRIES)), dim3(RED_ENTRIES * RED_SEGS), 0,
                       m->stream, m->partial, 4 * grid,
                       grad, loss, m->master, m->m1, m->m2, m->wbf, m->step, lr, 1.0 / (double)N,
                       two_over_n / scale, update);
    return hipGetLastError() == hipSuccess ? BFGS_OK : BFGS_ERR_HIP;
}

int bfgs_mlp_grad(bfgs_mlp_t m, const float* X, const float* target, int64_t N, float* grad, float* loss) {
    if (!m || !X || !target || N < 1) return BFGS_ERR_ARG;
    return mlp_grad_impl(m, X, target, N, grad, loss, 0.f, 0);
}

int bfgs_mlp_train_step(bfgs_mlp_t m, const float* X, const float* target, int64_t N, float lr, float* loss) {
    if (!m || !X || !target || N < 1 || !(lr > 0.f)) return BFGS_ERR_ARG;
    return mlp_grad_impl(m, X, target, N, nullptr, loss, lr, 1);
}

}  // extern "C"
