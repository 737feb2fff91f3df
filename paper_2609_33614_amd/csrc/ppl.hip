// Perplexity signal for the threshold's performance-based adjustment
// (Sec. 3.3), gfx950.
//
// The LM-head projection z = h W_V^T runs on the MFMA tiles (wide.hip) into
// fp32 rows, or on the streaming kernel (expert.hip) where it is the faster or
// the reduction too short for them (up to two slices of it, added in order here).
// ppl_kernel, one workgroup per sequence, folds the row into an online
// logsumexp pair (running max, sum of exp(z - max)): a thread's values a block
// at a time, then the lanes of a wave and then the waves over their maximum; its
// first thread forms the NLL from it and z[target] and the sequence's running state in
// fp64: sum of NLL, token count, perplexity exp(sum / count) and the trend (+1
// rose since the previous token, -1 did not, 0 first token).  Every merge has a
// fixed order, so results are bit-reproducible.
#include <math.h>

#include "eat_device.h"
#include "eat_internal.h"

namespace eat {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / kWave;
// float4s a thread has in flight: a row of 32000 logits is one block of loads
constexpr int kVec = 8;

// online logsumexp pair (m, s): the running max and sum of exp(z - m)
struct Lse {
    float m, s;
};

// exp(v - m) of a value with maximum m (the maximum itself counts 1 also where
// it is infinite)
__device__ __forceinline__ float term(float v, float m) { return v == m ? 1.f : expf(v - m); }

// (a pair of nothing but -inf holds s = 0, or NaN from NaN logits, which stays)
__device__ __forceinline__ Lse lse_merge(Lse a, Lse b) {
    if (a.m < b.m) { const Lse t = a; a = b; b = t; }
    return {a.m, a.s + b.s * term(b.m, a.m)};
}

// The pairs of a wave's lanes, over their maximum.
__device__ __forceinline__ Lse lse_wave(Lse a) {
    const float m = wave_max(a.m);
    return {m, wave_sum(a.s * term(a.m, m))};
}

// One workgroup per sequence: 128 KB of logits are a latency and a few us for
// a CU, less than the launch that a split over more workgroups needs to merge
// its parts.  1 sequence of 32000, 8.2 us, 16 chunks of 256 threads and a finishing
// launch 12.3 (64 sequences 9.6 and 13.5; 1 of 128256 23.7 and 26.6).  What a
// sequence waits for is a chain, so every load that needs no other is issued
// first: with the target, its head row and the state loaded where they are used,
// the waves' pairs merged one by one and a log more, it took 2 us longer.
// The target's logit, on whose rounding the NLL would depend most, is taken
// again from the hidden row and the head's row in fp64 (16 KB, under the logits'
// latency), on both sides of the NLL: the row's logsumexp leaves the target out,
// and NLL = log(1 + exp(rest - z[target])) = log1p(s exp(m - z[target])), or
// m - z[target] + log(s + exp(z[target] - m)) below m.  It is never negative, and its
// error is the rest's times the probability of the rest, however confident the
// prediction.
__global__ __launch_bounds__(kThreads) void ppl_kernel(const float* __restrict__ z, int splits, int64_t stride, int V,
                                                       const uint16_t* __restrict__ h,
                                                       const uint16_t* __restrict__ w_vocab, int d,
                                                       const int32_t* __restrict__ target, double* nll_sum,
                                                       int32_t* count, double* ppl_prev, int8_t* trend,
                                                       float* nll_out) {
    __shared__ Lse red[kWaves];
    __shared__ double zred[kWaves];
    const int s = blockIdx.x, lane = lane_id(), wave = threadIdx.x / kWave;
    const float* row = z + static_cast<size_t>(s) * V;
    const int y = target[s];
    const bool known = y >= 0 && y < V;
    const double sum0 = nll_sum[s], prev = ppl_prev[s];
    const int32_t n0 = count[s];
    // a block of a thread's logits (V is a multiple of 64; columns past V read the block's first)
    auto load = [&](int j0, float4 (&v)[kVec]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kVec; ++i) {
            const int j = j0 + 4 * kThreads * i;
            v[i] = *reinterpret_cast<const float4*>(row + (j < V ? j : j0));
        }
    };
    const int jbeg = 4 * threadIdx.x;
    float4 v[kVec] = {};
    if (jbeg < V) load(jbeg, v);
    double zt = 0.0;
    for (int k = 4 * threadIdx.x; k < d; k += 4 * kThreads) {     // (d is a multiple of 64)
        const uint2 p = *reinterpret_cast<const uint2*>(h + static_cast<size_t>(s) * d + k);
        const uint2 q = *reinterpret_cast<const uint2*>(w_vocab + static_cast<size_t>(known ? y : 0) * d + k);
        const uint32_t pw[2] = {p.x, p.y}, qw[2] = {q.x, q.y};
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            zt = fma(static_cast<double>(__uint_as_float(pw[i] << 16)),
                     static_cast<double>(__uint_as_float(qw[i] << 16)), zt);
            zt = fma(static_cast<double>(__uint_as_float(pw[i] & 0xffff0000u)),
                     static_cast<double>(__uint_as_float(qw[i] & 0xffff0000u)), zt);
        }
    }
    zt = wave_sum(zt);
    Lse a{-INFINITY, 0.f};
    for (int j0 = jbeg; j0 < V; j0 += 4 * kThreads * kVec) {
        for (int sp = 1; sp < splits; ++sp)
#pragma unroll
            for (int i = 0; i < kVec; ++i) {
                const int j = j0 + 4 * kThreads * i;
                const float4 q = *reinterpret_cast<const float4*>(row + sp * stride + (j < V ? j : j0));
                v[i].x += q.x; v[i].y += q.y; v[i].z += q.z; v[i].w += q.w;
            }
#pragma unroll
        for (int i = 0; i < kVec; ++i) {
            const int at = (known ? y : -1) - (j0 + 4 * kThreads * i);     // the target counts as no logit
            if (at == 0) v[i].x = -INFINITY;
            if (at == 1) v[i].y = -INFINITY;
            if (at == 2) v[i].z = -INFINITY;
            if (at == 3) v[i].w = -INFINITY;
        }
        Lse b{-INFINITY, 0.f};
#pragma unroll
        for (int i = 0; i < kVec; ++i)
            if (j0 + 4 * kThreads * i < V) b.m = fmaxf(b.m, fmaxf(fmaxf(v[i].x, v[i].y), fmaxf(v[i].z, v[i].w)));
#pragma unroll
        for (int i = 0; i < kVec; ++i)
            if (j0 + 4 * kThreads * i < V)
                b.s += (term(v[i].x, b.m) + term(v[i].y, b.m)) + (term(v[i].z, b.m) + term(v[i].w, b.m));
        if (b.m == -INFINITY) b.s -= b.s;     // no logit above -inf: 0, or NaN
        const int jn = j0 + 4 * kThreads * kVec;
        if (jn < V) load(jn, v);
        a = lse_merge(a, b);
    }
    a = lse_wave(a);
    if (lane == 0) {
        red[wave] = a;
        zred[wave] = zt;
    }
    __syncthreads();
    if (wave != 0) return;
    a = lane < kWaves ? red[lane] : Lse{-INFINITY, 0.f};
    zt = wave_sum(lane < kWaves ? zred[lane] : 0.0);
    a = lse_wave(a);
    if (lane != 0) return;
    const double m = static_cast<double>(a.m), rest = static_cast<double>(a.s);
    // (zt - zt is NaN for an infinite target, as its row's logsumexp less itself)
    const double nll = !known ? NAN
                       : zt >= m ? log1p(rest * exp(m - zt)) + (zt - zt)
                                 : m - zt + log(rest + exp(zt - m));
    const double sum = sum0 + nll;
    const int32_t n = n0 + 1;
    const double ppl = exp(sum / n);
    trend[s] = n > 1 ? (ppl > prev ? 1 : -1) : 0;
    nll_sum[s] = sum;
    count[s] = n;
    ppl_prev[s] = ppl;
    if (nll_out) nll_out[s] = static_cast<float>(nll);
}

__global__ __launch_bounds__(kThreads) void ppl_reset_kernel(int S, double* nll_sum, int32_t* count,
                                                             double* ppl_prev) {
    const int s = blockIdx.x * kThreads + threadIdx.x;
    if (s < S) { nll_sum[s] = 0.0; count[s] = 0; ppl_prev[s] = 0.0; }
}

}  // namespace

hipError_t launch_ppl(const float* z, int splits, int64_t stride, int32_t S, int V, const uint16_t* h,
                      const uint16_t* w_vocab, int d, const int32_t* target,
                      double* nll_sum, int32_t* count, double* ppl_prev, int8_t* trend, float* nll_out,
                      hipStream_t s) {
    ppl_kernel<<<S, kThreads, 0, s>>>(z, splits, stride, V, h, w_vocab, d, target, nll_sum, count, ppl_prev, trend, nll_out);
    return hipGetLastError();
}

hipError_t launch_ppl_reset(int32_t S, double* nll_sum, int32_t* count, double* ppl_prev, hipStream_t s) {
    ppl_reset_kernel<<<(S + kThreads - 1) / kThreads, kThreads, 0, s>>>(S, nll_sum, count, ppl_prev);
    return hipGetLastError();
}

}  // namespace eat
