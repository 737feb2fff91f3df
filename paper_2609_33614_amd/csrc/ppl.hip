// Perplexity signal for the threshold's performance-based adjustment
// (Sec. 3.3), gfx950.
//
// The LM-head projection z = h W_V^T runs on the MFMA tiles (wide.hip) into
// fp32 rows, or on the streaming kernel (expert.hip) where the reduction is too
// short for them (up to two slices of it, added in order here).
// ppl_kernel, one workgroup per sequence, folds the row into an online
// logsumexp pair (running max, sum of exp(z - max)): a thread's values a block
// at a time, then the wave by butterfly, then the waves in order; its first
// thread forms the NLL from it and z[target] and the sequence's running state in
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

// One workgroup per sequence: 128 KB of logits are a latency and a few us for
// a CU, less than the launch that a split over more workgroups needs to merge
// its parts (16 chunks a row, 256 threads each, and a finishing launch: 14.4 us
// at 64 x 32000 against 6.5).
// The target's logit, on whose rounding the NLL would depend most, is taken
// again from the hidden row and the head's row in fp64 (16 KB, under the logits'
// latency), on both sides of the NLL: the row's logsumexp leaves the target out,
// and NLL = log(1 + exp(rest - z[target])).  It is never negative, and its
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
    const int s = blockIdx.x;
    const float* row = z + static_cast<size_t>(s) * V;
    const int y = target[s];
    const bool known = y >= 0 && y < V;
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
    if (lane_id() == 0) zred[threadIdx.x / kWave] = zt;
    Lse a{-INFINITY, 0.f};
    // (V is a multiple of 64)
    for (int j0 = 4 * threadIdx.x; j0 < V; j0 += 4 * kThreads * kVec) {
        float4 v[kVec];
#pragma unroll
        for (int i = 0; i < kVec; ++i) {
            const int j = j0 + 4 * kThreads * i;
            v[i] = *reinterpret_cast<const float4*>(row + (j < V ? j : j0));
        }
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
        a = lse_merge(a, b);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const Lse b{__shfl_xor(a.m, off, kWave), __shfl_xor(a.s, off, kWave)};
        // merge in a fixed (lower lane first) order so partners agree bit for bit
        a = (lane_id() & off) ? lse_merge(b, a) : lse_merge(a, b);
    }
    if (lane_id() == 0) red[threadIdx.x / kWave] = a;
    __syncthreads();
    if (threadIdx.x != 0) return;
    Lse t = red[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) t = lse_merge(t, red[w]);
    zt = zred[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) zt += zred[w];
    const double rest = static_cast<double>(t.m) + log(static_cast<double>(t.s));
    // (zt - zt is NaN for an infinite target, as its row's logsumexp less itself)
    const double nll = !known ? NAN
                       : zt >= rest ? log1p(exp(rest - zt)) + (zt - zt)
                                    : rest - zt + log1p(exp(zt - rest));
    const double sum = nll_sum[s] + nll;
    const int32_t n = count[s] + 1;
    const double ppl = exp(sum / n);
    trend[s] = n > 1 ? (ppl > ppl_prev[s] ? 1 : -1) : 0;
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
