// Device-side helpers shared by the gfx950 kernels of the EAT layer.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "eat_internal.h"

namespace eat {

constexpr int kWave = 64;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int lane_id() { return __lane_id(); }

// Reductions over the 64 lanes of a wave.  Inside each 16-lane row, DPP
// lane swaps (neighbour pairs, quad pairs, then the 8-lane and 16-lane
// mirrors) leave every lane of the row holding the row's total -- the
// partners add a commutative pair, so the row's lanes agree bit for bit;
// then the four row totals, read through SGPRs, are combined in a fixed
// order.  Every lane ends with the same value, the order of operations never
// depends on timing, and no step goes through LDS (a ds_bpermute butterfly
// costs an LDS round trip per step).
template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) {
    return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false);
}
constexpr int kDppXor1 = 0xB1;          // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;          // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141;   // lane i <-> 7 - i within 8
constexpr int kDppMirror = 0x140;       // lane i <-> 15 - i within 16

template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
    return __int_as_float(dpp_i<CTRL>(__float_as_int(v)));
}
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
    const int lo = dpp_i<CTRL>(__double2loint(v)), hi = dpp_i<CTRL>(__double2hiint(v));
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float lane_f(float v, int j) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), j));
}
__device__ __forceinline__ double lane_d(double v, int j) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), j),
                            __builtin_amdgcn_readlane(__double2loint(v), j));
}

__device__ __forceinline__ float wave_sum(float v) {
    v += dpp_f<kDppXor1>(v);
    v += dpp_f<kDppXor2>(v);
    v += dpp_f<kDppHalfMirror>(v);
    v += dpp_f<kDppMirror>(v);
    return (lane_f(v, 0) + lane_f(v, 16)) + (lane_f(v, 32) + lane_f(v, 48));
}
__device__ __forceinline__ double wave_sum(double v) {
    v += dpp_d<kDppXor1>(v);
    v += dpp_d<kDppXor2>(v);
    v += dpp_d<kDppHalfMirror>(v);
    v += dpp_d<kDppMirror>(v);
    return (lane_d(v, 0) + lane_d(v, 16)) + (lane_d(v, 32) + lane_d(v, 48));
}
__device__ __forceinline__ int wave_sum(int v) {
    v += dpp_i<kDppXor1>(v);
    v += dpp_i<kDppXor2>(v);
    v += dpp_i<kDppHalfMirror>(v);
    v += dpp_i<kDppMirror>(v);
    return (__builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16)) +
           (__builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48));
}
__device__ __forceinline__ float wave_max(float v) {
    v = fmaxf(v, dpp_f<kDppXor1>(v));
    v = fmaxf(v, dpp_f<kDppXor2>(v));
    v = fmaxf(v, dpp_f<kDppHalfMirror>(v));
    v = fmaxf(v, dpp_f<kDppMirror>(v));
    return fmaxf(fmaxf(lane_f(v, 0), lane_f(v, 16)), fmaxf(lane_f(v, 32), lane_f(v, 48)));
}

// Inclusive prefix sum over the 64 lanes of a wave, by DPP (rows of 16 by
// shifts, then the row totals passed on): no LDS round trip per step.
__device__ __forceinline__ int wave_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 to rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 to rows 2 and 3
    return v;
}

// Tile table of expert-major row segments: tstart[g] = sum over h < g of
// ceil((offsets[h+1] - offsets[h]) / bm), for g = 0..groups.  Wave 0 reads
// one segment per lane and scans 64 at a time (integer sums, so the order
// does not matter); every thread of the workgroup must call it.  With
// COUNT, `used` (LDS) receives the number of non-empty segments.
template <bool COUNT = false>
__device__ __forceinline__ void tile_starts(const int32_t* offsets, int groups, int bm, int* tstart,
                                            int* used = nullptr) {
    if (threadIdx.x < kWave) {
        const int lane = __lane_id();
        int carry = 0, nonempty = 0;
        for (int g0 = 0; g0 < groups; g0 += kWave) {
            const int g = g0 + lane;
            int c = g < groups ? (offsets[g + 1] - offsets[g] + bm - 1) / bm : 0;
            if constexpr (COUNT) nonempty += __popcll(__ballot(c > 0));
            c = wave_scan(c);
            if (g < groups) tstart[g + 1] = carry + c;
            carry += __builtin_amdgcn_readlane(c, kWave - 1);
        }
        if (lane == 0) {
            tstart[0] = 0;
            if constexpr (COUNT) *used = nonempty;
        }
    }
    __syncthreads();
}

// Segment holding tile `tile` (0 <= tile < tstart[groups]): the first g with
// tstart[g + 1] > tile, by binary search (empty segments are skipped).
__device__ __forceinline__ int tile_group(const int* tstart, int groups, int tile) {
    int lo = 0, hi = groups - 1;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (tstart[mid + 1] > tile) hi = mid;
        else lo = mid + 1;
    }
    return lo;
}

// Lanes of one wave exchanging values through LDS: every lane's stores are
// ordered before the loads that follow (a wave's LDS operations run in
// issue order; the fences keep the compiler from moving them).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Bit e of lane t -> bit t of lane e, over a wave: six exchanges of the halves
// that lanes K apart hold of each other's bits.
template <int K>
__device__ __forceinline__ uint32_t lane_xor(uint32_t x) {
    const int v = static_cast<int>(x);
    if constexpr (K == 1) return dpp_i<kDppXor1>(v);
    else if constexpr (K == 2) return dpp_i<kDppXor2>(v);
    else if constexpr (K == 4) return dpp_i<kDppHalfMirror>(dpp_i<0x1B>(v));   // i ^ 3, then i ^ 7
    else if constexpr (K == 8) return dpp_i<0x128>(v);                         // row_ror:8
    else return static_cast<uint32_t>(__shfl_xor(v, K, kWave));
}
template <int K>
__device__ __forceinline__ uint32_t swap_bits(uint32_t x, bool upper) {
    constexpr uint32_t low = K == 1 ? 0x55555555u : K == 2 ? 0x33333333u : K == 4 ? 0x0f0f0f0fu
                             : K == 8 ? 0x00ff00ffu : 0x0000ffffu;             // bits b with b & K == 0
    const uint32_t y = lane_xor<K>(x);
    return upper ? (x & ~low) | ((y >> K) & low) : (x & low) | ((y & low) << K);
}
__device__ __forceinline__ uint64_t bit_transpose(uint64_t m) {
    const int lane = __lane_id();
    uint32_t lo = static_cast<uint32_t>(m), hi = static_cast<uint32_t>(m >> 32);
    const uint32_t ylo = static_cast<uint32_t>(__shfl_xor(static_cast<int>(lo), 32, kWave));
    const uint32_t yhi = static_cast<uint32_t>(__shfl_xor(static_cast<int>(hi), 32, kWave));
    if (lane & 32) lo = yhi;
    else hi = ylo;
    auto step = [&](auto k) __attribute__((always_inline)) {
        constexpr int K = decltype(k)::value;
        lo = swap_bits<K>(lo, (lane & K) != 0);
        hi = swap_bits<K>(hi, (lane & K) != 0);
    };
    step(std::integral_constant<int, 16>{});
    step(std::integral_constant<int, 8>{});
    step(std::integral_constant<int, 4>{});
    step(std::integral_constant<int, 2>{});
    step(std::integral_constant<int, 1>{});
    return static_cast<uint64_t>(hi) << 32 | lo;
}

// The expert-major rows of a call of up to 64 NC tokens from its selection
// masks ([T][W] words): cols[e * NC + c] holds expert e's tokens among tokens
// 64 c .. 64 c + 63 as bits, soff[e] the first row of its segment.  Every
// thread of the workgroup (NW waves) calls it; cols and soff are LDS.  A lane
// per token, a bit transpose per 64 tokens and mask word, so it costs about
// what reading the arrays of a permutation launch would, whose ~4 us it saves
// (16-layer EAT decode of 64 tokens 1068 -> 1032 us a step, the 32-token fp32
// layer 31 -> 28; layers of big experts within the noise; with a ballot per expert
// in place of the transpose the 64-expert layers gained nothing).
template <int NW, int NC>
__device__ __forceinline__ void build_segments(const uint64_t* __restrict__ mask, int T, int E, int W, uint64_t* cols,
                                               int* soff) {
    const int lane = __lane_id(), wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
    const int nc = (T + kWave - 1) / kWave;
    for (int q = wave; q < NC * W; q += NW) {
        const int c = q % NC, word = q / NC;
        const int t = kWave * c + lane;
        const uint64_t m = c < nc ? mask[static_cast<size_t>(t < T ? t : 0) * W + word] : 0ull;
        const uint64_t mine = bit_transpose(t < T ? m : 0ull);
        const int nb = min(kWave, E - kWave * word);
        if (lane < nb) cols[(kWave * word + lane) * NC + c] = mine;
    }
    __syncthreads();
    if (wave == 0) {
        int carry = 0;
        for (int g0 = 0; g0 < E; g0 += kWave) {
            const int e = g0 + lane;
            int n = 0;
#pragma unroll
            for (int c = 0; c < NC; ++c) n += e < E ? __popcll(cols[e * NC + c]) : 0;
            n = wave_scan(n);
            if (e < E) soff[e + 1] = carry + n;
            carry += __builtin_amdgcn_readlane(n, kWave - 1);
        }
        if (lane == 0) soff[0] = 0;
    }
    __syncthreads();
}

// Token of row r of an expert's segment: the position of the r-th set bit of
// its NC words (0 <= r < their bits; any valid token otherwise).
template <int NC>
__device__ __forceinline__ int nth_token(const uint64_t* col, int r) {
    uint64_t w = col[0];
    int base = 0;
#pragma unroll
    for (int c = 1; c < NC; ++c) {
        const int n = __popcll(w);
        const bool next = r >= n && base == kWave * (c - 1);
        if (next) {
            r -= n;
            w = col[c];
            base = kWave * c;
        }
    }
    const int nl = __popc(static_cast<uint32_t>(w));
    uint32_t v = static_cast<uint32_t>(w);
    int pos = 0;
    if (r >= nl) { r -= nl; v = static_cast<uint32_t>(w >> 32); pos = 32; }
#pragma unroll
    for (int s = 16; s >= 1; s >>= 1) {
        const int n = __popc(v & ((1u << s) - 1u));
        if (r >= n) { r -= n; v >>= s; pos += s; }
    }
    return base + pos;
}

// Writes the arrays the later kernels of the call read, the workgroups taking
// experts in turn (wave 0 of each; after its other work).
template <int NC>
__device__ __forceinline__ void publish_segments(const Segments& g, int E, const uint64_t* cols, const int* soff) {
    if (threadIdx.x >= kWave) return;
    const int lane = __lane_id();
    const uint64_t lt = lane == 0 ? 0ull : ~0ull >> (kWave - lane);
    for (int e = blockIdx.x; e < E; e += gridDim.x) {
        int row0 = soff[e];
        if (lane == 0) {
            g.offsets[e] = row0;
            if (e == E - 1) g.offsets[E] = soff[E];
            if (g.expert_load) g.expert_load[e] = soff[e + 1] - row0;
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const uint64_t w = cols[e * NC + c];
            const int t = kWave * c + lane;
            if ((w >> lane) & 1ull) {
                const int row = row0 + __popcll(w & lt);
                g.tok_idx[row] = t;
                g.inv[static_cast<size_t>(t) * E + e] = row;
            }
            row0 += __popcll(w);
        }
    }
}

// Broadcast lane j's value (j uniform across the wave) through an SGPR.
__device__ __forceinline__ float read_lane(float v, int j) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), j));
}

__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }

__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
    return __uint_as_float(static_cast<uint32_t>(b) << 16);
}
// Round-to-nearest-even fp32 -> bf16 bits; a NaN stays a (quiet) NaN.
// Written as a select, not a branch, so that converting a tile of results
// stays straight-line code.
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
    const uint32_t u = __float_as_uint(f);
    const uint32_t rne = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
    const uint32_t qnan = (u >> 16) | 0x40u;
    return static_cast<uint16_t>((u & 0x7fffffffu) > 0x7f800000u ? qnan : rne);
}

// Two fp32 values -> packed bf16 bits (a in the low half), round to nearest
// even by the hardware conversion (one instruction; NaN stays NaN).
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

__device__ __forceinline__ float silu(float a) { return a / (1.0f + __expf(-a)); }

// Workgroup barrier that only waits for this wave's LDS traffic.  Global
// loads issued before it stay in flight (__syncthreads() would drain them
// with a full fence); the "memory" clobber keeps the compiler from moving
// LDS accesses across it.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Wait until at most N vector-memory operations of this wave are
// outstanding (vmcnt(N); expcnt and lgkmcnt left unconstrained, gfx9
// encoding).  Loads complete in issue order for this counter, so a count of
// the loads issued after the one awaited names it exactly.
template <int N>
__device__ __forceinline__ void wait_vm() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

}  // namespace eat
