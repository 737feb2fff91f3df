// MFMA tiles for grouped GEMMs over many tokens (gfx950): calls of more than
// 64 tokens.
//
// A workgroup of 8 waves owns a tile of TM token rows x NW weight rows (the
// gated projection: NW / 2 rows of W1 and the matching ones of W3) of one
// expert and walks the reduction dimension in 64-wide chunks (128-byte rows)
// through a ring of LDS stages filled by direct global->LDS loads, several
// chunks ahead of the one it computes with v_mfma_f32_32x32x16_bf16 (weights
// as A, tokens as B: a lane ends with 4 consecutive output features of one
// token).  The waves of a SIMD cover different token groups of the tile, and
// lanes whose token row is past the expert's load nothing, so a tile that
// holds fewer rows costs fewer loads and MFMAs.
//
// Three tiles (measured on the expert loads of real calls; up/gate us):
//   Wide 256 x 256, 2 stages: prefill-sized calls (hundreds of rows per
//     expert).  64 experts of ~512 rows: 345 us; the 256 x 128 tile 353, the
//     128 x 128 one 440.  Bound by the operand bytes a CU pulls through its vector
//     L1: the tile moves about 33 GB/s per CU however deep the ring (a probe of
//     such loads alone, L2 hits and misses mixed, all CUs, 45), and only a
//     larger tile area needs fewer bytes.
//   Tall 256 x 128, 3 stages: about 100 rows per expert and up.  8 experts of
//     ~125 rows, 14336 x 4096: 478-497 us against 520-560 with the 128 x 128
//     tile, which reads the weights of an expert with more than 128 rows twice.
//   Mid 128 x 128, 4 stages: fewer rows per expert, or too few Tall items for
//     the CUs.  60 experts of ~13 rows: 126 us against 151; 8 experts of 256
//     rows (d 2048, F 1024): 31 against 38.
// Against the streaming kernel (expert.hip) with 128-token tiles, whose waves
// keep 24 KB of weights in flight per CU: qwen3-shaped 1000-token Top-K call,
// whole layer, 379 -> 316 us; shared-expert layer's 128-token Top-P decode
// 316 -> 250; fine-grained 256-token EAT decode 94 -> 81.
//
// The grid is persistent: the work list (per expert, its weight tiles in
// turn and each one's token tiles adjacent) is cut into contiguous parts,
// one per XCD (workgroups are dealt to XCDs round-robin), so the workgroups
// that share an expert's weight tiles share one L2 and read them together.
// A workgroup's ring runs on from one item to the next, so the refill after
// an item overlaps its output stores.
#include <type_traits>

#include "eat_device.h"
#include "eat_internal.h"

namespace eat {
namespace {

constexpr int kBK = 64;                   // reduction chunk per stage (bf16 elements)
constexpr int kRB = kBK * 2;              // bytes per LDS row
constexpr int kVPR = kBK / 8;             // 16-byte vectors per row
constexpr int kRPB = 1024 / kRB;          // rows per 1 KB DMA block

// A tile: TM token rows x NW weight rows per workgroup, WT x WW waves over
// them, a ring of STAGES chunks in LDS.
template <int TM_, int NW_, int WT_, int WW_, int STAGES_, bool NT_>
struct Tile {
    static constexpr bool NT = NT_;
    static constexpr int TM = TM_, NW = NW_, WT = WT_, WW = WW_, STAGES = STAGES_;
    static constexpr int kWaves = WT * WW;
    static constexpr int kThreads = kWaves * kWave;
    static constexpr int TF = TM / (32 * WT);     // 32-row token fragments per wave
    static constexpr int WF = NW / (32 * WW);     // 32-row weight fragments per wave
    static constexpr int kRegion = TM * kRB;      // bytes of a stage's token rows
    static constexpr int kStage = (TM + NW) * kRB;
    static constexpr int kBT = TM / kRPB / kWaves;        // 1 KB token blocks per wave and stage
    static constexpr int kBW = NW / kRPB / kWaves;        // weight blocks
    static constexpr int kBPW = kBT + kBW;
    static constexpr int kP = STAGES - 1;         // chunks in flight ahead of the one computed
    static_assert(kBT * kRPB * kWaves == TM && kBW * kRPB * kWaves == NW, "blocks split evenly over the waves");
    static_assert(TF * 32 * WT == TM && WF * 32 * WW == NW && WF % 2 == 0, "fragments cover the tile");
    static_assert(kP >= 1 && kP <= 3, "wait counts cover up to three chunks in flight");
};

// (Wide's weights at device scope: every weight line serves several token
// tiles, and non-temporal loads cost it 3-5%; the other tiles' are read once or
// twice and stream past the caches.)
using Wide = Tile<256, 256, 2, 4, 2, false>;
using Tall = Tile<256, 128, 4, 2, 3, true>;
using Mid = Tile<128, 128, 4, 2, 4, true>;

struct WideArgs {
    const uint16_t* wa;        // [groups][M][K]  (W1, or W2 for the plain projection)
    const uint16_t* wb;        // [groups][M][K]  (W3, gated only)
    const uint16_t* src;       // activation rows, K wide
    const int32_t* gather;     // row -> source row, or null (identity)
    const int32_t* offsets;    // [groups+1] expert-major row offsets, or null
    int groups, nrows, M, K;
    void* out;                 // gated: bf16 H [rows][M]; plain: fp32 [rows][M] (bf16 with ROWS)
    float* nrm2;               // plain with ROWS: [rows][M / 32] sums of squares of 32 features of each row
    int xcds;                  // XCDs the grid is dealt over (the grid is a multiple of it)
    int max_splits;            // plain fp32: most slices of the reduction dimension (tile_split)
    int64_t split_stride;      // elements between slices of out
    int32_t* splits_out;       // the slices taken, written by workgroup 0 (or null)
    Segments seg;              // gated: set when this launch works out the permutation
};

// Byte offset of 16-byte vector v of row r in a region of kRB-byte rows.
// An MFMA operand read takes one vector of 16 consecutive rows per pass of
// the 64 LDS banks (256 bytes = kRowsPerLine rows); the XOR of the vector
// index with the row's line number spreads those 16 rows over distinct
// banks.
constexpr int kRowsPerLine = 256 / kRB;
// (unsigned: a signed division by the power of two costs a rounding fix-up
// and, in the wide kernel, the registers that then spill)
__device__ __forceinline__ int swz(int r) { return (static_cast<unsigned>(r) / kRowsPerLine) & (kVPR - 1); }
__device__ __forceinline__ int wswz(int r, int v) { return r * kRB + ((v ^ swz(r)) << 4); }

// The same for weight rows, which packed weights keep in LDS in their own
// order (pack.hip): a 1 KB block per 16 rows and 32 reduction elements, a
// fragment of 16 consecutive rows one line.  A load instruction then copies one
// contiguous kilobyte; gathered into 128-byte rows, every lane of a quad
// fetched from another line, and packed weights were slower than row-major
// ones (8 experts, 1024 EAT tokens on Wide tiles 893 against 832 us, now 836; 256
// Top-K tokens on Mid tiles 551 against 521, now 524).
template <bool PACKED>
__device__ __forceinline__ int weight_at(int r, int v) {
    return PACKED ? (((r >> 4) * 2 + (v >> 2)) << 10) + (((v & 3) * 16 + (r & 15)) << 4) : wswz(r, v);
}

// One work item: token rows [r0, r0 + n) of expert e's segment against the
// expert's weight rows from m0 (W1 and W3 rows m0.. in the gated tile), over
// reduction slice sp.
struct Item {
    int e, r0, n, m0, sp;
};

// Lane l of a DMA instruction writes LDS bytes [16 l, 16 l + 16) of its 1 KB
// block = row l / kVPR, slot l % kVPR; it fetches the global vector that
// belongs in that slot under the swizzle (packed weights, weight block b: vector
// l of 16-row group b / 2 and k-step b % 2).  Token blocks have a 64-bit source per
// lane (rows are gathered), weight blocks hold rows of expert e -- one matrix per block (W1 or W3 in the gated tile), so the
// block's base is uniform and each lane keeps a 32-bit element offset into
// the expert's matrix (M K < 2^31, checked on the host).
template <class C>
struct ItemLoads {
    const uint16_t* srct[C::kBT];
    uint64_t tmask[C::kBT];               // lanes whose token row is in the item
    uint32_t woff[C::kBW];
    const uint16_t* wbase[C::kBW];
};

// The source row of each of this lane's token blocks (rows past the expert's
// segment load a valid row; their results are unused).  Issued an item
// ahead, so the index loads complete under the previous item's chunks.
template <class C>
__device__ __forceinline__ void token_rows(const WideArgs& a, const Item& it, int (&srow)[C::kBT]) {
    const int lane = lane_id(), wave = threadIdx.x / kWave;
#pragma unroll
    for (int j = 0; j < C::kBT; ++j) {
        const int r = kRPB * (wave + C::kWaves * j) + lane / kVPR;
        const int g = r < it.n ? it.r0 + r : it.r0;
        srow[j] = a.gather ? a.gather[g] : g;
    }
}

template <class C, bool GATED, bool PACKED>
__device__ __forceinline__ ItemLoads<C> item_loads(const WideArgs& a, const Item& it, int kbeg,
                                                   const int (&srow)[C::kBT]) {
    const int lane = lane_id(), wave = threadIdx.x / kWave;
    const int slot = lane % kVPR;
    ItemLoads<C> L;
    const size_t emat = static_cast<size_t>(it.e) * a.M * a.K;
#pragma unroll
    for (int j = 0; j < C::kBT; ++j) {
        const int r = kRPB * (wave + C::kWaves * j) + lane / kVPR;
        const int v = slot ^ swz(r);
        L.tmask[j] = ballot(r < it.n);
        L.srct[j] = a.src + static_cast<size_t>(srow[j]) * a.K + kbeg + 8 * v;
    }
#pragma unroll
    for (int j = 0; j < C::kBW; ++j) {
        const int b = wave + C::kWaves * j;
        const int rb0 = PACKED ? 16 * (b / 2) : kRPB * b;     // the block's first weight row
        // (a last tile past M, where M is not a multiple of NW, loads rows of
        // the matrix again; their results are not stored)
        if constexpr (PACKED) {
            const int row = min(it.m0 + (GATED ? (rb0 & (C::NW / 2 - 1)) : rb0), a.M - 16);
            L.woff[j] = static_cast<uint32_t>(((row / 16) * (a.K / 32) + kbeg / 32 + (b & 1)) * 512 + 8 * lane);
        } else {
            const int r = rb0 + lane / kVPR;
            const int row = min(it.m0 + (GATED ? (r & (C::NW / 2 - 1)) : r), a.M - 1);
            L.woff[j] = static_cast<uint32_t>(row * a.K + kbeg + 8 * (slot ^ swz(r)));
        }
        L.wbase[j] = (GATED && rb0 >= C::NW / 2 ? a.wb : a.wa) + emat;
    }
    return L;
}

// Chunk c of an item into LDS stage st.  asm keeps the compiler from adding
// waits of its own for these loads; the ring's waits and barriers order
// them.  Weight blocks load non-temporally (NT) or at device scope (sc1: no
// allocation in the CU's vector L1 -- a weight line is read once per
// workgroup); token rows keep the default policy.
template <class C, bool PACKED>
__device__ __forceinline__ void issue_weights(const ItemLoads<C>& L, uint8_t* st, int c) {
    // elements a lane's source moves per chunk: row-major weights by the
    // chunk width, packed weights by its 512-element blocks
    constexpr int wstep = PACKED ? (kBK / 32) * 512 : kBK;
    const int wave = threadIdx.x / kWave;
#pragma unroll
    for (int j = 0; j < C::kBW; ++j) {
        const uint16_t* src = L.wbase[j] + L.woff[j] + static_cast<size_t>(c) * wstep;
        const uint32_t lds = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(
            reinterpret_cast<uintptr_t>(st + C::kRegion + 1024 * (wave + C::kWaves * j))));
        if constexpr (C::NT)
            asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off nt"
                         :: "v"(src), "s"(lds) : "memory", "m0");
        else
            asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off sc1"
                         :: "v"(src), "s"(lds) : "memory", "m0");
    }
}
// Token rows of the chunk; lanes whose row is past the item's load nothing
// (an instruction without lanes still counts as one load of the wave, so the
// waits below are constants).
template <class C>
__device__ __forceinline__ void issue_tokens(const ItemLoads<C>& L, uint8_t* st, int c) {
    const int wave = threadIdx.x / kWave;
#pragma unroll
    for (int j = 0; j < C::kBT; ++j) {
        const uint16_t* src = L.srct[j] + static_cast<size_t>(c) * kBK;
        const uint32_t lds = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(
            reinterpret_cast<uintptr_t>(st + 1024 * (wave + C::kWaves * j))));
        uint64_t save;
        asm volatile("s_mov_b64 %0, exec\n\ts_mov_b64 exec, %3\n\ts_mov_b32 m0, %2\n\t"
                     "global_load_lds_dwordx4 %1, off\n\ts_mov_b64 exec, %0"
                     : "=&s"(save) : "v"(src), "s"(lds), "s"(L.tmask[j]) : "memory", "m0");
    }
}
template <class C, bool PACKED>
__device__ __forceinline__ void issue_chunk(const ItemLoads<C>& L, uint8_t* st, int c) {
    issue_tokens<C>(L, st, c);
    issue_weights<C, PACKED>(L, st, c);
}

// Waits until at most `after` chunks' loads of this wave, and `stores` output
// stores issued since, are still in flight (vector memory operations complete
// in issue order for this counter; counting fewer only waits longer).
template <class C>
__device__ __forceinline__ void wait_chunks(int after, int stores) {
    auto wait = [&](auto n) __attribute__((always_inline)) {
        constexpr int N = decltype(n)::value;
        if (stores == 0) wait_vm<N>();
        else if (stores < 4) wait_vm<N + 1>();
        else if (stores < 8) wait_vm<N + 4>();
        else if (stores < 16) wait_vm<N + 8>();
        else wait_vm<N + 16>();
    };
    if (C::kP >= 3 && after >= 2) wait(std::integral_constant<int, (C::kP >= 3 ? 2 : 0) * C::kBPW>{});
    else if (C::kP >= 2 && after >= 1) wait(std::integral_constant<int, (C::kP >= 2 ? 1 : 0) * C::kBPW>{});
    else wait(std::integral_constant<int, 0>{});
}

// a / (1 + e^-a) with the hardware reciprocal (1 ulp) for the tiles' hidden
// values, which are rounded to bf16 at once: the IEEE division's scaling and
// refinement took 11 of a value's ~20 instructions, and every wave of a
// workgroup runs its epilogue in the same moment (64 experts of ~512 rows, up/gate
// 354 -> 344 us).  Over all fp32 values it is off by at most 1.9e-7 of the result
// above -1 (the division 1.5e-7), 5.6e-7 (5.4e-7) down to -8 and the same below,
// where e^-a carries the error; bf16 rounds by 3.9e-3, and the layers' error
// against 64 bits is unchanged.  Both factors are scaled by 1/4: the reciprocal
// returns no denormals, and 1 / (1 + e^-a) is one from -87.4 on, where the result
// still is not.  Overflow and non-finite inputs come out as with the division
// (e^-a = inf gives -0, a = -inf NaN).
__device__ __forceinline__ float silu_rcp(float a) {
    return 0.25f * a * __builtin_amdgcn_rcpf(fmaf(0.25f, __expf(-a), 0.25f));
}

// ROWS (plain tiles): the output rows are stored in bf16, and each lane
// writes the sum of squares of the 32 output features it holds of a row
// (half of its wave's 64), taken from the fp32 accumulators (the row norms
// of the account update).
template <bool GATED, class C, bool PACKED, bool ROWS = false>
__global__ __launch_bounds__(C::kThreads) void wide_kernel(WideArgs a) {
    constexpr int TM = C::TM, NW = C::NW, TF = C::TF, WF = C::WF;
    __shared__ __attribute__((aligned(1024))) uint8_t ring[C::STAGES * C::kStage];
    __shared__ int tstart[kMaxExperts + 1];
    __shared__ int soff[kMaxExperts + 1];     // the segment offsets, read per item without a memory wait
    // (the prefill tile's calls come with the permutation launch, whatever their size)
    constexpr bool kFuse = GATED && C::TM * C::NW < 256 * 256;
    constexpr int NC = kFusedTokens / kWave;
    __shared__ uint64_t cols[kFuse ? kMaxExperts * NC : 1];
    const bool fused = kFuse && a.seg.mask != nullptr;

    int ntiles;
    if (a.offsets) {
        if (fused) {
            build_segments<C::kWaves, NC>(a.seg.mask, a.seg.T, a.groups, a.seg.words, cols, soff);
            tile_starts(soff, a.groups, TM, tstart);     // ends with a barrier
        } else {
            for (int g = threadIdx.x; g <= a.groups; g += C::kThreads) soff[g] = a.offsets[g];
            tile_starts(a.offsets, a.groups, TM, tstart);
        }
        ntiles = tstart[a.groups];
    } else {
        ntiles = (a.nrows + TM - 1) / TM;
    }
    constexpr int kOut = GATED ? NW / 2 : NW;       // output features per tile
    const int nxm = (a.M + kOut - 1) / kOut;
    int splits = 1;
    if constexpr (!GATED && !ROWS) {
        splits = tile_split(static_cast<int64_t>(ntiles) * nxm, a.K, a.max_splits,
                            a.offsets ? a.offsets[a.groups] : a.nrows, a.M, TM > 128 ? kTallChunkNs : kMidChunkNs);
        if (a.splits_out && blockIdx.x == 0 && threadIdx.x == 0) *a.splits_out = splits;
    }
    const int nx = nxm * splits;
    const int work = ntiles * nx;
    const int xcd = blockIdx.x % a.xcds, slot = blockIdx.x / a.xcds;
    const int per_xcd = gridDim.x / a.xcds;
    const int part = (work + a.xcds - 1) / a.xcds;
    const int wbeg = xcd * part, wend = min(work, wbeg + part);

    // a workgroup's items only increase, so its segment search resumes where
    // the previous item's ended
    int es = 0;
    auto item_at = [&](int wid) __attribute__((always_inline)) {
        Item it;
        int tile = wid / nx, xt = wid % nx;
        if (a.offsets) {
            // an expert's items (the same range of wid as in tile-major
            // order) go weight tile by weight tile, its token tiles adjacent:
            // the workgroups that read one weight tile run in the same round,
            // even where the expert straddles a round of the XCD's slots
            while (tstart[es + 1] <= tile) ++es;
            const int nt = tstart[es + 1] - tstart[es];
            const int local = wid - tstart[es] * nx;
            xt = local / nt;
            tile = tstart[es] + local % nt;
            it.e = es;
            it.r0 = soff[es] + (tile - tstart[es]) * TM;
            it.n = min(TM, soff[es + 1] - it.r0);
        } else {
            it.e = 0;
            it.r0 = tile * TM;
            it.n = min(TM, a.nrows - it.r0);
        }
        it.sp = 0;
        if constexpr (!GATED && !ROWS) {
            it.sp = xt / nxm;
            xt -= it.sp * nxm;
        }
        it.m0 = xt * kOut;
        // uniform: keep the item in scalar registers
        it.e = __builtin_amdgcn_readfirstlane(it.e);
        it.r0 = __builtin_amdgcn_readfirstlane(it.r0);
        it.n = __builtin_amdgcn_readfirstlane(it.n);
        it.m0 = __builtin_amdgcn_readfirstlane(it.m0);
        it.sp = __builtin_amdgcn_readfirstlane(it.sp);
        return it;
    };

    int wid = wbeg + slot;
    if (wid >= wend) {                        // uniform over the workgroup
        if constexpr (kFuse) {
            if (fused) publish_segments<NC>(a.seg, a.groups, cols, soff);
        }
        return;
    }
    auto source_rows = [&](const Item& it, int (&srow)[C::kBT]) __attribute__((always_inline)) {
        if constexpr (kFuse) {
            if (fused) {
#pragma unroll
                for (int j = 0; j < C::kBT; ++j) {
                    const int r = kRPB * (static_cast<int>(threadIdx.x) / kWave + C::kWaves * j) + lane_id() / kVPR;
                    srow[j] = nth_token<NC>(cols + it.e * NC, it.r0 - soff[it.e] + (r < it.n ? r : 0));
                }
                return;
            }
        }
        token_rows<C>(a, it, srow);
    };

    const int lane = lane_id(), wave = threadIdx.x / kWave;
    const int l32 = lane & 31, lh = lane >> 5;
    const int wm = wave / C::WW, wn = wave % C::WW;   // token group, weight group
    const int brow = 32 * TF * wm;            // this wave's first token row of the tile
    // first LDS weight row of fragment i: the gated tile's second half of
    // fragments are the W3 rows of the first half's features
    auto arow = [&](int i) __attribute__((always_inline)) {
        return GATED ? (i < WF / 2 ? 0 : NW / 2) + 16 * WF * wn + 32 * (i % (WF / 2)) : 32 * WF * wn + 32 * i;
    };
    const int nch = a.K / splits / kBK;       // at least kP (the launcher's condition)
    const int ks = a.K / splits;

    // Ring of STAGES stages, loads issued kP chunks ahead.  One step: wait
    // for this wave's loads of chunk c (later chunks' loads may stay in
    // flight), barrier (every wave's loads of chunk c have landed and every
    // wave is done with chunk c - 1's stage), refill that stage with chunk
    // c + kP, compute chunk c.  The ring runs on across items: an item's last
    // steps issue the next item's first chunks, and the next item's source
    // rows are loaded an item ahead, so neither the index loads nor the
    // refill wait behind the item's output stores.
    Item cur = item_at(wid);
    int srow[C::kBT];
    source_rows(cur, srow);
    ItemLoads<C> ld = item_loads<C, GATED, PACKED>(a, cur, cur.sp * ks, srow);
#pragma unroll
    for (int c = 0; c < C::kP; ++c)
        if (c < nch) {
            issue_chunk<C, PACKED>(ld, ring + c * C::kStage, c);
        }
    int sc = 0;                               // stage of the chunk computed next
    // output stores of the previous item, which may still be in flight when
    // this item's first chunks are awaited
    int stored = 0;

    for (;;) {
        const int nwid = wid + per_xcd;
        const bool more = nwid < wend;        // uniform
        Item nxt = cur;
        if (more) {
            nxt = item_at(nwid);
            source_rows(nxt, srow);
        }
        // this wave's token group holds rows of the expert
        const bool active = brow < cur.n;
        f32x16 acc[WF][TF];                   // [weight fragment][token fragment]
#pragma unroll
        for (int i = 0; i < WF; ++i)
#pragma unroll
            for (int j = 0; j < TF; ++j) acc[i][j] = f32x16{};

        // one step of the ring; L/ci: the loads to issue after the barrier
        // (ci < 0: none)
        auto step = [&](int c, const ItemLoads<C>& L, int ci) __attribute__((always_inline)) {
            // chunks issued after c: the item's own, then the next item's.
            // The first kP chunks of an item were issued before the previous
            // item's output stores, which need not have completed.
            wait_chunks<C>(more ? C::kP - 1 : min(C::kP - 1, nch - 1 - c), c < C::kP ? stored : 0);
            lds_barrier();
            const int si = sc == 0 ? C::STAGES - 1 : sc - 1;
            if (ci >= 0) issue_chunk<C, PACKED>(L, ring + si * C::kStage, ci);
            const uint8_t* st = ring + sc * C::kStage;
            sc = sc + 1 == C::STAGES ? 0 : sc + 1;
            if (!active) return;
#pragma unroll
            for (int k = 0; k < kBK / 16; ++k) {
                const int v = 2 * k + lh;
                bf16x8 B[TF], A[WF];
#pragma unroll
                for (int j = 0; j < TF; ++j)
                    B[j] = *reinterpret_cast<const bf16x8*>(st + wswz(brow + 32 * j + l32, v));
#pragma unroll
                for (int i = 0; i < WF; ++i)
                    A[i] = *reinterpret_cast<const bf16x8*>(st + C::kRegion + weight_at<PACKED>(arow(i) + l32, v));
#pragma unroll
                for (int j = 0; j < TF; ++j)
#pragma unroll
                    for (int i = 0; i < WF; ++i)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[i], B[j], acc[i][j], 0, 0, 0);
            }
        };
        // steps that refill from this item, then (its loads all issued) the
        // last kP steps, which start the next item
        for (int c = 0; c + C::kP < nch; ++c) step(c, ld, c + C::kP);
        if (more) ld = item_loads<C, GATED, PACKED>(a, nxt, nxt.sp * ks, srow);
        for (int c = max(0, nch - C::kP); c < nch; ++c) step(c, ld, more ? c + C::kP - nch : -1);

        // A lane holds weight rows 8 (q / 4) + 4 lh + q % 4 of each 32-row
        // fragment, for token row brow + 32 j + l32: its pieces of an output
        // row are 8 or 16 bytes.  The wave turns a fragment's rows around
        // through its share of the stage computed last (free after a
        // barrier: the next step refills it after one of its own), so that
        // adjacent lanes store adjacent 16-byte pieces, whole 128-byte lines
        // of a row where it has them (64 bytes in the gated tile).  Slots are
        // XORed with the row as in the ring.
        lds_barrier();
        static_assert(C::kStage / C::kWaves >= 4096, "a fragment's rows fit a wave's share of a stage");
        uint8_t* const tb =
            ring + (sc == 0 ? C::STAGES - 1 : sc - 1) * C::kStage + wave * (C::kStage / C::kWaves);
        stored = 0;
#pragma unroll
        for (int j = 0; j < TF; ++j) {
            const int nv = min(32, cur.n - brow - 32 * j);    // rows of the fragment (uniform)
            if (nv <= 0) break;
            const size_t row0 = static_cast<size_t>(cur.r0 + brow + 32 * j);
            if constexpr (GATED) {
                static_assert(WF == 2, "32 features per wave");
                // 64-byte rows
                auto at = [&](int r, int v) { return r * 64 + ((v ^ ((r >> 1) & 3)) << 4); };
#pragma unroll
                for (int qb = 0; qb < 4; ++qb) {
                    float hv[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) hv[q] = silu_rcp(acc[0][j][4 * qb + q]) * acc[1][j][4 * qb + q];
                    *reinterpret_cast<uint2*>(tb + at(l32, qb) + 8 * lh) =
                        uint2{pack_bf16x2(hv[0], hv[1]), pack_bf16x2(hv[2], hv[3])};
                }
                wave_lds_sync();
                uint16_t* const op = static_cast<uint16_t*>(a.out) + cur.m0 + 32 * wn;
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    if (16 * k >= nv) break;
                    const int r = 16 * k + lane / 4, v = lane % 4;
                    const u32x4 d = *reinterpret_cast<const u32x4*>(tb + at(r, v));
                    if (r < nv) *reinterpret_cast<u32x4*>(op + (row0 + r) * a.M + 8 * v) = d;
                    ++stored;
                }
                wave_lds_sync();
            } else {
                // 128-byte rows: 64 bf16 features, or 32 fp32 ones at a time
                auto at = [&](int r, int v) { return r * 128 + ((v ^ (r & 7)) << 4); };
                auto rows_out = [&](uint8_t* op, size_t pitch) __attribute__((always_inline)) {
                    wave_lds_sync();
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        if (8 * k >= nv) break;
                        const int r = 8 * k + lane / 8, v = lane % 8;
                        const u32x4 d = *reinterpret_cast<const u32x4*>(tb + at(r, v));
                        if (r < nv) *reinterpret_cast<u32x4*>(op + (row0 + r) * pitch + 16 * v) = d;
                        ++stored;
                    }
                    wave_lds_sync();
                };
                if constexpr (ROWS) {
                    static_assert(WF == 2, "64 features per wave");
                    float ss = 0.f;
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int qb = 0; qb < 4; ++qb) {
                            *reinterpret_cast<uint2*>(tb + at(l32, 4 * i + qb) + 8 * lh) =
                                uint2{pack_bf16x2(acc[i][j][4 * qb + 0], acc[i][j][4 * qb + 1]),
                                      pack_bf16x2(acc[i][j][4 * qb + 2], acc[i][j][4 * qb + 3])};
#pragma unroll
                            for (int q = 0; q < 4; ++q) ss = fmaf(acc[i][j][4 * qb + q], acc[i][j][4 * qb + q], ss);
                        }
                    rows_out(reinterpret_cast<uint8_t*>(static_cast<uint16_t*>(a.out) + cur.m0 + 64 * wn),
                             static_cast<size_t>(a.M) * 2);
                    // lanes l and l + 32 each hold half of the row's 64
                    // features: slot (m0 + 64 wn) / 32 + lh of the row
                    if (l32 < nv) a.nrm2[(row0 + l32) * (a.M / 32) + (cur.m0 >> 5) + 2 * wn + lh] = ss;
                    ++stored;
                } else {
#pragma unroll
                    for (int i = 0; i < WF; ++i) {
                        const int f = cur.m0 + 32 * (WF * wn + i);
                        if (NW <= 128 && f >= a.M) break;     // a last tile past M (M a multiple of 64)
#pragma unroll
                        for (int qb = 0; qb < 4; ++qb)
                            *reinterpret_cast<f32x4*>(tb + at(l32, 2 * qb + lh)) =
                                f32x4{acc[i][j][4 * qb + 0], acc[i][j][4 * qb + 1], acc[i][j][4 * qb + 2],
                                      acc[i][j][4 * qb + 3]};
                        rows_out(reinterpret_cast<uint8_t*>(static_cast<float*>(a.out) + cur.sp * a.split_stride + f),
                                 static_cast<size_t>(a.M) * 4);
                    }
                }
            }
        }
        if (!more) break;
        cur = nxt;
        wid = nwid;
    }
    if constexpr (kFuse) {
        if (fused) publish_segments<NC>(a.seg, a.groups, cols, soff);
    }
}

}  // namespace

bool wide_fits(bool gated, int M, int K) {
    return M % (gated ? Wide::NW / 2 : Wide::NW) == 0 && K % 128 == 0;
}

bool mid_fits(int M, int K) { return M % 64 == 0 && K % kBK == 0 && K >= kBK * Mid::kP; }

namespace {

// The part's geometry, asked once on the device current at the first call
// (every device a process uses is assumed to be the same part): its CUs,
// the XCDs the workgroups are dealt over, and how many workgroups of a
// kernel it keeps resident.
struct Geometry {
    int cus, xcds;
};

const Geometry& geometry() {
    static const Geometry g = [] {
        int dev = 0, cus = 0, xccs = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
            cus = 256;
        if (hipDeviceGetAttribute(&xccs, hipDeviceAttributeNumberOfXccs, dev) != hipSuccess || xccs < 1 ||
            xccs > cus)
            xccs = 1;
        return Geometry{cus, xccs};
    }();
    return g;
}

template <class C, bool GATED, bool PACKED, bool ROWS>
hipError_t launch_tile(const WideArgs& a, int64_t work, hipStream_t s) {
    static const int64_t resident = [] {
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, wide_kernel<GATED, C, PACKED, ROWS>, C::kThreads,
                                                         0) != hipSuccess ||
            per_cu < 1)
            per_cu = 1;
        return static_cast<int64_t>(geometry().cus) * per_cu;
    }();
    // persistent: the workgroups the part keeps resident (or one per item),
    // a multiple of the XCD count
    int64_t blocks = std::min<int64_t>(work, resident);
    blocks = std::max<int64_t>(a.xcds, (blocks + a.xcds - 1) / a.xcds * a.xcds);
    wide_kernel<GATED, C, PACKED, ROWS><<<static_cast<int>(blocks), C::kThreads, 0, s>>>(a);
    return hipGetLastError();
}

// Most token tiles the rows can take: every group may end in a partial tile.
int64_t most_tiles(const int32_t* offsets, int64_t rows_cap, int groups, int nrows, int tm) {
    return offsets ? std::min<int64_t>(rows_cap, (rows_cap + tm - 1) / tm + groups) : (nrows + tm - 1) / tm;
}

}  // namespace

hipError_t launch_wide(bool gated, const uint16_t* wa, const uint16_t* wb, const uint16_t* src,
                       const int32_t* gather, const int32_t* offsets, int groups, int nrows, int M, int K,
                       void* out, int64_t rows_cap, bool packed, float* nrm2, hipStream_t s) {
    if (nrm2 && gated) return hipErrorInvalidValue;
    WideArgs a{wa, wb, src, gather, offsets, groups, nrows, M, K, out, nrm2, geometry().xcds, 1, 0, nullptr, {}};
    const int64_t work =
        most_tiles(offsets, rows_cap, groups, nrows, Wide::TM) * (M / (gated ? Wide::NW / 2 : Wide::NW));
    if (gated) return packed ? launch_tile<Wide, true, true, false>(a, work, s) : launch_tile<Wide, true, false, false>(a, work, s);
    if (nrm2) return packed ? launch_tile<Wide, false, true, true>(a, work, s) : launch_tile<Wide, false, false, true>(a, work, s);
    return packed ? launch_tile<Wide, false, true, false>(a, work, s) : launch_tile<Wide, false, false, false>(a, work, s);
}

namespace {

template <class C>
hipError_t launch_mid_t(bool gated, WideArgs& a, int64_t rows_cap, bool packed, hipStream_t s) {
    const int out_w = gated ? C::NW / 2 : C::NW;
    const int64_t work =
        most_tiles(a.offsets, rows_cap, a.groups, a.nrows, C::TM) * ((a.M + out_w - 1) / out_w) * a.max_splits;
    if (gated) return packed ? launch_tile<C, true, true, false>(a, work, s) : launch_tile<C, true, false, false>(a, work, s);
    return packed ? launch_tile<C, false, true, false>(a, work, s) : launch_tile<C, false, false, false>(a, work, s);
}

}  // namespace

hipError_t launch_mid(bool gated, bool tall, const uint16_t* wa, const uint16_t* wb, const uint16_t* src,
                      const int32_t* gather, const int32_t* offsets, int groups, int nrows, int M, int K,
                      void* out, int64_t rows_cap, bool packed, int max_splits, int64_t split_stride,
                      int32_t* splits_out, const Segments& seg, hipStream_t s) {
    if (seg.mask && !gated) return hipErrorInvalidValue;
    WideArgs a{wa, wb, src, gather, offsets, groups, nrows, M, K, out, nullptr, geometry().xcds,
               max_splits, split_stride, splits_out, seg};
    return tall ? launch_mid_t<Tall>(gated, a, rows_cap, packed, s) : launch_mid_t<Mid>(gated, a, rows_cap, packed, s);
}

}  // namespace eat
