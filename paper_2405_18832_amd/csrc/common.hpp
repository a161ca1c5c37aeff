// Shared declarations of the MoE FFN library for gfx950: storage helpers, the
// workspace layout and the internal launch functions that the C ABI composes.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "moe.h"

namespace moe {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kWave = 64;

// ---- bf16 storage <-> fp32 ------------------------------------------------
__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
    return __uint_as_float(static_cast<uint32_t>(b) << 16);
}
// round to nearest, ties to even; NaN stays NaN: the hardware conversion (v_cvt_pk_bf16_f32), two values
// per instruction
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_t;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2_t;
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    const f32x2_t v = {lo, hi};
    const bf16x2_t r = __builtin_convertvector(v, bf16x2_t);
    return __builtin_bit_cast(uint32_t, r);
}
__device__ __forceinline__ uint16_t f32_to_bf16(float f) { return static_cast<uint16_t>(pack_bf16x2(f, 0.f) & 0xffffu); }

template <typename ST> struct Storage;
template <> struct Storage<float> {
    static __device__ __forceinline__ float load(const float* p) { return *p; }
    static __device__ __forceinline__ void store(float* p, float v) { *p = v; }
};
template <> struct Storage<uint16_t> {
    static __device__ __forceinline__ float load(const uint16_t* p) { return bf16_to_f32(*p); }
    static __device__ __forceinline__ void store(uint16_t* p, float v) { *p = f32_to_bf16(v); }
};

// ---- expert tiles: the unit the FFN kernels schedule ------------------------
// A tile is up to `tile_rows` consecutive rows of one expert's segment of x_perm.
struct Tile {
    int32_t expert;
    int32_t row0;    // first row in x_perm / h / y_perm
    int32_t rows;    // 1 .. tile_rows
    int32_t pad;
};

// Tiles of experts with at least kBigMinRows rows go to the LDS-tiled MFMA kernel (tiles of
// kBigTileRows rows); smaller experts are weight-streaming work.
constexpr int kBigTileRows = 256;
constexpr int kBigMinRows = 128;
// The same experts are listed in tiles of kHalfTileRows rows too, for products whose large tiles are too few to
// occupy the chip (tiled_product_units in tile_schedule.hpp).
constexpr int kHalfTileRows = 128;
constexpr int kHalfCount = 4;           // int of the `ntiles` array that holds their number
// Experts between one streaming tile and kBigMinRows rows would have their weights streamed once per
// streaming tile; as one mostly empty tile of tiled units they cost about what a single pass over their
// weights costs -- where there are rounds of tiled units anyway, which hide the additional units:
//  - with whole rounds of units, i.e. when the tiles of the experts with kBigMinRows rows already number `join_tiles`
//    (the host's figure: one full round of units in the narrower product);
//  - in half-sized units, as long as all of them, `half_tiles_joined` tiles of them and the experts that are large in any
//    case, are at most one round in the wider product (`join_half_tiles`): then they occupy CUs that would be idle.
//    (Experts of 327, 112, 85, 71 and 12 times at most 45 rows, 1024 x 4096: streaming 41.8 + 39.8 -> 23.8 + 25.5 us, tiled
//    15.2 + 14.2 -> 19.6 + 18.6 us.)
// Else an under-filled round would only get longer.
constexpr int kJoinMinRows = 65;
inline __host__ __device__ int tiled_min_rows(int big_tiles_at_min, int join_tiles, int half_tiles_joined, int join_half_tiles) {
    if (join_tiles > 0 && big_tiles_at_min >= join_tiles) return kJoinMinRows;
    if (big_tiles_at_min > 0 && half_tiles_joined <= join_half_tiles) return kJoinMinRows;
    return kBigMinRows;
}
// The units of the last, partly filled round of tiled units are cut along K; the parts are handed out through a counter and leave
// fp32 partial tiles (kBigTileRows x 256) in the workspace.
constexpr int kSplitSlots = 256;        // partial tiles in the workspace
constexpr int kSplitCounter = 2;        // ints [2] and [3] of the `ntiles` array: the part counters of the
                                        // first and of the second product
// Counters of a layer that may have large experts, behind the first 64 ints of the `ntiles` array, zero when its products start:
// per product, the streaming units taken from each of 8 runs (a 128-byte line each: every XCD counts in its own), and how many
// of the two sums that meet at a node have got there (join_parts in ffn_tile.hip)
constexpr int kTakenStride = 32, kTakenAt = 64, kJoinedAt = kTakenAt + 2 * 8 * kTakenStride;
constexpr int kListCounters = 2 * 8 * kTakenStride + 2 * kSplitSlots;
constexpr int kListThreads = 1024;      // threads of the block that makes the lists
static_assert(kListCounters == kListThreads, "a thread each clears them");

// trailing activation of the first linear layer (Section 3.4): 0 = ReLU, 1 = GeLU in its defining form
// z * Phi(z) = 0.5 z (1 + erf(z / sqrt 2))
#ifdef __HIPCC__
__device__ __forceinline__ float gelu_erf(float z) { return 0.5f * z * (1.f + erff(z * 0.70710678118654752f)); }

__device__ __forceinline__ float activate(float z, int act) { return act == MOE_ACT_GELU ? gelu_erf(z) : fmaxf(z, 0.f); }

// GeLU where the result is rounded to bf16, without branches and in half the instructions of erff:
//   Phi(-|z|) = erfc(a) / 2 = exp(-a^2) t Q(t),  a = |z| / sqrt 2,  t = 1 / (1 + a / 2)
// (the form of Numerical Recipes' erfcc; Q is a Chebyshev fit of degree 8 over 0 <= a <= 10, relative error 4e-8), and
// Phi(z) = 1 - Phi(-z).  Against 64 bits over |z| <= 8, in fp32: largest error 3.8e-7, relative error for |z| < 4 at most
// 8.4e-7 (gelu_erf: 4.5e-7 and, because 1 + erf cancels for negative z, 4.6e-4).
__device__ __forceinline__ float gelu_exp(float z) {
    const float t = __builtin_amdgcn_rcpf(fmaf(fabsf(z), 0.35355339059327378f, 1.f));
    float q = -2.953637950e-02f;
    q = fmaf(q, t, 1.422964782e-01f);
    q = fmaf(q, t, -2.436179519e-01f);
    q = fmaf(q, t, 1.390533745e-01f);
    q = fmaf(q, t, -1.332583465e-02f);
    q = fmaf(q, t, 1.013486385e-01f);
    q = fmaf(q, t, 1.215506494e-01f);
    q = fmaf(q, t, 1.411878169e-01f);
    q = fmaf(q, t, 1.410432011e-01f);
    const float tail = q * t * __builtin_amdgcn_exp2f(z * z * -0.72134752044448170f);
    return z * (z < 0.f ? tail : 1.f - tail);
}

// Four values at once, the activation a compile-time constant: the MFMA kernels are instantiated per
// activation (as a run-time choice in their epilogues it cost the ReLU layers 5-10 % of the kernel).
template <int ACT>
__device__ __forceinline__ f32x4 activate4(f32x4 v) {
    if (ACT == MOE_ACT_GELU) return f32x4{gelu_exp(v[0]), gelu_exp(v[1]), gelu_exp(v[2]), gelu_exp(v[3])};
    return f32x4{fmaxf(v[0], 0.f), fmaxf(v[1], 0.f), fmaxf(v[2], 0.f), fmaxf(v[3], 0.f)};
}

// template argument FIRST of the product kernels: 0 = second product, else first product with ...
constexpr int kFirstRelu = 1;
constexpr int kFirstGelu = 2;
#endif

// Layout of the bf16 row operands that the products read 32 k at a time (the intermediate
// h = act(x . W1^T) and the gathered token rows): blocks of kRowBlock rows, and inside a block k-step-major,
// [rows / 256][K / 32][256][32].  The 32 values of consecutive rows are 64 bytes apart, so a 16-row MFMA
// operand fragment is one contiguous KiB (row-major, each row would contribute half a cache line), a row
// tile of one k-step is at most two contiguous runs, and consecutive k-steps of a row are 16 KiB apart: a
// block that walks along K reads one linear stream.  (With the k-step outermost over all A rows, [K / 32][A][32],
// consecutive steps of a 32 k-row layer were 2 MiB apart and the global-to-LDS copies of the tiled units ran
// at two thirds of the rate they reach on a linear stream.)  Element (row, n) of a tensor with `ksteps` = K / 32:
constexpr int kRowBlock = 256;
#ifdef __HIPCC__
__device__ __forceinline__ size_t h_index(int row, int n, int ksteps) {
    return ((static_cast<size_t>(row >> 8) * ksteps + (n >> 5)) * kRowBlock + (row & (kRowBlock - 1))) * 32 + (n & 31);
}
constexpr int kStepStride = kRowBlock * 32;     // elements between consecutive k-steps of a row
#endif

#ifdef __HIPCC__
typedef const void __attribute__((address_space(1))) * gptr_t;
typedef void __attribute__((address_space(3))) * lptr_t;

// byte address inside LDS of a pointer to __shared__ memory
__device__ __forceinline__ uint32_t lds_address(const void* p) {
    return static_cast<uint32_t>(reinterpret_cast<size_t>((lptr_t)(p)));
}

// 16 bytes per lane from global memory straight into LDS at `lds_base + 16 * lane` (no registers);
// `lds_base` (an LDS byte address) is the same for the whole wavefront and goes into M0.  Written as inline assembly: after the
// compiler's own builtin for this instruction it makes every later wait for an LDS read a wait for all
// outstanding LDS reads (as long as a copy is in flight, which here is always), and the loops that
// use it depend on waiting only for the oldest ones.  The copies are counted by vmcnt; the code waits for
// them explicitly, and orders them against LDS reads with barriers.  M0 is not live across statements
// in compiled code for this target (the compiler sets it right before each use of its own); it cannot be named
// in the clobber list, the compiler rejects reserved registers there ("may not be preserved across the asm
// statement"), so that property is what the statement relies on.
__device__ __forceinline__ void copy16_to_lds(const void* src, uint32_t lds_base) {
    const uint32_t dst = __builtin_amdgcn_readfirstlane(lds_base);
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(src), "s"(dst) : "memory");
}

#endif

#ifdef __HIPCC__
// fp32 matrix products read 16 k of a row per step, lane group g = lane / 16 the four at k0 + 4g (ffn_f32.hip says how
// the MFMAs use them).
// 4 consecutive k of a row; VEC: the widest load the row pitch and the base addresses allow
template <int VEC>
__device__ __forceinline__ f32x4 load_k4(const float* __restrict__ p) {
    if constexpr (VEC == 4) return *reinterpret_cast<const f32x4*>(p);
    if constexpr (VEC == 2) {
        const float2 a = *reinterpret_cast<const float2*>(p), b = *reinterpret_cast<const float2*>(p + 2);
        return f32x4{a.x, a.y, b.x, b.y};
    }
    return f32x4{p[0], p[1], p[2], p[3]};
}
// the same at the end of a row: only `left` of the four exist (none if left <= 0), the others are zero
__device__ __forceinline__ f32x4 load_k4_tail(const float* __restrict__ p, int left) {
    f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (i < left) v[i] = p[i];
    return v;
}
#endif

struct TileLists {
    Tile* small_tiles;     // capacity A / small_rows + E
    Tile* big_tiles;       // capacity A / kBigTileRows + E (unused when big_min == 0)
    Tile* half_tiles;      // the same experts in tiles of kHalfTileRows rows, capacity A / kHalfTileRows + E
    int32_t* ntiles;       // [0] small count, [1] big count, [2], [3] part counters of the tiled products, [4] half count, [8] and
                           // [20]: the TileSchedule of the first and of the second product (if big_min > 0)
    float* partials;       // kSplitSlots partial tiles (nullptr when big_min == 0)
    int small_rows;        // rows per small tile
    int big_min;           // experts with >= big_min rows are "big"; 0 = none
    int join_tiles;        // tiles of big experts from which the mid-sized experts join them (tiled_min_rows); 0 = never
    int join_half_tiles;   // half-sized tiles, with the mid-sized experts', up to which they do
    int d_model, d_ff, cus;       // what the schedules depend on besides the tiles
    bool gelu;
};

#ifdef __HIPCC__
// Places one chunk of consecutive flat assignment ids (counting sort, last step): called by one whole
// wavefront.  `next` (LDS, E ints, private to the wavefront) holds each expert's first free slot for this
// chunk and is advanced.  The wavefront walks its chunk 64 flat ids at a time; lanes that hold the same
// expert find each other with one ballot per bit of the expert id, take consecutive slots in lane order,
// and the last of them advances the expert's slot.  Writes (each may be NULL) perm[pos] = a,
// inv_perm[a] = pos, tokmap[pos] = a / k.
// `first`: the chunk's first 256 experts, fetched by the caller (chunk_experts) ahead of what it does before.
constexpr int kChunkAhead = 4;
struct ChunkExperts { int e[kChunkAhead]; };
__device__ __forceinline__ ChunkExperts chunk_experts(const int32_t* __restrict__ idx, int A, int chunk, int c) {
    const int lane = threadIdx.x & 63;
    ChunkExperts r;
#pragma unroll
    for (int i = 0; i < kChunkAhead; ++i) {
        const int o = i * 64 + lane;
        r.e[i] = (o < chunk && c * chunk + o < A) ? idx[c * chunk + o] : 0;
    }
    return r;
}
__device__ __forceinline__ void place_chunk(const int32_t* __restrict__ idx, const ChunkExperts& first, int32_t* next,
                                            int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm,
                                            int32_t* __restrict__ tokmap, int A, int E, int k, int ebits, int chunk,
                                            int c) {
    const int lane = threadIdx.x & 63;
    const int base = c * chunk;
    for (int i0 = 0; i0 < chunk; i0 += 64) {
        const int a = base + i0 + lane;
        const bool live = (i0 + lane < chunk) && a < A;
        int ex = 0;
#pragma unroll
        for (int i = 0; i < kChunkAhead; ++i)
            if (i0 == i * 64) ex = first.e[i];
        if (i0 >= kChunkAhead * 64 && live) ex = idx[a];
        const int e = live ? min(max(ex, 0), E - 1) : 0;       // clamped: a bad index must not fault
        uint64_t same = __ballot(live);
        for (int b = 0; b < ebits; ++b) {
            const uint64_t has = __ballot(live && ((e >> b) & 1));
            same &= ((e >> b) & 1) ? has : ~has;
        }
        const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
        const int rank = __popcll(same & below);
        int pos = 0;
        if (live) pos = next[e] + rank;
        __builtin_amdgcn_wave_barrier();
        const bool last = live && ((same >> lane) >> 1) == 0;   // no higher lane with this expert
        if (last) next[e] = pos + 1;
        __builtin_amdgcn_wave_barrier();
        if (live && pos >= 0 && pos < A) {   // offsets that do not belong to idx must not fault
            if (perm) perm[pos] = a;
            if (inv_perm) inv_perm[a] = pos;
            if (tokmap) tokmap[pos] = a / k;
        }
    }
}

// Inclusive prefix sum over the lanes of a wavefront, all of them active: inside the rows of 16, then from row to row (DPP moves,
// no LDS traffic).
__device__ __forceinline__ int wave_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);        // from 1, 2, 4 and 8 lanes below in the row
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);        // the last lane of rows 0 and 2 to rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);        // lane 31 to rows 2 and 3
    return v;
}

// Inclusive prefix sums of N values at once over the threads of a block's first `nw` wavefronts (thread e contributes v[i]) and their
// totals.  Called by all threads of the block; the other wavefronts only meet the barrier and get nothing: a block of 16 wavefronts
// that all went through this for the one or two that hold experts was bound by issuing it.  `tmp`: 16 * N ints of LDS, for
// this call alone.
template <int N>
__device__ __forceinline__ void block_scan(const int (&v)[N], int (&incl)[N], int (&total)[N], int32_t* tmp, int nw) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < N; ++i) incl[i] = total[i] = 0;
    if (wave < nw) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            incl[i] = wave_scan(v[i]);
            if (lane == 63) tmp[i * 16 + wave] = incl[i];
        }
    }
    __syncthreads();
    if (wave < nw) {
        for (int w = 0; w < nw; ++w) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int t = tmp[i * 16 + w];
                if (w < wave) incl[i] += t;
                total[i] += t;
            }
        }
    }
}
constexpr int kScanInts = 96;           // LDS of two scans of three values

// what an expert of m rows contributes to the two sums that tiled_min_rows is asked with
inline __host__ __device__ int big_tiles_at_min(int m, const TileLists& tl) {
    return tl.big_min > 0 && m >= tl.big_min ? (m + kBigTileRows - 1) / kBigTileRows : 0;
}
inline __host__ __device__ int half_tiles_joined(int m, const TileLists& tl) {
    return tl.big_min > 0 && m >= kJoinMinRows ? (m + kHalfTileRows - 1) / kHalfTileRows : 0;
}

// The tiles of one expert (row0, m rows), `rows` rows each, to out[0 ...].  Called by whole wavefronts, a lane per
// expert.  An expert with more than two tiles is written by all lanes of its wavefront (thousands of rows make dozens
// of tiles, which one lane alone would store one after the other).
__device__ __forceinline__ void write_tiles(Tile* __restrict__ out, int e, int row0, int m, int rows, int nt) {
    for (int i = 0; i < 2; ++i)
        if (nt <= 2 && i < nt) out[i] = Tile{e, row0 + i * rows, min(rows, m - i * rows), 0};
    uint64_t many = __ballot(nt > 2);
    while (many != 0) {                                    // wave-uniform
        const int src = __builtin_ctzll(many);
        many &= many - 1;
        const int r0 = __builtin_amdgcn_readlane(row0, src), mm = __builtin_amdgcn_readlane(m, src);
        const int n = __builtin_amdgcn_readlane(nt, src), ee = __builtin_amdgcn_readlane(e, src);
        const uint64_t at = reinterpret_cast<uint64_t>(out);
        const uint64_t lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(at), src));
        const uint64_t hi = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(at >> 32), src));
        Tile* o = reinterpret_cast<Tile*>(lo | hi << 32);
        for (int i = threadIdx.x & 63; i < n; i += 64) o[i] = Tile{ee, r0 + i * rows, min(rows, mm - i * rows), 0};
    }
}
#endif

// ---- workspace ----------------------------------------------------------------
struct WsLayout {
    size_t hist;       // int32 [ceil(T/16), E]  chunk histograms / slot bases of the counting sort
    size_t ntiles;     // int32 [64 + kListCounters, or 64 without large experts]  ([0] = tiles of small experts, [1] = of large experts, [2], [3] counters)
    size_t tiles;      // Tile [A/16 + E + 1]   row tiles of the streaming units
    size_t tiles_big;  // Tile [A/256 + E + 1]  row tiles of the big and narrow units
    size_t tiles_half; // Tile [A/128 + E + 1]  the same rows in the half-sized tiles of that kernel (if an expert can have them)
    size_t h;          // dtype [A rounded up to kRowBlock, f]
    size_t idx;        // int32 [A]         -- the rest is used by moe_layer_forward only
    size_t gate;       // float [A]
    size_t counts;     // int32 [E]
    size_t offsets;    // int32 [E + 1]
    size_t perm;       // int32 [A]
    size_t inv_perm;   // int32 [A]
    size_t mask;       // uint8 [E]
    size_t tokmap;     // int32 [A]  token row of each permuted position
    size_t y_perm;     // float [A, d]
    size_t partials;   // float [kSplitSlots, 256, 256]  (only when an expert can reach kBigMinRows rows)
    size_t x_kmajor;   // bf16 [A rounded up to kRowBlock, d]  gathered token rows in the blocked layout (same condition)
    size_t gate_part;  // float [kGateSplit, T rounded up to 16, E]  partial gate logits (layers with route_is_split)
    size_t total;
};

// Layers with few tokens (decode steps) cut the gate product over many one-wavefront blocks and along the
// contraction into kGateSplit slices (partial logits in the workspace).  Measured: a gain up to 64 tokens
// (one block per 16 tokens leaves reading the gate weights to a few CUs), none at 2048 tokens.
constexpr int kGateSplit = 8;
#ifndef MOE_SPLIT_ROUTE_TOKENS
#define MOE_SPLIT_ROUTE_TOKENS 64
#endif
constexpr int kSplitRouteTokens = MOE_SPLIT_ROUTE_TOKENS;
inline bool route_is_split(const moe_shape& s) { return s.dtype == MOE_BF16 && s.T <= kSplitRouteTokens; }
constexpr int kPermChunk = 256;   // assignments per counting-sort chunk (one wavefront)

inline size_t elem_size(int32_t dtype) { return dtype == MOE_BF16 ? 2 : 4; }

inline WsLayout ws_layout(const moe_shape& s) {
    WsLayout L{};
    const size_t A = static_cast<size_t>(s.T) * s.k, E = s.E, es = elem_size(s.dtype);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t at = off;
        off += (bytes + 255) & ~static_cast<size_t>(255);
        return at;
    };
    L.hist = take(((static_cast<size_t>(s.T) + 15) / 16 + 1) * E * 4);
    const bool big = s.dtype == MOE_BF16 && s.T >= kBigMinRows;
    L.ntiles = take((64 + (big ? kListCounters : 0)) * 4);
    L.tiles = take((A / 16 + E + 1) * sizeof(Tile));
    L.tiles_big = take((A / 256 + E + 1) * sizeof(Tile));
    L.tiles_half = take(big ? (A / kHalfTileRows + E + 1) * sizeof(Tile) : 0);
    const size_t Ab = (A + kRowBlock - 1) / kRowBlock * kRowBlock;     // the blocked layouts hold whole row blocks
    L.h = take(Ab * s.d_ff * es);
    L.idx = take(A * 4);
    L.gate = take(A * 4);
    L.counts = take(E * 4);
    L.offsets = take((E + 1) * 4);
    L.perm = take(A * 4);
    L.inv_perm = take(A * 4);
    L.mask = take(E);
    L.tokmap = take(A * 4);
    L.y_perm = take(A * s.d_model * 4);
    L.partials = take(big ? static_cast<size_t>(kSplitSlots) * kBigTileRows * 256 * 4 : 0);
    L.x_kmajor = take(big ? Ab * s.d_model * es : 0);
    L.gate_part = take(route_is_split(s) ? static_cast<size_t>(kGateSplit) * ((s.T + 15) / 16 * 16) * E * 4 : 0);
    L.total = off;
    return L;
}

// ---- internal launchers (all asynchronous on `st`; return hipSuccess or the launch error)
hipError_t launch_route(const moe_shape& s, const void* x, const void* w_gate, const float* bias,
                        int32_t* idx, float* gate, float* margin, int32_t* counts,
                        int32_t* offsets, int32_t H, uint8_t* hot_mask, int32_t* hist_ws, float* gate_part_ws,
                        hipStream_t st);
int route_chunk_tokens(const moe_shape& s);
hipError_t launch_select_hot(int E, const int32_t* counts, double alpha, double bw_a, double bw_b, int32_t* H_out,
                             uint8_t* hot_mask, hipStream_t st);
hipError_t launch_route_fused(const moe_shape& s, const void* x, const void* w_gate, const float* bias,
                              int32_t* idx, float* gate, float* margin, int32_t* chunk_hist, float* gate_part_ws,
                              hipStream_t st);
// Top-1 layers without an expert mask: the second product writes the layer output itself.  Row p of the
// permuted order belongs to token tokmap[p] and to nobody else, so out[tokmap[p]] = gate[tokmap[p]] * y[p],
// rounded to the storage type, is the combine step's result for that token (same operations, same rounding) and the
// rows of y never go to memory.  out == nullptr: the product writes y as usual.
struct FoldOut {
    void* out;               // [T, N] of the storage type
    const int32_t* tokmap;   // [A]
    const float* gate;       // [T] (k = 1)
};

// what placing the assignments needs (the counting sort's last step)
struct PlaceArgs {
    const int32_t* idx;    // nullptr: do not place
    int32_t* perm;
    int32_t* inv_perm;
    int32_t* tokmap;
    int A, k, chunk;
};
hipError_t launch_route_finalize(const moe_shape& s, const void* x, const void* w_gate, const float* bias,
                                 int32_t* idx, float* gate, float* margin, int32_t* hist_ws, float* gate_part_ws,
                                 int32_t* counts, int32_t* offsets, int H, uint8_t* hot_mask, uint8_t* mask_copy,
                                 const uint8_t* mask_in, const TileLists* lists, const PlaceArgs* place, hipStream_t st);
hipError_t launch_place(int32_t* chunk_hist, int nchunks, int E, const int32_t* offsets, const PlaceArgs& place,
                        hipStream_t st);
TileLists ffn_tile_lists(const moe_shape& s, Tile* small_ws, Tile* big_ws, Tile* half_ws, int32_t* ntiles_ws, float* partials_ws);
int ffn_tile_rows(const moe_shape& s);
int tiled_join_tiles(const moe_shape& s);
hipError_t launch_expert_products(const moe_shape& s, const void* act, const int32_t* rowmap, bool act_kmajor,
                                  const void* w1, const void* w2, const float* b1, const float* b2, float* y_perm,
                                  void* h_ws, const TileLists& lists, const FoldOut& fold, hipStream_t st);
bool layer_gathers_kmajor(const moe_shape& s);
hipError_t launch_gather_kmajor(const moe_shape& s, const void* x, const int32_t* tokmap, void* xk, hipStream_t st);
hipError_t launch_tiled_product(bool first, int ksplit, const uint16_t* act, const int32_t* rowmap, const uint16_t* wpk,
                               void* outp, const TileLists& lists, int N, int K, bool act_kmajor, int activation,
                               const float* bias, const FoldOut& fold, int kinds, hipStream_t st);
constexpr int kTiledUnits = 1, kStreamUnits = 2;        // kinds of units that a launch of a product runs
int tile_product_grid();
hipError_t launch_f32_product(bool first, long rows, const float* act, const int32_t* rowmap, const float* w, float* outp,
                              const Tile* tiles, const int32_t* ntiles, long max_tiles, int N, int K, int activation,
                              const float* bias, const FoldOut& fold, hipStream_t st);
bool layer_sorts_in_first(const moe_shape& s);
hipError_t launch_f32_sorted_products(const moe_shape& s, const float* x, const int32_t* idx, const float* w1, const float* w2,
                                      const float* b1, const float* b2, int32_t* counts, int32_t* offsets, int32_t* perm,
                                      int32_t* inv_perm, int32_t* tokmap, const TileLists& lists, float* h, float* y_perm,
                                      const FoldOut& fold, hipStream_t st);
hipError_t launch_permute(const moe_shape& s, const void* x, const int32_t* idx,
                          const int32_t* offsets, int32_t* perm, int32_t* inv_perm, void* x_perm,
                          int32_t* hist_ws, hipStream_t st);
hipError_t launch_expert_ffn(const moe_shape& s, const void* x_perm, const void* w1, const void* w2,
                             const float* b1, const float* b2,
                             const int32_t* offsets, const uint8_t* mask, float* y_perm,
                             void* h_ws, Tile* tiles_ws, Tile* tiles_big_ws, Tile* tiles_half_ws, int32_t* ntiles_ws, float* partials_ws,
                             void* x_kmajor_ws, hipStream_t st);
hipError_t launch_combine(const moe_shape& s, const float* y_perm, const int32_t* inv_perm,
                          const int32_t* idx, const float* gate, const uint8_t* mask, void* out,
                          hipStream_t st);
hipError_t launch_gate_partial(const moe_shape& s, const void* x, const void* w_gate, float* part, hipStream_t st);
bool layer_is_few(const moe_shape& s);
hipError_t launch_few_products(const moe_shape& s, const void* x, const float* gate_bias, const float* gate_part, const void* w1,
                               const void* w2, const float* b1, const float* b2, int32_t* idx, float* gate, int32_t* counts,
                               int32_t* offsets, int32_t* perm, int32_t* inv_perm, int32_t* tokmap, void* h, void* out,
                               hipStream_t st);
hipError_t launch_pack(const moe_shape& s, int which, const void* src, void* dst, hipStream_t st);
hipError_t launch_mask_out(const uint8_t* mask_or_null, uint8_t* dst, int E, hipStream_t st);

void set_profile_events(const hipEvent_t* five_events_or_null);
hipError_t mark_profile_event(int i, hipStream_t st);     // records the caller's event i, if there is one

// number of compute units of the current device (cached)
int device_cu_count();

// ---- one-time set-up per device ---------------------------------------------------------------
// Raising a kernel's dynamic-LDS limit and asking for its occupancy are calls into the runtime that do not
// belong on a launch path (they cost time, and a first call made while a stream is being captured would
// land inside the capture).  ensure_ready() makes them all, for every kernel of the library, once per
// device and under a lock; every entry point that launches kernels calls it first.
constexpr int kMaxDevices = 64;
constexpr size_t kLdsPerCu = 160 * 1024;
hipError_t ensure_ready();                       // api.hip
int current_device_index();                      // api.hip: hipGetDevice clamped to [0, kMaxDevices)
hipError_t configure_ffn_kernels(int dev);       // ffn.hip
hipError_t configure_tile_kernels(int dev);      // ffn_tile.hip
hipError_t configure_f32_kernels();              // ffn_f32.hip
hipError_t configure_route_kernels(int dev);     // route.hip

}  // namespace moe
