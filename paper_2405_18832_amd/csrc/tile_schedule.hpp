// Schedule of the LDS-tiled units, (row tile, column tile) pairs of the large experts, made with the tile lists and read by the kernel
// that runs them (ffn_tile.hip).
//
// All units cost the same.  G blocks run U / G full rounds of whole units in a fixed, XCD-aware order.
// The R = U mod G units left over would keep R blocks busy for a whole round and the rest of the chip
// idle, so each of them is cut along K into `split` parts; blocks take parts from a counter as they
// become free, and the sums of a unit's parts meet in the workspace, in a tree over the part numbers (join_parts).
#pragma once
#include "common.hpp"

namespace moe {

constexpr int kMaxSplit = 8;        // parts per left-over unit, at most ...
#ifndef MOE_MIN_SPLIT_STEPS
#define MOE_MIN_SPLIT_STEPS 32
#endif
#ifndef MOE_MIN_SPLIT_STEPS_FINE
#define MOE_MIN_SPLIT_STEPS_FINE 24
#endif

// The shapes of a unit: rows x columns of its output, the groups of wavefronts that share its contraction inside the
// block (each adds up an equal run of its 32-k steps), and the fewest steps of a part.
struct BigUnits {
    static constexpr int kRows = kBigTileRows, kCols = 256, kGroups = 1, kMinSplitSteps = MOE_MIN_SPLIT_STEPS;
};
struct FineUnits {
    static constexpr int kRows = kHalfTileRows, kCols = 128, kGroups = 2, kMinSplitSteps = MOE_MIN_SPLIT_STEPS_FINE;
};
struct NarrowUnits {
    static constexpr int kRows = kBigTileRows, kCols = 128, kGroups = 1, kMinSplitSteps = MOE_MIN_SPLIT_STEPS;
};

// Which of them a product of `kblk` 32-k steps runs in.  Fine ones where they are at most one round: the big units would leave
// most of the chip idle, or be half empty (experts of up to 128 rows).  Narrow ones where these are at most one round (65 to 128
// full-width units: big units would run on that many of 256 CUs, or be cut along K and added up afterwards), unless the contraction
// is so long that the cut units win: a step takes about 0.5 us in a narrow unit and 0.7 in a big one.  Big units that can be cut in
// three win from about 100 steps on, those cut in two from about 190; and with few row tiles the narrow units of an XCD share too
// little of their rows: sooner.  Else big ones, but fine ones for the first product of a GeLU layer with less than half a round of
// big units, whose epilogue all CUs work on then instead of those that have a big unit; up to 85 big units these are ahead of the
// narrow ones too from about 60 steps on.
// us, what ran without narrow units -> narrow, the pass that adds up parts included, tiles of 256 rows: 96 units of 24 steps
// 39 -> 31 (188 rows 35 -> 28), 112 of 32 44 -> 37, 72 of 36 42 -> 32, 80 of 64 55 -> 46, 112 of 64 65 -> 52, 108 of 96 80 -> 68, 96 of 128
// 88 -> 81, 128 of 128 104 -> 90; not taken, with few row tiles and up to 85 units: 72 of 96 56.8 -> 62.7 (140 rows), 72 of 72
// 62 -> 64, 72 of 128 71 -> 75; nor 3 x 32 of 128 96 -> 103, 96 of 192 115 -> 117, 80 of 256 126 -> 143.
// GeLU first products: 96 of 24 44 -> 36, 128 of 64 75 -> 55, 112 of 128 107 -> 89; fine, not narrow: 72 of 63 0.88, 77 of 77 0.94,
// 69 of 92 0.80, 88 of 96 and 4 row tiles 0.94 of the time; fine, not big: 80 of 144 (130 rows) 73 and 79, 75 of 171 (196 rows) 82 and
// 95, 72 of 131 70 and 79 (full row tiles and long contractions are the other way: 112 of 256 184 and 157).
enum class UnitShape { kBig, kNarrow, kFine };
inline __host__ __device__ UnitShape tiled_product_units(long big_tiles, long half_tiles, int N, int kblk, int cus, bool gelu) {
    if (half_tiles * ((N + FineUnits::kCols - 1) / FineUnits::kCols) <= cus) return UnitShape::kFine;
    const long big_units = big_tiles * ((N + BigUnits::kCols - 1) / BigUnits::kCols);
    if (big_tiles * ((N + NarrowUnits::kCols - 1) / NarrowUnits::kCols) <= cus) {
        const bool cut_in_three = big_units * 3 <= cus;
        const int longest = cut_in_three ? (gelu ? 56 : big_tiles >= 9 ? 96 : 70) : (big_tiles >= 8 ? 128 : gelu ? 80 : 96);
        if (kblk <= longest) return UnitShape::kNarrow;
    }
    return gelu && big_units * 2 < cus ? UnitShape::kFine : UnitShape::kBig;
}

struct TileSchedule {
    UnitShape shape;
    int ntiles, ntn;    // row tiles, column tiles
    int rounds, R;      // full rounds of G units; units left over
    int split;          // parts per left-over unit (1: not cut, written directly)
    int GM, GN;         // patch of consecutive units: GM row tiles x GN column tiles
    int sums;           // narrow units: partial sums of the contraction that an output is added up from (run_units)
    int pad[3];
};
constexpr int kScheduleAt = 8, kScheduleInts = 12;     // in the `ntiles` array, one per product
static_assert(sizeof(TileSchedule) == kScheduleInts * 4, "as laid out in the array");

#ifdef __HIPCC__
template <typename Units>
__host__ __device__ __forceinline__ TileSchedule schedule_of(UnitShape shape, int ntiles, int N, int kblk, int G) {
    TileSchedule s;
    s.shape = shape;
    s.ntiles = ntiles;
    s.ntn = (N + Units::kCols - 1) / Units::kCols;
    const int U = ntiles * s.ntn;
    s.rounds = U / G;
    s.R = U - s.rounds * G;
    s.split = s.sums = 1;
    if (shape == UnitShape::kNarrow) {                     // as many as big units would have been cut into
        const int big = ntiles * ((N + BigUnits::kCols - 1) / BigUnits::kCols);
        s.sums = max(1, min(G / max(big, 1), min(kMaxSplit, kblk / BigUnits::kMinSplitSteps)));
    }
    if (s.R > 0 && shape != UnitShape::kNarrow) {          // narrow units are more than half a round: never cut
        constexpr int slots = kSplitSlots * (kBigTileRows * 256 / (Units::kRows * Units::kCols));
        const int by_blocks = G / s.R, by_steps = kblk / Units::kMinSplitSteps, by_slots = slots / s.R;
        s.split = min(min(by_blocks, kMaxSplit), min(by_steps, min(by_slots, kSplitSlots / s.R)));     // kSplitSlots nodes, too
        if (s.split < 2) s.split = 1;
    }
    s.GN = min(s.ntn, 8);
    s.GM = (G % 8 == 0 && (G / 8) % s.GN == 0) ? (G / 8) / s.GN : 1;
    return s;
}

// Left-over units are cut whatever the small experts leave to stream beside them: a long sum is further from the exact one than the sum
// of its parts (ffn_tile.hip, narrow_sums), and a large expert's rows do not depend on the small ones.  Whole ones of a first product where
// streaming fills the chip are 1 to 2 % faster: a layer of 5003 tokens, k = 2, hot share of 32 experts, 2048 x 8192, 847 us, cut 857 to 864.
__host__ __device__ __forceinline__ TileSchedule product_schedule(int big_tiles, int half_tiles, int N, int kblk, int G, bool gelu) {
    const UnitShape shape = tiled_product_units(big_tiles, half_tiles, N, kblk, G, gelu);
    if (shape == UnitShape::kFine) return schedule_of<FineUnits>(shape, half_tiles, N, kblk, G);
    if (shape == UnitShape::kNarrow) return schedule_of<NarrowUnits>(shape, big_tiles, N, kblk, G);
    return schedule_of<BigUnits>(shape, big_tiles, N, kblk, G);
}

// Called by all 1024 threads of a block, thread e owning expert e < E (row0, m rows; m = 0 when the
// expert is empty or masked out).  `big_at_min`, `half_joined`: the block's sums of big_tiles_at_min and half_tiles_joined.
// `tmp`: 48 ints of LDS.
__device__ __forceinline__ void emit_tiles(int e, int E, int row0, int m, int big_at_min, int half_joined, const TileLists tl,
                                           int32_t* tmp) {
    const int nw = (E + 63) >> 6, wave = threadIdx.x >> 6;
    const int small = (m + tl.small_rows - 1) >> __builtin_ctz(tl.small_rows);         // 16, 32 or 64 rows
    if (tl.big_min <= 0) {                                 // no large experts possible: one list (uniform)
        const int nt[1] = {small};
        int incl[1], total[1];
        block_scan(nt, incl, total, tmp, nw);
        if (wave >= nw) return;                            // no barrier from here on
        write_tiles(tl.small_tiles + incl[0] - nt[0], e, row0, m, tl.small_rows, nt[0]);
        if (e == 0) {
            tl.ntiles[0] = total[0];
            tl.ntiles[1] = tl.ntiles[kHalfCount] = 0;
        }
        return;
    }
    tl.ntiles[kTakenAt + threadIdx.x] = 0;                 // all counters: kListThreads of them
    const bool big = m >= tiled_min_rows(big_at_min, tl.join_tiles, half_joined, tl.join_half_tiles);
    const int nt[3] = {big ? 0 : small, big ? (m + kBigTileRows - 1) / kBigTileRows : 0,
                       big ? (m + kHalfTileRows - 1) / kHalfTileRows : 0};
    int incl[3], total[3];
    block_scan(nt, incl, total, tmp, nw);
    if (wave < nw) {
        write_tiles(tl.small_tiles + incl[0] - nt[0], e, row0, m, tl.small_rows, nt[0]);
        write_tiles(tl.big_tiles + incl[1] - nt[1], e, row0, m, kBigTileRows, nt[1]);
        write_tiles(tl.half_tiles + incl[2] - nt[2], e, row0, m, kHalfTileRows, nt[2]);
        if (e == 0) {
            tl.ntiles[0] = total[0];
            tl.ntiles[1] = total[1];
            tl.ntiles[kHalfCount] = total[2];
            tl.ntiles[kSplitCounter] = tl.ntiles[kSplitCounter + 1] = 0;
        }
    }
    // The schedules, by a wavefront without experts if there is one: all kernels of both products would else begin with these
    // divisions.
    if (wave == min(nw, 15)) {
        int big_tiles = 0, half_tiles = 0;
        for (int w = 0; w < nw; ++w) {
            big_tiles += tmp[16 + w];
            half_tiles += tmp[32 + w];
        }
        const int lane = threadIdx.x & 63;
        if (lane < 2)
            *reinterpret_cast<TileSchedule*>(tl.ntiles + kScheduleAt + lane * kScheduleInts) = product_schedule(
                big_tiles, half_tiles, lane ? tl.d_model : tl.d_ff, (lane ? tl.d_ff : tl.d_model) >> 5, tl.cus,
                lane == 0 && tl.gelu);
    }
}

// Unit u of the ntiles x ntn grid.  Units are numbered so that a run of consecutive units is a compact
// patch: column tiles in groups of GN, and inside a group GM row tiles at a time.  Every u in
// [0, ntiles * ntn) maps to exactly one (row tile, column tile).
__device__ __forceinline__ void unit_of(const TileSchedule& s, int u, int& mt, int& nt) {
    const int per_group = s.ntiles * s.GN;
    const int cg = u / per_group;                       // the last group may hold fewer than GN columns
    const int wn = min(s.GN, s.ntn - cg * s.GN);
    const int v = u - cg * per_group;                   // < ntiles * wn
    const int chunk = v / (s.GM * wn), slot = v - chunk * (s.GM * wn);
    mt = chunk * s.GM + slot / wn;                      // < ntiles, also in a last, shorter chunk
    nt = cg * s.GN + slot % wn;
}

// The lane's number, opaque to the compiler: what follows from it is worked out per unit instead of being kept in registers (and
// spilled) from before the loop over units, for every variant of the unit.
__device__ __forceinline__ int lane_of_unit() {
    int lane = static_cast<int>(__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0)));
    asm volatile("" : "+v"(lane));
    return lane;
}

// 4 values of one output row, columns n ... n + 3 (n a multiple of 4).  FIRST != 0 (first product; the value
// names the activation, kFirstRelu or kFirstGelu): activation, bf16, into the blocked h of N columns; FIRST == 0 (second product): fp32 into row-major y of N columns.  `bias`: the expert's N bias values
// (fp32) or NULL, added before the activation / the store.  STREAMED: the store carries the non-temporal
// hint, so the rows go to memory while the kernel runs instead of staying behind as dirty L2 lines that the
// next kernel's weight stream has to push out (the streaming units' stores; measured on the Switch-base
// preset: following product 65 -> 62 us; no effect on the fp32 rows of the second product, which are stored
// plainly).  The tiled units' rows are re-read from L2 and are stored plainly.
template <int FIRST, bool STREAMED = false>
__device__ __forceinline__ void store_out(void* outp, int row, int n, int N, const float* bias,
                                          f32x4 v) {
    if (bias != nullptr) v += *reinterpret_cast<const f32x4*>(bias + n);
    if (FIRST) {
        const f32x4 z = activate4<FIRST == kFirstGelu ? MOE_ACT_GELU : MOE_ACT_RELU>(v);
        uint2 pk;
        pk.x = pack_bf16x2(z[0], z[1]);
        pk.y = pack_bf16x2(z[2], z[3]);
        uint32_t* q = reinterpret_cast<uint32_t*>(static_cast<uint16_t*>(outp) + h_index(row, n, N >> 5));
        if (STREAMED) {
            __builtin_nontemporal_store(pk.x, q);      // merged into one 8-byte store
            __builtin_nontemporal_store(pk.y, q + 1);
        } else {
            *reinterpret_cast<uint2*>(q) = pk;
        }
    } else {
        *reinterpret_cast<f32x4*>(static_cast<float*>(outp) + static_cast<size_t>(row) * N + n) = v;
    }
}

// First-product output of two adjacent 16-column blocks (columns n0 ... n0 + 31: one k-step block of h) for
// the 16 rows of an accumulator pair.  Called by a whole wavefront (no divergence around it): lane (r, g),
// r = lane % 16 the row, g = lane / 16, holds columns n0 + 4g ... + 3 in v0 and n0 + 16 + 4g ... + 3 in v1.
// After activation and rounding, one v_permlane16_swap per packed register trades the odd 16-lane rows of the
// first block with the even rows of the second, which leaves every lane with 8 consecutive columns of its
// row: the wavefront's store is one contiguous KiB of h (16 rows x 64 bytes) instead of two stores of
// 32-byte pieces.  `row_ok`: the lane's row exists (the others take part in the exchange only).
template <int FIRST, bool STREAMED>
__device__ __forceinline__ void store_h_pair(void* outp, int row, bool row_ok, int n0, int N,
                                             const float* bias, f32x4 v0, f32x4 v1) {
    static_assert(FIRST != 0, "first product only");
    const int g = lane_of_unit() >> 4;
    if (bias != nullptr) {
        v0 += *reinterpret_cast<const f32x4*>(bias + n0 + g * 4);
        v1 += *reinterpret_cast<const f32x4*>(bias + n0 + 16 + g * 4);
    }
    constexpr int ACT = FIRST == kFirstGelu ? MOE_ACT_GELU : MOE_ACT_RELU;
    const f32x4 z0 = activate4<ACT>(v0), z1 = activate4<ACT>(v1);
    const auto lo = __builtin_amdgcn_permlane16_swap(pack_bf16x2(z0[0], z0[1]), pack_bf16x2(z1[0], z1[1]), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(pack_bf16x2(z0[2], z0[3]), pack_bf16x2(z1[2], z1[3]), false, false);
    // even g: columns 4g ... 4g + 7 of the first block; odd g: columns 4(g-1) ... + 7 of the second
    const int n = n0 + (g & 1) * 16 + (g & 2) * 4;
    if (!row_ok) return;
    uint32_t* q = reinterpret_cast<uint32_t*>(static_cast<uint16_t*>(outp) + h_index(row, n, N >> 5));
    if (STREAMED) {
        __builtin_nontemporal_store(lo[0], q);             // merged into one 16-byte store
        __builtin_nontemporal_store(hi[0], q + 1);
        __builtin_nontemporal_store(lo[1], q + 2);
        __builtin_nontemporal_store(hi[1], q + 3);
    } else {
        *reinterpret_cast<uint4*>(q) = uint4{lo[0], hi[0], lo[1], hi[1]};
    }
}

// Second-product output of rows whose layer output is written directly (FoldOut): columns n0 ... n0 + 31 of out[t] for the 16 rows of an
// accumulator pair, t and the row's gate weight w looked up by the caller.  fmaf(w, y, 0) and one rounding to bf16: what the
// combine step does for a token with a single expert.  By a whole wavefront, with the lane exchange of store_h_pair: every lane ends up with 8 consecutive
// columns of its row, one 16-byte store (64 contiguous bytes per token row and instruction).  The output is
// not read again by the layer: non-temporal.
__device__ __forceinline__ void store_folded_pair(uint16_t* out, int t, float w, bool row_ok, int n0, int N,
                                                  const float* bias, f32x4 v0, f32x4 v1) {
    const int g = lane_of_unit() >> 4;
    if (bias != nullptr) {
        v0 += *reinterpret_cast<const f32x4*>(bias + n0 + g * 4);
        v1 += *reinterpret_cast<const f32x4*>(bias + n0 + 16 + g * 4);
    }
    const auto lo = __builtin_amdgcn_permlane16_swap(pack_bf16x2(fmaf(w, v0[0], 0.f), fmaf(w, v0[1], 0.f)),
                                                     pack_bf16x2(fmaf(w, v1[0], 0.f), fmaf(w, v1[1], 0.f)), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(pack_bf16x2(fmaf(w, v0[2], 0.f), fmaf(w, v0[3], 0.f)),
                                                     pack_bf16x2(fmaf(w, v1[2], 0.f), fmaf(w, v1[3], 0.f)), false, false);
    const int n = n0 + (g & 1) * 16 + (g & 2) * 4;
    if (!row_ok) return;
    uint32_t* q = reinterpret_cast<uint32_t*>(out + static_cast<size_t>(t) * N + n);
    __builtin_nontemporal_store(lo[0], q);                 // merged into one 16-byte store
    __builtin_nontemporal_store(hi[0], q + 1);
    __builtin_nontemporal_store(lo[1], q + 2);
    __builtin_nontemporal_store(hi[1], q + 3);
}

#endif

}  // namespace moe
