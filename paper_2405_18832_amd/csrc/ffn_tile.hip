// One product of a layer that may have large experts, as one kernel:
//
//   out[row, n] = sum_k act[row, k] * W_e[n, k]          (FIRST: activation, rounded to bf16)
//
// Experts with many rows (the compute-bound "hot" experts of the paper's Section 3.3: enough tokens that the product is bound by matrix
// throughput, not by reading the expert's parameters) run in LDS-tiled MFMA units, the others in weight-streaming units
// (stream_unit.hpp), which the blocks turn to as they run out of tiled ones.  As two kernels one after the other the CUs without a unit
// of a partly filled round waited for the last one twice per product, the sums of cut units were added up by the second kernel, and
// where one kind does not occur its launch cost 2 to 3 us all the same.  Whole layers, us, two kernels -> one, with what is said of its
// units below and in stream_unit.hpp: 1501 tokens, 8 experts, 768 x 3072, GeLU 70.9 -> 64.9; 2048 tokens, 64 experts 137.1 -> 130.3; 5003
// tokens, hot share of 32 experts, 2048 x 8192, k = 2 910 -> 853; 16384 tokens, 41 experts 2240 -> 2191; 4096 tokens, skewed, 1024 x 4096
// 147.4 -> 145.3; hot share of 777 tokens, in four calls, 127.6 -> 117.0.
// The four wavefronts that stream do so within the 256 registers that 8 wavefronts per CU leave each: their loads are issued step by
// step (stream_unit.hpp) and their share of a sum is a quarter.  No register is spilled: a kernel that has scratch memory starts several us later.
//
// Big units: block = 8 wavefronts on a 256 (rows) x 256 (columns) output tile, K in steps of 32 through a
// ring of four LDS stages of 32 KiB: the copies of two stages are in flight while two are being
// read (the current one, and the next one into registers ahead of its MFMAs).  Both operands sit in LDS in MFMA-fragment order (16 x 32 fragments of
// 1 KiB, one 16-byte piece per lane), so every LDS read of the inner loop is a conflict-free
// 1 KiB wavefront read.  Global memory is copied straight into LDS (16 bytes per lane, no
// registers in between): the packed weights are already in fragment order in HBM, and for the
// activation rows (optionally gathered through `rowmap`) each lane fetches the piece that
// belongs at its own slot.  Wavefront (wm, wn) of the 2 x 4 grid owns 128 rows x 64 columns:
// 4 weight fragments (MFMA A operand) x 8 row fragments (B operand) of 16x16x32 per 32-k step,
// 128 accumulator registers.
//
// Narrow units, where big ones would leave up to half of the chip idle (tiled_product_units): 256 x 128, wavefronts 4 x 2 of
// 64 x 64 each.  Bound by the copies like the fine ones below (24 KB per step, about 48 GB/s per CU), with a quarter less of them
// per output and no exchange: 8 experts of 137 ... 228 rows, 768 x 3072, GeLU, first product 29.7 -> 25.4 us.
//
// Fine units, for products whose big units would leave most of the chip idle: 128 x 128, the
// 8 wavefronts as two groups of four (64 x 64 each) that take half of the contraction each, through a ring of their own
// with stages half the size, and add up in LDS.  A CU can pull about 35 GB/s from beyond its L2 however much it has in
// flight, so a handful of big units is bound by the CUs they run on, not by memory or matrix units.  Per output they copy
// twice the bytes of big units, and they are cut less along K into parts that go through memory.  Measured, big ->
// fine, the second figure of a sum being the kernel that adds up the parts: 8 experts of 137 ... 228 rows, 768 x 3072:
// 39.7 -> 35.7 us (96 big units of 24 steps, GeLU) and 33.2 + 8.9 -> 19.4 + 8.9 us (24 units of 96 steps); one expert
// of 327 rows, 1024 x 4096: 28 -> 14 and 32 -> 14 us; 16 big row tiles, K = 4096, N = 1024: 40.6 + 43.4 -> 37.6 + 23.9 us.
// As blocks of one group, two per CU, the last was 50.1 + 36.7 us: twice the parts.
//
// Blocks are persistent over (row tile, column tile) pairs taken
// from the device-built list of large-expert row tiles.  (Figures of sums above: the parts added up by a kernel of its own.)
#include <type_traits>

#include <algorithm>

#include "stream_unit.hpp"

namespace moe {

constexpr int kTK = 32;             // k per LDS stage
constexpr int kStages = 4;          // ring of LDS stages: two being read, two in flight (a fifth, which
                                    // fits, bought nothing: the copies are not limited by ring depth)
constexpr int kAhead = kStages - 1; // the iteration for stage j issues the copies of stage j + kAhead
constexpr int kWaves = 8;           // wavefronts of a block
constexpr int kRingBytes = kStages * 2 * kBigTileRows * kTK * 2;   // 128 KiB of stages
constexpr int kTileLds = kRingBytes + 32 * 1024;                   // and where the groups of a fine unit exchange sums

// Wait until at most `stages` stages' worth of this wavefront's copies (COPIES each, 3 or 4) are still in flight.
template <int COPIES>
__device__ __forceinline__ void wait_copies(int stages) {
    static_assert(COPIES <= 5, "vmcnt up to 15 sits in the low four bits");
    if (stages >= 3) __builtin_amdgcn_s_waitcnt(0x0F70 + 3 * COPIES);
    else if (stages == 2) __builtin_amdgcn_s_waitcnt(0x0F70 + 2 * COPIES);
    else if (stages == 1) __builtin_amdgcn_s_waitcnt(0x0F70 + COPIES);
    else __builtin_amdgcn_s_waitcnt(0x0F70);
}

// Register fragments of one wavefront: the 4 weight fragments of a stage, double-buffered over stages,
// and the 8 row fragments as 4 pairs (big units) or the 4 row fragments as 2 pairs, double-buffered like the weights.
struct StageFrags {
    bf16x8 w[2][4];
    bf16x8 x[4][2];
};

__device__ __forceinline__ void lds_read_w(bf16x8 (&w)[4], const unsigned char* base) {
#pragma unroll
    for (int nf = 0; nf < 4; ++nf) w[nf] = *reinterpret_cast<const bf16x8*>(base + nf * 1024);
}

__device__ __forceinline__ void lds_read_x(bf16x8 (&x)[2], const unsigned char* base, int pair) {
    x[0] = *reinterpret_cast<const bf16x8*>(base + (2 * pair) * 1024);
    x[1] = *reinterpret_cast<const bf16x8*>(base + (2 * pair + 1) * 1024);
}

// 4 weight fragments x row-fragment pair P: 8 MFMAs
template <int P, int RF>
__device__ __forceinline__ void mfma_pair(const bf16x8 (&w)[4], const bf16x8 (&x)[2], f32x4 (&acc)[4][RF]) {
#pragma unroll
    for (int nf = 0; nf < 4; ++nf) {
        acc[nf][2 * P] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[nf], x[0], acc[nf][2 * P], 0, 0, 0);
        acc[nf][2 * P + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[nf], x[1], acc[nf][2 * P + 1], 0, 0, 0);
    }
}

// Partial sums of a narrow unit's contraction: no fewer than in the units that would run without narrow ones, because the rounding
// error of a sum grows with its length.  Those were big ones, cut or not (sch.sums), or, for the first product of a GeLU layer, fine
// ones, which add up two halves, the left-over ones of them cut again from 48 steps on.
// fp32 rows of 72 narrow units against 64 bits, relative error: 64 steps in one sum 9.1e-8, in two 6.7e-8; 96 in one 11.6e-8, in three
// 7.1e-8.
template <int FIRST>
__device__ __forceinline__ int narrow_sums(const TileSchedule& sch, int kblk) {
    return FIRST == kFirstGelu ? max(sch.sums, kblk < 2 * FineUnits::kMinSplitSteps ? min(kblk, 2) : 4) : sch.sums;
}

// 16 bytes per lane of memory that another XCD's blocks read or have written in the same launch: sc1 (bit 4 of the cache-policy
// operand) sends the store through this XCD's L2 to memory, and makes the load miss in it.
constexpr int kAgentScope = 16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

// Adds up the parts of a unit that was cut along K, in a tree over the part numbers: (0 + 1) + (2 + 3) and so on, whichever block
// computed them.  Of the two blocks that meet at a node, the one that gets there first leaves its sum in the workspace and is done;
// the other adds that to its own and goes on to the next level.  Nobody waits for anybody, so that it does not matter which blocks
// are resident, and the sum does not depend on the order of arrival.  Returns whether this block has the whole sum.
// `first_slot`: number of the unit's part 0 among all parts; part p owns partial tile first_slot + p (tile_floats floats), and the
// node whose right-hand side begins with part p the counter joined[first_slot + p], zero at the start of the launch.
// A wavefront reads only what the same wavefront of the other block has stored (the tile lies in accumulator order).
// Visibility: the sums are stored with agent scope and have arrived in memory (vmcnt) for every wavefront (barrier) before the
// counter is raised; a counter that reads 1 therefore means that the other block's sum can be loaded.  (A fence would write back
// all of the XCD's L2 for these few lines: such a version cost more than it saved.)
template <int OF, int RF>
__device__ __forceinline__ bool join_parts(f32x4 (&acc)[4][RF], int part, int nparts, int first_slot, int tile_floats,
                                           int32_t* joined, float* partials, int wave, int* flag) {
    const int lane = threadIdx.x & 63;
    const int wave_bytes = OF * 4 * 1024;
    auto tile_of = [&](int p) {
        return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<char*>(partials + static_cast<size_t>(first_slot + p) * tile_floats),
                                                 0, tile_floats * 4, 0x00027000);
    };
    const int at = wave * wave_bytes + lane * 16;
    for (int level = 0; (1 << level) < nparts; ++level) {
        const int mine = part >> level, other = mine ^ 1;
        if ((other << level) >= nparts) continue;              // nobody there: up to the next level
        int32_t* const node = joined + first_slot + ((mine | 1) << level);
        if (threadIdx.x == 0) *flag = __hip_atomic_load(node, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        bool second = __builtin_amdgcn_readfirstlane(*flag) != 0;
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");          // the flag is read
        if (!second) {
            const auto tile = tile_of(mine << level);
#pragma unroll
            for (int tf = 0; tf < OF; ++tf)
#pragma unroll
                for (int nf = 0; nf < 4; ++nf)
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[nf][tf]), tile, at + nf * 1024, tf * 4096,
                                                           kAgentScope);
            asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
            if (threadIdx.x == 0) *flag = __hip_atomic_fetch_add(node, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            second = __builtin_amdgcn_readfirstlane(*flag) != 0;
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            if (!second) return false;
        }
        const auto tile = tile_of(other << level);
#pragma unroll
        for (int tf = 0; tf < OF; ++tf) {
            u32x4 v[4];
#pragma unroll
            for (int nf = 0; nf < 4; ++nf) v[nf] = __builtin_amdgcn_raw_buffer_load_b128(tile, at + nf * 1024, tf * 4096, kAgentScope);
#pragma unroll
            for (int nf = 0; nf < 4; ++nf) acc[nf][tf] += __builtin_bit_cast(f32x4, v[nf]);
        }
    }
    return true;
}

template <int FIRST, bool FOLD, typename Units>
__device__ __forceinline__ void run_units(const uint16_t* __restrict__ act, const int32_t* __restrict__ rowmap,
                                          const uint16_t* __restrict__ wpk, void* __restrict__ outp,
                                          const Tile* __restrict__ tiles, const TileSchedule& sch,
                                          int32_t* part_counter, int32_t* joined, float* partials, int N, int K,
                                          int act_kmajor, const float* __restrict__ bias, const FoldOut& fold,
                                          unsigned char* smem) {
    constexpr bool FINE = Units::kGroups == 2;
    constexpr bool NARROW = std::is_same_v<Units, NarrowUnits>;
    constexpr int kTM = Units::kRows, kTN = Units::kCols;
    constexpr int kGroupWaves = kWaves / Units::kGroups;
    constexpr int WN = kTN / 64;                        // wavefronts of a group side by side
    constexpr int WM = kGroupWaves / WN;                // and in the row direction
    constexpr int RF = kTM / WM / 16;                   // row fragments of a wavefront
    constexpr bool FOUR = RF == 4;                      // 64 x 64 per wavefront, else 128 x 64
    constexpr int kRowBytes = kTM * kTK * 2;            // rows of a stage; the weights lie behind them
    constexpr int kStageBytes = kRowBytes + kTN * kTK * 2;
    constexpr int RC = kTM / 16 / kGroupWaves, WC = kTN / 16 / kGroupWaves;    // row and weight fragments a wavefront copies per stage
    static_assert((RF == 4 || RF == 8) && RC == 2 && (WC == 1 || WC == 2), "the shapes the loop is written for");
    static_assert(Units::kGroups * kStages * kStageBytes <= kRingBytes, "the groups' rings fit into the LDS");
    // between units, when no stage is in use, the first word of the ring passes the next part's number on
    int* next_part = reinterpret_cast<int*>(smem);
    f32x4* exchange = reinterpret_cast<f32x4*>(smem + kRingBytes);
    const int block_wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int group = FINE ? block_wave / kGroupWaves : 0;
    // stage st of a group: kTM / 16 row fragments at ring + st * kStageBytes, kTN / 16 weight fragments behind them
    unsigned char* ring = smem + group * (kStages * kStageBytes);

    const int t = threadIdx.x, wave = block_wave % kGroupWaves, lane = t & 63;
    const int wm = wave / WN, wn = wave % WN;
    const int r = lane & 15, g = lane >> 4;
    const int nblk = N >> 4, kblk = K >> 5;
    const int G = gridDim.x;
    // LDS byte address of the first row fragment that this wavefront copies in, stage 0, and where its weight fragments lie from there
    const uint32_t copy_base = lds_address(ring) + RC * wave * 1024, weights_at = kRowBytes - (RC - WC) * wave * 1024;

    // Blocks are handed to the 8 XCDs round-robin, and each XCD has its own L2: block b takes position pb
    // of a round, so that the blocks of one XCD hold G / 8 consecutive units, a GM x GN patch whose
    // activation panels that L2 serves GN times and whose weight panels GM times.
    const int pb = (G % 8 == 0) ? static_cast<int>(blockIdx.x & 7) * (G >> 3) + static_cast<int>(blockIdx.x >> 3)
                                : static_cast<int>(blockIdx.x);
    const int nleft = sch.R * sch.split;                // parts of the left-over units
    const int sums = narrow_sums<FIRST>(sch, kblk);     // of a narrow unit

    // A unit of work: (row tile mt, column tile nt) over k-steps [kb0, kb0 + nk), whole (nparts == 1) or
    // one of nparts parts of a left-over unit.
    struct Unit {
        int u, part, nparts, nt;
        int kb0, nk, longest;       // the group's run of k-steps; the number of steps of the first group
        Tile tl;
        bool valid;
    };
    auto unit_at = [&](int it) {
        Unit w;
        w.valid = true;
        w.part = 0;
        if (it < sch.rounds) {
            w.u = it * G + pb;
            w.nparts = 1;
        } else {
            // The parts of the left-over units; there are no more of them than blocks.
            int id;
            if (sch.rounds > 0) {
                // After full rounds the blocks arrive at different times (a few per cent of the rounds' time):
                // a counter hands the parts out in order of arrival (which block computes a part has no
                // influence on the result).  The first word of the ring is free now: every wavefront that
                // gets past the first barrier has read its last stage.
                __syncthreads();
                if (t == 0) *next_part = (nleft > 0) ? atomicAdd(part_counter, 1) : 0;
                __syncthreads();
                id = *next_part;
                w.valid = id < nleft;                      // block-uniform; every block ends up here
            } else {
                // No full round: all blocks start together, one part each.  Part-major numbering and an
                // equal run of consecutive numbers per XCD, so that the blocks of an XCD hold the same
                // K-slice of neighbouring units, which share their row and weight panels in that XCD's L2
                // (handed out in order of arrival, the parts of a Switch-large-sized second product hit in
                // L2 0.46 of the time and ran at the rate their CUs could pull from memory).
                const int n8 = (nleft + 7) >> 3;
                const bool xcds = G % 8 == 0;
                id = xcds ? static_cast<int>(blockIdx.x & 7) * n8 + static_cast<int>(blockIdx.x >> 3)
                          : static_cast<int>(blockIdx.x);
                w.valid = it == 0 && id < nleft && (!xcds || static_cast<int>(blockIdx.x >> 3) < n8);
                id = id % max(sch.R, 1) * sch.split + id / max(sch.R, 1);     // (unit, part) from part-major
            }
            w.u = sch.rounds * G + (w.valid ? id / sch.split : 0);
            w.part = w.valid ? id % sch.split : 0;
            w.nparts = sch.split;
        }
        int mt = 0;
        w.nt = 0;
        if (w.valid) unit_of(sch, w.u, mt, w.nt);
        w.kb0 = kblk * w.part / w.nparts;                  // kblk * kMaxSplit fits easily
        w.nk = w.longest = kblk * (w.part + 1) / w.nparts - w.kb0;
        if constexpr (FINE) {
            w.longest = (w.nk + 1) >> 1;
            if (group == 1) w.kb0 += w.longest;
            w.nk = group == 0 ? w.longest : w.nk - w.longest;
        }
        w.tl = tiles[w.valid ? mt : 0];
        return w;
    };

    // RC + WC copies per wavefront and stage; stages are copied in order, so the pointers just advance.  A lane fetches the 16
    // bytes that belong at its own slot of the fragment: row (lane % 16), k-group (lane / 16).
    const uint16_t* arow[RC];
    const uint16_t* brow[WC];
    const size_t kstride = act_kmajor ? kStepStride : 32;   // elements per k-step
    auto copy_piece = [&](int st, int q) {             // q = 0 ... 3: row fragment 0, weight 0, row 1, weight 1
        const int i = q >> 1;
        if ((q & 1) == 0) {
            copy16_to_lds(arow[i], copy_base + st * kStageBytes + i * 1024);
            arow[i] += kstride;
        } else if (i < WC) {
            copy16_to_lds(brow[i % WC], copy_base + st * kStageBytes + weights_at + i * 1024);
            brow[i % WC] += 512;
        }
    };
    auto stage_in = [&](int st) {
#pragma unroll
        for (int q = 0; q < 4; ++q) copy_piece(st, q);
    };
    // Point the copies at a unit's first k-step.
    auto point_copies_at = [&](const Unit& w) {
#pragma unroll
        for (int i = 0; i < RC; ++i) {
            int row = w.tl.row0 + min((RC * wave + i) * 16 + r, w.tl.rows - 1);
            if (rowmap != nullptr) row = rowmap[row];
            // operand rows are row-major (the caller's x or x_perm) or k-step-major (h, gathered x)
            arow[i] = act_kmajor ? act + h_index(row, w.kb0 * 32 + g * 8, kblk)
                                 : act + static_cast<size_t>(row) * K + static_cast<size_t>(w.kb0) * 32 + g * 8;
        }
#pragma unroll
        for (int i = 0; i < WC; ++i) {
            const int nb = min(w.nt * (kTN / 16) + WC * wave + i, nblk - 1);
            brow[i] = wpk + ((static_cast<size_t>(w.tl.expert) * nblk + nb) * kblk + w.kb0) * 512 + lane * 8;
        }
    };
    // The ring runs on across units: `slot` is the slot of the current unit's current stage, and the first
    // stage of the next unit follows the last stage of this one.
    int slot = 0;
    // Start a unit from a standstill: its first stages into the slots from `slot` on.  Every wavefront must be
    // done reading the ring (its MFMAs have consumed the last stage): a bare barrier, so that output stores
    // still in flight need not complete first.
    auto start_unit = [&](const Unit& w) {
        point_copies_at(w);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
        for (int sidx = 0; sidx < kAhead; ++sidx)
            if (sidx < w.nk) stage_in((slot + sidx) % kStages);
    };

    const int wave_w = kRowBytes + (wn * 4 * 64 + lane) * 16, wave_x = (wm * RF * 64 + lane) * 16;
    Unit cur = unit_at(0);
    if (cur.valid) start_unit(cur);
    for (int it = 0; cur.valid; ++it) {
        const int nk = cur.nk;
        // Inside the full rounds the next unit is known in advance: its tile descriptor is fetched now, not
        // between the units, where the load's latency would be exposed (1.5 us per unit).
        const bool next_known = it + 1 < sch.rounds;
        Unit nxt;
        if (next_known) nxt = unit_at(it + 1);
        // The next unit's first stages go out during this unit's last iterations, in the slots that fall free
        // there, when the unit is known by then, needs no row lookups (a vector load here would make the
        // compiler wait for every copy in flight) and both units are at least as long as the ring is deep.
        const bool ahead = !FOUR && next_known && nxt.valid && rowmap == nullptr && nk >= kAhead && nxt.nk >= kAhead;
        f32x4 acc[4][RF];
#pragma unroll
        for (int nf = 0; nf < 4; ++nf)
#pragma unroll
            for (int tf = 0; tf < RF; ++tf) acc[nf][tf] = f32x4{0.f, 0.f, 0.f, 0.f};
        // Narrow units: the contraction is added up in `sums` about equal runs of steps, one after the other, and these in order.
        f32x4 done[NARROW ? 4 : 1][NARROW ? RF : 1];
        int run = 1, run_end = NARROW ? nk / sums : 0;
        if constexpr (NARROW) {
#pragma unroll
            for (int nf = 0; nf < 4; ++nf)
#pragma unroll
                for (int tf = 0; tf < RF; ++tf) done[nf][tf] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        auto end_run = [&](int j) {
            if constexpr (NARROW) {
                if (j != run_end || run == sums) return;    // block-uniform
#pragma unroll
                for (int nf = 0; nf < 4; ++nf)
#pragma unroll
                    for (int tf = 0; tf < RF; ++tf) {
                        done[nf][tf] += acc[nf][tf];
                        acc[nf][tf] = f32x4{0.f, 0.f, 0.f, 0.f};
                    }
                ++run;
                run_end = nk * run / sums;
            }
        };
        StageFrags fr;
        // One stage of 32 k, software-pipelined across stages so that the MFMA pipe never waits for LDS.
        // The iteration for stage j starts by making sure that stage j + 1 has landed for every wavefront
        // (own copies by vmcnt, the others' by the barrier; __syncthreads() would drain every outstanding
        // copy and empty the ring) and by refilling the slot of stage j - 1, which nobody reads any more,
        // with stage j + kAhead.  The fragments of stage j are in registers by then, except row pair 3: every
        // group of 8 MFMAs is followed by the LDS reads that refill the registers it has just freed with
        // stage j + 1, so each read has at least 8 MFMAs to complete.  (At its first use of an LDS result
        // after a global-to-LDS copy was issued the compiler waits for all outstanding LDS reads, not
        // only the needed ones: here that is at the first MFMA, when only old reads are outstanding.)
        // `steady`: stage j + kAhead exists, so nothing in the iteration is conditional.
        auto iterate = [&](auto cbuf, auto steady, int j) {
            constexpr int C = decltype(cbuf)::value;
            constexpr bool STEADY = decltype(steady)::value;
            end_run(j);
            const int slot_next = slot + 1 == kStages ? 0 : slot + 1;
            const int slot_free = slot == 0 ? kStages - 1 : slot - 1;          // held stage j - 1
            const unsigned char* st_cur = ring + slot * kStageBytes;
            const unsigned char* st_nxt = ring + slot_next * kStageBytes;
            const bool more = STEADY || j + 1 < nk;        // block-uniform
            if (more) {
                // stages j + 2 ... j + kAhead - 1 (as far as they exist) may stay in flight; with the next unit's
                // stages behind them that is always kAhead - 2 stages' worth
                wait_copies<RC + WC>((STEADY || ahead) ? kAhead - 2 : min(j + kAhead - 1, nk - 1) - (j + 1));
                asm volatile("s_barrier" ::: "memory");
            } else if (ahead) {
                asm volatile("s_barrier" ::: "memory");   // the slot of stage j - 1 is about to be refilled
            }
            // from here on the stages that go out are the next unit's
            if (!STEADY && ahead && j + kAhead == nk) point_copies_at(nxt);
            // the four copies of stage j + kAhead are issued between the first MFMAs, whose execution
            // covers the scalar and address arithmetic of the copies
            const bool refill = (more && (STEADY || j + kAhead < nk)) || (!STEADY && ahead && j + kAhead >= nk);
            // 64 x 64: both row pairs of stage j are in registers, and the second group of MFMAs covers the reads of
            // stage j + 1 into the other buffers.
            const bf16x8 (&x0)[2] = fr.x[FOUR ? 2 * C : 0];
#pragma unroll
            for (int nf = 0; nf < 4; ++nf) {
                __builtin_amdgcn_sched_barrier(0);
                acc[nf][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr.w[C][nf], x0[0], acc[nf][0], 0, 0, 0);
                acc[nf][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr.w[C][nf], x0[1], acc[nf][1], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (refill) copy_piece(slot_free, nf);
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (FOUR) {
                if (more) {
                    lds_read_w(fr.w[C ^ 1], st_nxt + wave_w);
                    lds_read_x(fr.x[2 * (C ^ 1)], st_nxt + wave_x, 0);
                    lds_read_x(fr.x[2 * (C ^ 1) + 1], st_nxt + wave_x, 1);
                }
                __builtin_amdgcn_sched_barrier(0);
                mfma_pair<1>(fr.w[C], fr.x[2 * C + 1], acc);
                __builtin_amdgcn_sched_barrier(0);
            } else {
                lds_read_x(fr.x[3], st_cur + wave_x, 3);
                if (more) {
                    lds_read_w(fr.w[C ^ 1], st_nxt + wave_w);
                    lds_read_x(fr.x[0], st_nxt + wave_x, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                mfma_pair<1>(fr.w[C], fr.x[1], acc);
                __builtin_amdgcn_sched_barrier(0);
                if (more) lds_read_x(fr.x[1], st_nxt + wave_x, 1);
                __builtin_amdgcn_sched_barrier(0);
                mfma_pair<2>(fr.w[C], fr.x[2], acc);
                __builtin_amdgcn_sched_barrier(0);
                if (more) lds_read_x(fr.x[2], st_nxt + wave_x, 2);
                __builtin_amdgcn_sched_barrier(0);
                mfma_pair<3>(fr.w[C], fr.x[3], acc);
                __builtin_amdgcn_sched_barrier(0);
            }
            slot = slot_next;
        };

        // The first waits may also wait for the previous unit's output stores, which were issued after this
        // unit's first copies and count in vmcnt like them: never too short, since no more than the given
        // number of operations stays outstanding and the copies complete in order.
        wait_copies<RC + WC>(min(kAhead, nk) - 1);                  // stage 0 has landed ...
        asm volatile("s_barrier" ::: "memory");           // ... for every wavefront
        lds_read_w(fr.w[0], ring + slot * kStageBytes + wave_w);
        lds_read_x(fr.x[0], ring + slot * kStageBytes + wave_x, 0);
        lds_read_x(fr.x[1], ring + slot * kStageBytes + wave_x, 1);
        if constexpr (!FOUR) lds_read_x(fr.x[2], ring + slot * kStageBytes + wave_x, 2);
        int j = 0;
        for (; j + 1 + kAhead < nk; j += 2) {
            iterate(std::integral_constant<int, 0>{}, std::true_type{}, j);
            iterate(std::integral_constant<int, 1>{}, std::true_type{}, j + 1);
        }
        // at most kAhead + 1 stages are left, and j is even: the buffers keep alternating
        if (j < nk) iterate(std::integral_constant<int, 0>{}, std::false_type{}, j);
        if (j + 1 < nk) iterate(std::integral_constant<int, 1>{}, std::false_type{}, j + 1);
        if (j + 2 < nk) iterate(std::integral_constant<int, 0>{}, std::false_type{}, j + 2);
        if (j + 3 < nk) iterate(std::integral_constant<int, 1>{}, std::false_type{}, j + 3);
        if (j + 4 < nk) iterate(std::integral_constant<int, 0>{}, std::false_type{}, j + 4);

        if constexpr (NARROW) {
#pragma unroll
            for (int nf = 0; nf < 4; ++nf)
#pragma unroll
                for (int tf = 0; tf < RF; ++tf) acc[nf][tf] = done[nf][tf] + acc[nf][tf];
        }
        if constexpr (FINE) {
            // the second group may have one step and so one barrier less
            for (int i = cur.longest - max(nk, 1); i > 0; --i) asm volatile("s_barrier" ::: "memory");
            // The groups' sums meet in LDS: the first keeps row fragments 0 and 1 of every wavefront, the second 2 and 3, and
            // each takes the other's share of its own, a fragment row at a time (first group's sum + second group's).
            f32x4* to = exchange + (group * kGroupWaves + wave) * 4 * 64 + lane;
            const f32x4* from = exchange + ((1 - group) * kGroupWaves + wave) * 4 * 64 + lane;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
#pragma unroll
                for (int nf = 0; nf < 4; ++nf) to[nf * 64] = group == 0 ? acc[nf][2 + i] : acc[nf][i];
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
                for (int nf = 0; nf < 4; ++nf) acc[nf][i] = (group == 0 ? acc[nf][i] : acc[nf][2 + i]) + from[nf * 64];
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            }
        }
        constexpr int OF = RF / Units::kGroups;            // row fragments of output per wavefront, from the first on:
        const int lr0 = wm * (RF * 16) + group * OF * 16;

        // The next unit's first copies go out before this unit's output is stored: the copies' latency and
        // the stores overlap, and the load of the next tile's descriptor does not wait behind the stores.
        if (!next_known) nxt = unit_at(it + 1);
        if (nxt.valid && !ahead) start_unit(nxt);

        // The last of a cut unit's parts to finish adds them all up and stores the unit's output.
        const bool whole = cur.nparts == 1 ||
                           join_parts<OF>(acc, cur.part, cur.nparts, (cur.u - sch.rounds * G) * cur.nparts, kTM * kTN, joined,
                                          partials, block_wave, reinterpret_cast<int*>(exchange));
        // Lane holds 4 consecutive columns of one row per accumulator.
        if (whole) {
            const int el = lane_of_unit(), er = el & 15, eg = el >> 4;
            const float* be = bias ? bias + static_cast<size_t>(cur.tl.expert) * N : nullptr;
#pragma unroll
            for (int tf = 0; tf < OF; ++tf) {
                if (lr0 + tf * 16 >= cur.tl.rows) break;     // wave-uniform: no row from here on
                const int lr = lr0 + tf * 16 + er;
                const bool ok = lr < cur.tl.rows;
                if constexpr (FIRST != 0) {
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        const int nb = cur.nt * (kTN / 16) + wn * 4 + 2 * m;   // N / 16 is even: a pair exists as a whole
                        if (nb >= nblk) continue;                       // wave-uniform
                        store_h_pair<FIRST, false>(outp, cur.tl.row0 + lr, ok, nb * 16, N, be, acc[2 * m][tf],
                                                   acc[2 * m + 1][tf]);
                    }
                } else {
                    if constexpr (FOLD) {                               // folded layer output (top-1, no mask)
                        const int ftok = ok ? fold.tokmap[cur.tl.row0 + lr] : 0;
                        const float fw = ok ? fold.gate[ftok] : 0.f;
#pragma unroll
                        for (int m = 0; m < 2; ++m) {
                            const int nb = cur.nt * (kTN / 16) + wn * 4 + 2 * m;
                            if (nb >= nblk) continue;                   // wave-uniform
                            store_folded_pair(static_cast<uint16_t*>(fold.out), ftok, fw, ok, nb * 16, N, be, acc[2 * m][tf], acc[2 * m + 1][tf]);
                        }
                    } else {
#pragma unroll
                        for (int nf = 0; nf < 4; ++nf) {
                            const int nb = cur.nt * (kTN / 16) + wn * 4 + nf;
                            if (ok && nb < nblk)
                                store_out<0>(outp, cur.tl.row0 + lr, nb * 16 + eg * 4, N, be, acc[nf][tf]);
                        }
                    }
                }
            }
        }
        cur = nxt;
    }
}

// The streaming units of a product (stream_unit.hpp), by the first four wavefronts of every block of the product kernel; the others
// have ended, and barriers do not wait for wavefronts that have.  Four are as many as stream fastest: a second set on every CU was
// slower (64 experts of about 32 rows, 768 x 3072: 67 -> 78 us a product).
// Each XCD has a run of consecutive units, the column groups of one tile after the other, so that a tile's rows are fetched into one
// L2; within a run, blocks that had no tiled unit begin with the first units, and from then on units are handed out in order of
// arrival, from the other XCDs' runs too when the block's own is empty.
template <int KSPLIT, int FIRST, bool FOLD>
__device__ __forceinline__ void run_stream_units(const uint16_t* __restrict__ act, const int32_t* __restrict__ rowmap,
                                                 const uint16_t* __restrict__ wpk, void* __restrict__ outp,
                                                 const Tile* __restrict__ tiles, int ntiles, int32_t* taken, int busy, int N, int K,
                                                 int act_kmajor, const float* __restrict__ bias,
                                                 const FoldOut& fold, unsigned char* smem, const int wave) {
    constexpr int TFMAX = 4, NGB = 4 / KSPLIT;              // row fragments of a tile; column groups (of 64) per unit
    unsigned char* tok_lds = smem;
    f32x4* red = reinterpret_cast<f32x4*>(smem);
    static_assert((KSPLIT - 1) * NGB * 4 * TFMAX * 1024 <= kRingBytes && kStreamRowLdsMax <= kRingBytes, "both fit in front of `next_unit`");
    int* next_unit = reinterpret_cast<int*>(smem + kRingBytes);
    const int lane = static_cast<int>(__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0)));
    const int ks = wave % KSPLIT, ngs = wave / KSPLIT;
    const int nblk = N >> 4, kblk = K >> 5;
    const int ngchunks = (nblk + 4 * NGB - 1) / (4 * NGB);
    const int kb_per = (kblk + KSPLIT - 1) / KSPLIT;
    const int kb0 = min(kblk, ks * kb_per), kb1 = min(kblk, kb0 + kb_per);
    const int units = ntiles * ngchunks;

    const int G = gridDim.x, nx = G % 8 == 0 ? 8 : 1, blocks = G / nx;
    const int x = static_cast<int>(blockIdx.x) % nx, rank = static_cast<int>(blockIdx.x) / nx;
    const int fixed = blocks - busy;                        // units at the head of a run that are not handed out
    auto run_begin = [&](int i) { return static_cast<int>(static_cast<long>(units) * i / nx); };
    auto take = [&](int i) { return __hip_atomic_fetch_add(taken + i * kTakenStride, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    // A unit for a block whose own run is empty, or -1: by the first wavefront, which looks at all runs at once.
    auto take_any = [&]() {
        for (;;) {                                          // ends: counters only rise, and every turn raises one that is not at its end
            const int i = min(lane, nx - 1);
            const int end = run_begin(i + 1) - run_begin(i) - fixed;
            const int c = __hip_atomic_load(taken + i * kTakenStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint64_t left = __ballot(lane < nx && c < end);
            if (left == 0) return -1;
            const uint64_t from = left >> x << x;           // the next run after the block's own that has some
            const int y = __builtin_ctzll(from != 0 ? from : left);
            int n = 0;
            if (lane == 0) n = take(y);
            n = run_begin(y) + fixed + __builtin_amdgcn_readfirstlane(n);
            if (n < run_begin(y + 1)) return n;
        }
    };
    // The next unit is asked for when the current one's last loads are out, so that its number is there when they are consumed and no
    // block holds a unit that an idle one could run; its tile is looked up while the current one's output is stored.  (Asked for at the
    // start of the current unit: 16 experts of the hot share of 777 tokens, 1024 x 4096: 117 -> 131 us for the four calls.)
    // Without tiled units all blocks start together and units cost about the same: every block takes its share, nothing is counted.
    // Layers without a large expert, us, counted -> shares: 64 experts, 768 x 3072, 256, 700, 2048 and 2900 tokens 121.0, 125.0, 133.9, 139.0 ->
    // 117.8, 121.3, 129.6, 133.1; 128 experts, 900 tokens 224.8 -> 218.9.  It is the other way with units for some of the XCDs only (8 experts,
    // 160 and 400 tokens 34.0, 40.9 -> 39.8, 43.8), where a run for each XCD spreads them, and with long units in several rounds (2048 x 8192,
    // k = 2, 208 tokens 1281 -> 1341; 1024 x 4096, 128 experts, 300 to 3000 tokens 328 to 386 -> 331 to 388).
    struct NextUnit {
        decltype(take)& take_;
        const Tile* tiles;
        int* slot;
        int x, fixed, x0, x1, ngchunks;
        bool counted, first;                                // first: the block's first lane
        int asked, unit;
        Tile tl;
        __device__ __forceinline__ void look_up() {
            if (unit >= 0) tl = tiles[unit / ngchunks];
        }
        __device__ __forceinline__ void loads_out() {
            if (counted && first) asked = take_(x);
        }
        __device__ __forceinline__ void loads_done() {
            if (counted && first) *slot = asked;
        }
        __device__ __forceinline__ bool meet() const { return counted; }
        __device__ __forceinline__ void met() {
            unit = counted ? x0 + fixed + __builtin_amdgcn_readfirstlane(*slot) : unit + static_cast<int>(gridDim.x);
            if (unit >= x1) unit = -1;
            look_up();
        }
    };
    const bool counted = busy > 0;
    NextUnit next{take, tiles, next_unit, x, fixed, run_begin(x), counted ? run_begin(x + 1) : units, ngchunks, counted,
                  wave == 0 && lane == 0, 0, 0, {}};
    next.unit = counted ? (rank >= busy ? next.x0 + rank - busy : next.x1) : x * blocks + rank;
    if (next.unit >= next.x1) next.unit = -1;
    next.look_up();
    for (;;) {
        if (next.unit < 0) {                                // block-uniform
            if (!next.counted) return;
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");      // the last number has been read by all
            if (wave == 0) {
                const int got = take_any();
                if (lane == 0) *next_unit = got;
            }
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            next.unit = __builtin_amdgcn_readfirstlane(*next_unit);
            if (next.unit < 0) return;
            next.look_up();
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");      // read by all before it is written again
        }
        const Tile tl{__builtin_amdgcn_readfirstlane(next.tl.expert), __builtin_amdgcn_readfirstlane(next.tl.row0),
                      __builtin_amdgcn_readfirstlane(next.tl.rows), 0};
        const int ng = next.unit % ngchunks * NGB + ngs;
        const bool active = ng * 4 < nblk;                  // wave-uniform
        const int tfc = (tl.rows + 15) >> 4;                // token fragments in use: block-uniform
        const bool km = act_kmajor != 0;
        auto run = [&](auto frags) {
            constexpr int TFC = decltype(frags)::value;
            if constexpr (KSPLIT == 1)
                stream_unit_lds<TFC, FIRST, FOLD>(act, rowmap, wpk, outp, tl, ng, active, N, K, km, bias, tok_lds, fold, wave, next);
            else
                stream_unit<TFC, TFMAX, KSPLIT, FIRST, FOLD, 4>(act, rowmap, wpk, outp, tl, ng, active, N, K, kb0, kb1, red, km, bias,
                                                                fold, wave, next);
        };
        if (tfc == 4) run(std::integral_constant<int, 4>{});
        else if (tfc == 3) run(std::integral_constant<int, 3>{});
        else if (tfc == 2) run(std::integral_constant<int, 2>{});
        else run(std::integral_constant<int, 1>{});
    }
}

// The arguments of one product: in the kernel's argument segment, read where they are needed.
struct ProductArgs {
    const uint16_t* act;
    const int32_t* rowmap;
    const uint16_t* wpk;
    void* outp;
    const Tile* small_tiles;
    const Tile* big_tiles;
    const Tile* half_tiles;
    int32_t* lists;
    float* partials;
    const float* bias;
    FoldOut fold;
    int N, K, act_kmajor;
    int kinds;                          // kTiledUnits, kStreamUnits or both
};
typedef const ProductArgs __attribute__((address_space(4))) * product_args_t;

// One product of a layer that may have large experts: these experts' units first, then the small experts' on whichever blocks are
// free, side by side with the tiled units that still run.  Profiled calls that time the two kinds apart launch it once for each.
template <int KSPLIT, int FIRST, bool FOLD>
__global__ __launch_bounds__(kWaves * 64, 2) void ffn_product_kernel(const ProductArgs by_value) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int product = FIRST != 0 ? 0 : 1;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // the grid is the number of CUs that the schedule was made for
    const TileSchedule sch = *reinterpret_cast<const TileSchedule*>(by_value.lists + kScheduleAt + product * kScheduleInts);
    if (by_value.lists[1] > 0 && (by_value.kinds & kTiledUnits)) {         // block-uniform, as all of these
        int32_t* const parts = by_value.lists + kSplitCounter + product;
        int32_t* const joined = by_value.lists + kJoinedAt + product * kSplitSlots;
        const ProductArgs& p = by_value;
        // Big units first: their loop is the one that matters most, and its place in the code makes a difference (with the other
        // shapes in front of them the first product of 16384 tokens x 2048 x 8192, k = 2, took 888 us instead of 878).
        if (sch.shape == UnitShape::kBig)
            run_units<FIRST, FOLD, BigUnits>(p.act, p.rowmap, p.wpk, p.outp, p.big_tiles, sch, parts, joined, p.partials, p.N, p.K,
                                             p.act_kmajor, p.bias, p.fold, smem);
        else if (sch.shape == UnitShape::kFine)
            run_units<FIRST, FOLD, FineUnits>(p.act, p.rowmap, p.wpk, p.outp, p.half_tiles, sch, parts, joined, p.partials, p.N, p.K,
                                              p.act_kmajor, p.bias, p.fold, smem);
        else
            run_units<FIRST, FOLD, NarrowUnits>(p.act, p.rowmap, p.wpk, p.outp, p.big_tiles, sch, parts, joined, p.partials, p.N, p.K,
                                                p.act_kmajor, p.bias, p.fold, smem);
    }
    // From here on everything is read anew (the pointer is opaque to the compiler), so that nothing of it takes registers above.
    product_args_t args = (product_args_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    const int32_t* lists = args->lists;
    const int kinds = args->kinds;
    if (lists[0] <= 0 || !(kinds & kStreamUnits)) return;   // no small expert
    int busy = 0;                                           // blocks of an XCD that began with a tiled unit
    if (lists[1] > 0 && (kinds & kTiledUnits)) {
        const TileSchedule* s = reinterpret_cast<const TileSchedule*>(lists + kScheduleAt + product * kScheduleInts);
        busy = s->rounds > 0 ? static_cast<int>(gridDim.x) : s->R * s->split;
        if (gridDim.x % 8 == 0) busy = (busy + 7) >> 3;
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");       // the LDS changes hands
    if (wave >= 4) return;
    const FoldOut fold{args->fold.out, args->fold.tokmap, args->fold.gate};
    run_stream_units<KSPLIT, FIRST, FOLD>(args->act, args->rowmap, args->wpk, args->outp, args->small_tiles, lists[0],
                                          args->lists + kTakenAt + product * 8 * kTakenStride, busy, args->N, args->K, args->act_kmajor,
                                          args->bias, fold, smem, wave);
}

template <int KSPLIT, int FIRST, bool FOLD>
static hipError_t launch_product_kernel(const uint16_t* act, const int32_t* rowmap, const uint16_t* wpk, void* outp,
                                        const TileLists& lists, int N, int K, bool act_kmajor, const float* bias, const FoldOut& fold,
                                        int kinds, hipStream_t st) {
    // An uncut contraction is read from rows in LDS (pick_ksplit cuts the others).
    if (KSPLIT == 1 && stream_row_lds(64, K) > kStreamRowLdsMax) return hipErrorInvalidValue;
    const ProductArgs args{act, rowmap, wpk, outp, lists.small_tiles, lists.big_tiles, lists.half_tiles, lists.ntiles, lists.partials,
                           bias, fold, N, K, act_kmajor ? 1 : 0, kinds};
    // Always the whole chip, one block per CU (the LDS allows no more): how many units there are is only known on the device.
    hipLaunchKernelGGL((ffn_product_kernel<KSPLIT, FIRST, FOLD>), dim3(static_cast<unsigned>(tile_product_grid())), dim3(kWaves * 64),
                       kTileLds, st, args);
    return hipGetLastError();
}

int tile_product_grid() { return device_cu_count(); }

template <int KSPLIT, int FIRST, bool FOLD>
static hipError_t configure_product() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(ffn_product_kernel<KSPLIT, FIRST, FOLD>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, kTileLds);
}

template <int KSPLIT>
static hipError_t configure_products() {
    hipError_t e;
    if ((e = configure_product<KSPLIT, kFirstRelu, false>()) != hipSuccess) return e;
    if ((e = configure_product<KSPLIT, kFirstGelu, false>()) != hipSuccess) return e;
    if ((e = configure_product<KSPLIT, 0, false>()) != hipSuccess) return e;
    return configure_product<KSPLIT, 0, true>();
}

hipError_t configure_tile_kernels(int) {
    hipError_t e;
    if ((e = configure_products<1>()) != hipSuccess) return e;
    if ((e = configure_products<2>()) != hipSuccess) return e;
    return configure_products<4>();
}

template <int KSPLIT>
static hipError_t launch_product_split(bool first, const uint16_t* act, const int32_t* rowmap, const uint16_t* wpk, void* outp,
                                       const TileLists& lists, int N, int K, bool act_kmajor, int activation, const float* bias,
                                       const FoldOut& fold, int kinds, hipStream_t st) {
    if (first && activation == MOE_ACT_GELU)
        return launch_product_kernel<KSPLIT, kFirstGelu, false>(act, rowmap, wpk, outp, lists, N, K, act_kmajor, bias, fold, kinds, st);
    if (first)
        return launch_product_kernel<KSPLIT, kFirstRelu, false>(act, rowmap, wpk, outp, lists, N, K, act_kmajor, bias, fold, kinds, st);
    if (fold.out != nullptr)
        return launch_product_kernel<KSPLIT, 0, true>(act, rowmap, wpk, outp, lists, N, K, act_kmajor, bias, fold, kinds, st);
    return launch_product_kernel<KSPLIT, 0, false>(act, rowmap, wpk, outp, lists, N, K, act_kmajor, bias, fold, kinds, st);
}

hipError_t launch_tiled_product(bool first, int ksplit, const uint16_t* act, const int32_t* rowmap, const uint16_t* wpk,
                                void* outp, const TileLists& lists, int N, int K, bool act_kmajor, int activation,
                                const float* bias, const FoldOut& fold, int kinds, hipStream_t st) {
    if (ksplit == 4)
        return launch_product_split<4>(first, act, rowmap, wpk, outp, lists, N, K, act_kmajor, activation, bias, fold, kinds, st);
    if (ksplit == 2)
        return launch_product_split<2>(first, act, rowmap, wpk, outp, lists, N, K, act_kmajor, activation, bias, fold, kinds, st);
    return launch_product_split<1>(first, act, rowmap, wpk, outp, lists, N, K, act_kmajor, activation, bias, fold, kinds, st);
}

}  // namespace moe
