// LDS-tiled MFMA product for experts with many rows (the compute-bound "hot" experts of the
// paper's Section 3.3: enough tokens per expert that the product is bound by matrix throughput,
// not by reading the expert's parameters):
//
//   out[row, n] = sum_k act[row, k] * W_e[n, k]          (FIRST: relu, rounded to bf16)
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
// from the device-built list of large-expert row tiles.
#include <type_traits>

#include "tile_schedule.hpp"

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

template <int FIRST, typename Units>
__device__ __forceinline__ void run_units(const uint16_t* __restrict__ act, const int32_t* __restrict__ rowmap,
                                          const uint16_t* __restrict__ wpk, void* __restrict__ outp,
                                          const Tile* __restrict__ tiles, const TileSchedule& sch,
                                          int32_t* __restrict__ part_counter, float* __restrict__ partials, int N, int K,
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

        // Lane holds 4 consecutive columns of one row per accumulator.
        if (cur.nparts > 1) {
            // part of a unit: the partial tile goes to the workspace; the next kernel adds the parts up
            float* mine = partials + (static_cast<size_t>(cur.u - sch.rounds * G) * cur.nparts + cur.part) * (kTM * kTN);
#pragma unroll
            for (int tf = 0; tf < OF; ++tf)
#pragma unroll
                for (int nf = 0; nf < 4; ++nf)
                    *reinterpret_cast<f32x4*>(mine + (lr0 + tf * 16 + r) * kTN + (wn * 4 + nf) * 16 + g * 4) =
                        acc[nf][tf];
        } else {
            const float* be = bias ? bias + static_cast<size_t>(cur.tl.expert) * N : nullptr;
#pragma unroll
            for (int tf = 0; tf < OF; ++tf) {
                if (lr0 + tf * 16 >= cur.tl.rows) break;     // wave-uniform: no row from here on
                const int lr = lr0 + tf * 16 + r;
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
                    int ftok = 0;
                    float fw = 0.f;
                    if (fold.out != nullptr && ok) {                    // folded layer output (top-1, no mask)
                        ftok = fold.tokmap[cur.tl.row0 + lr];
                        fw = fold.gate[ftok];
                    }
                    if (fold.out != nullptr) {                          // block-uniform
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
                                store_out<0>(outp, cur.tl.row0 + lr, nb * 16 + g * 4, N, be, acc[nf][tf]);
                        }
                    }
                }
            }
        }
        cur = nxt;
    }
}

template <int FIRST>
__global__ __launch_bounds__(kWaves * 64, 2) void ffn_tile_kernel(const uint16_t* __restrict__ act, const int32_t* __restrict__ rowmap,
                                                                  const uint16_t* __restrict__ wpk, void* __restrict__ outp,
                                                                  const Tile* __restrict__ big_tiles,
                                                                  const Tile* __restrict__ half_tiles,
                                                                  const int32_t* __restrict__ ntiles_p,
                                                                  int32_t* __restrict__ part_counter,
                                                                  float* __restrict__ partials, int N, int K, int act_kmajor,
                                                                  const float* __restrict__ bias, const FoldOut fold) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    // the grid is the number of CUs that the schedule was made for
    const TileSchedule sch = *reinterpret_cast<const TileSchedule*>(ntiles_p + kScheduleAt + (FIRST != 0 ? 0 : kScheduleInts));
    if (ntiles_p[1] <= 0) return;                       // no large expert in this call (block-uniform)
    // Big units first: their loop is the one that matters most, and its place in the code makes a difference (with the other shapes
    // in front of them the first product of 16384 tokens x 2048 x 8192, k = 2, took 888 us instead of 878).
    if (sch.shape == UnitShape::kBig)
        run_units<FIRST, BigUnits>(act, rowmap, wpk, outp, big_tiles, sch, part_counter, partials, N, K, act_kmajor, bias, fold,
                                   smem);
    else if (sch.shape == UnitShape::kFine)
        run_units<FIRST, FineUnits>(act, rowmap, wpk, outp, half_tiles, sch, part_counter, partials, N, K, act_kmajor, bias, fold,
                                    smem);
    else
        run_units<FIRST, NarrowUnits>(act, rowmap, wpk, outp, big_tiles, sch, part_counter, partials, N, K, act_kmajor, bias, fold,
                                      smem);
}

template <int FIRST>
static hipError_t launch_tile(const uint16_t* act, const int32_t* rowmap, const uint16_t* wpk, void* outp,
                              const TileLists& lists, int N, int K, bool act_kmajor, const float* bias, const FoldOut& fold,
                              hipStream_t st) {
    // Always the whole chip, one block per CU (the LDS allows no more): how many units there are is
    // only known on the device, and few units are cut along K over blocks that would otherwise idle.
    hipLaunchKernelGGL(ffn_tile_kernel<FIRST>, dim3(static_cast<unsigned>(tile_product_grid())), dim3(kWaves * 64), kTileLds, st,
                       act, rowmap, wpk, outp, lists.big_tiles, lists.half_tiles, lists.ntiles,
                       lists.ntiles + kSplitCounter + (FIRST != 0 ? 0 : 1), lists.partials, N, K, act_kmajor ? 1 : 0, bias, fold);
    return hipGetLastError();
}

int tile_product_grid() { return device_cu_count(); }

template <int FIRST>
static hipError_t configure_tile() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(ffn_tile_kernel<FIRST>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, kTileLds);
}

hipError_t configure_tile_kernels(int) {
    hipError_t e;
    if ((e = configure_tile<0>()) != hipSuccess) return e;
    if ((e = configure_tile<kFirstRelu>()) != hipSuccess) return e;
    return configure_tile<kFirstGelu>();
}

hipError_t launch_tile_product(bool first, const uint16_t* act, const int32_t* rowmap, const uint16_t* wpk,
                               void* outp, const TileLists& lists, int N, int K, bool act_kmajor, int activation,
                               const float* bias, const FoldOut& fold, hipStream_t st) {
    if (!first) return launch_tile<0>(act, rowmap, wpk, outp, lists, N, K, act_kmajor, bias, fold, st);
    if (activation == MOE_ACT_GELU)
        return launch_tile<kFirstGelu>(act, rowmap, wpk, outp, lists, N, K, act_kmajor, bias, fold, st);
    return launch_tile<kFirstRelu>(act, rowmap, wpk, outp, lists, N, K, act_kmajor, bias, fold, st);
}

}  // namespace moe
