// Expert FFN products of fp32 layers on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32: fp32 operands, fp32
// accumulation, nothing rounded in between):
//
//   out[row, n] = sum_k act[row, k] * W_e[n, k]          (FIRST: bias and activation, else bias)
//
// Weights are plain rows [N][K].  A unit is one row tile (up to 64 rows of one expert) x 16 columns; the four
// wavefronts of a block split the contraction and add their partial sums in LDS in a fixed order.  Per 32 k a wavefront
// loads one 128-byte line of each of its rows, eight consecutive lanes a line, turns the fragments round in its own part
// of LDS, and reads them back as matrix operands: lane (r, g) holds k0 + 4g ... + 3 of row r and feeds element j to the
// j-th of four MFMAs (the four k of one MFMA are k0 + j + {0, 4, 8, 12}, the same for both operands).  Loading the
// operands straight into that form puts 16 different rows under 16 consecutive lanes: 64 cache accesses per load
// instruction instead of 16, which bounded the kernel (57 + 67 us on the layer below).
//
// Rounding: a result is no further from the exact sum than with four interleaved sums over k mod 4, added in pairs.  Four
// about equal shares of a contraction are as good as those.  Where they are not (K below 128, or a few hundred and no multiple
// of 128), a wavefront's MFMAs take turns in two chains of sums, and in four, one per k mod 4, where the contraction is too
// short for a step per wavefront (the weights of such units are few, so tiles of more than 32 rows read them twice).  Relative
// error of a layer's two products, mean of 24 layers of random inputs, one chain per wavefront throughout -> these: d = 20,
// f = 33: 1.12 -> 0.82e-7; d = 32: 1.35 -> 1.08e-7; d = 64: 1.54 -> 1.32e-7; d = 96: 1.71 -> 1.51e-7 (four interleaved sums:
// 0.96, 1.07, 1.38 and 1.64e-7).  Further chains cost registers: layers of 300 tokens, 8 experts, 96 x 384 22.6 -> 23.3 us;
// 500 tokens, 258 x 1032, would take 41.3 -> 44.0 us and stay with one at the error they have.
//
// What bounds it: with about 64 rows per expert the MFMA time (64 flop per clock and SIMD) and reading the weights once
// are about equal, 17 and 14 us on a layer of 500 tokens, 8 experts, 768 x 3072, one expert per token (2.4 GFLOP and
// 75 MB of weights per product); the rest is the start of the units (tile, row numbers, first lines: three dependent
// trips to memory) and the last round.  Measured there: 47 + 46 us for the two products; a thread per column with
// fused multiply-adds took 1353 + 2432 us.  Units of 32 columns with operands through registers like these needed fewer row loads but
// left room for two blocks per CU only: 48 + 63 us.  Copied straight into LDS (ffn_f32_wide_kernel) they take 39.0 us where there are several
// for every CU, as in the first product; the second has too few of them (60.9 us) and stays with units of 16.
#include <algorithm>
#include <type_traits>

#include "common.hpp"

namespace moe {

constexpr int kF32Waves = 4;        // wavefronts of a block: slices of the contraction
constexpr int kF32Step = 32;        // k per step: one 128-byte line of every row
constexpr int kF32FragFloats = 16 * kF32Step;

// A wavefront's first step: shares differ by one step at most, and the last wavefront, which also takes the rest of the row,
// has one of the smaller ones.
__host__ __device__ __forceinline__ int f32_first_step(int steps, int wave) {
    const int q = steps / kF32Waves, r = steps % kF32Waves;
    return wave * q + (wave < r ? wave : r);
}

// 16-byte piece p (of 8) of row r of a fragment in LDS.  The pieces of a row are permuted by its row number: the eight
// rows that a read touches at once then lie in different banks.
__device__ __forceinline__ int f32_slot(int r, int p) { return r * kF32Step + ((p ^ (r & 7)) << 2); }

// A second product's output: rows of y, the layer output itself (FoldOut), or either as the launch says.  The last takes a register for
// the token's number: with two chains 18 spilled instead of 13 (layers of 2000 tokens, 16 experts, k = 2, 320 x 288 57.9 -> 59.1 us), so
// only kernels of one chain, which have one to spare, leave it to the launch (500 tokens, 8 experts, k = 2, 768 x 3072: 156.8 us so,
// 158.9 as a kernel for rows of y alone).
enum F32Fold { kF32Rows, kF32Folded, kF32Either };

// CHAINS: accumulators per output, taken in turn by the four MFMAs of 16 k
template <int TFC, int CHAINS, int VEC, bool FIRST, int FOLD>
__device__ __forceinline__ void f32_unit(const float* __restrict__ act, const int32_t* __restrict__ rowmap,
                                         const float* __restrict__ w, float* __restrict__ outp, const Tile tl,
                                         const int n0, const int N, const int K, const int activation,
                                         const float* __restrict__ bias, const FoldOut& fold, float* lds) {
    constexpr int F = 1 + TFC;                            // fragments per step: the 16 weight rows, the token rows
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    // loads: half a fragment (8 rows x 128 bytes) per instruction, 8 consecutive lanes a row
    const int lrow = lane >> 3, lpiece = lane & 7;
    const float* src[F][2];
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int fr = h * 8 + lrow;
            if (i == 0) {
                src[i][h] = w + (static_cast<size_t>(tl.expert) * N + min(n0 + fr, N - 1)) * K + lpiece * 4;
            } else {
                int row = tl.row0 + min((i - 1) * 16 + fr, tl.rows - 1);
                if (rowmap != nullptr) row = rowmap[row];
                src[i][h] = act + static_cast<size_t>(row) * K + lpiece * 4;
            }
        }
    // A folded output: the token of the row that this lane stores, looked up here and its gate weight at the end of the contraction, so
    // that neither is waited for.  Whole layers, us, with combine -> this: 500 tokens, 8 experts, 768 x 3072
    // 100.2 -> 95.5; 300 tokens, 8 experts, 256 x 1024 29.4 -> 25.2; 16 tokens, 4 experts, 64 x 256 21.2 -> 16.6.
    static_assert(!FIRST || FOLD == kF32Rows, "second products only");
    const bool folded = FOLD == kF32Folded || (FOLD == kF32Either && fold.out != nullptr);
    constexpr bool EARLY = FIRST || CHAINS == 1 || FOLD != kF32Rows;      // the row's number: a register during the contraction
    int orow = EARLY ? tl.row0 + min(wave * 16 + r, tl.rows - 1) : 0;
    if (FOLD != kF32Rows && folded) orow = fold.tokmap[orow];
    f32x4 acc[CHAINS][TFC];
#pragma unroll
    for (int c = 0; c < CHAINS; ++c)
#pragma unroll
        for (int tf = 0; tf < TFC; ++tf) acc[c][tf] = f32x4{0.f, 0.f, 0.f, 0.f};
    float* mine = lds + wave * (F * kF32FragFloats);      // private to the wavefront: its LDS accesses stay in order
    f32x4 raw[F][2];
    auto issue = [&]() {                                  // loads a step and moves on to the next
#pragma unroll
        for (int i = 0; i < F; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                raw[i][h] = load_k4<VEC>(src[i][h]);
                src[i][h] += kF32Step;
            }
    };
    auto to_lds = [&]() {
#pragma unroll
        for (int i = 0; i < F; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                *reinterpret_cast<f32x4*>(mine + i * kF32FragFloats + f32_slot(h * 8 + lrow, lpiece)) = raw[i][h];
    };
    auto fma = [&]() {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            f32x4 v[F];
#pragma unroll
            for (int i = 0; i < F; ++i) v[i] = *reinterpret_cast<const f32x4*>(mine + i * kF32FragFloats + f32_slot(r, q * 4 + g));
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int tf = 0; tf < TFC; ++tf)
                    acc[j % CHAINS][tf] =
                        __builtin_amdgcn_mfma_f32_16x16x4f32(v[0][j], v[1 + tf][j], acc[j % CHAINS][tf], 0, 0, 0);
        }
    };
    const int steps = K / kF32Step;                       // whole steps; the rest of the row below
    const int s0 = f32_first_step(steps, wave), s1 = f32_first_step(steps, wave + 1);
    auto start_at = [&](int step) {
#pragma unroll
        for (int i = 0; i < F; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) src[i][h] += step * kF32Step;
    };
    if (s0 < s1) {
        start_at(s0);
        issue();
        for (int s = s0; s < s1; ++s) {
            to_lds();
            // the next step's loads go out before this step's MFMAs (the compiler would move them behind)
            __builtin_amdgcn_sched_barrier(0);
            if (s + 1 < s1) issue();
            __builtin_amdgcn_sched_barrier(0);
            fma();
        }
        start_at(-s1);
    }
    if (K % kF32Step != 0 && wave == kF32Waves - 1) {     // wave-uniform
        const int left = K % kF32Step - lpiece * 4;
#pragma unroll
        for (int i = 0; i < F; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) raw[i][h] = load_k4_tail(src[i][h] + steps * kF32Step, left);
        to_lds();
        fma();
    }
    float gate = 1.f;
    if (FOLD != kF32Rows && folded) gate = fold.gate[orow];
    f32x4* red = reinterpret_cast<f32x4*>(lds);
    __syncthreads();                                      // the operands in LDS give way to the partial sums

    // row fragment i of every wavefront at red[(wave * TFC + i) * 64 + lane]; wavefront i adds and stores it
#pragma unroll
    for (int tf = 0; tf < TFC; ++tf) {
        f32x4 sum = acc[0][tf];
        if constexpr (CHAINS >= 2) sum += acc[1][tf];
        if constexpr (CHAINS == 4) sum += acc[2][tf] + acc[3][tf];
        red[(wave * TFC + tf) * 64 + lane] = sum;
    }
    __syncthreads();
    if (wave < TFC) {
        const int lr = wave * 16 + r, n = n0 + g * 4;
        static_assert(kF32Waves == 4, "partial sums are added in pairs");
        const f32x4* part = red + wave * 64 + lane;
        f32x4 v = (part[0] + part[TFC * 64]) + (part[2 * TFC * 64] + part[3 * TFC * 64]);
        if (lr < tl.rows) {
            float* o = outp + static_cast<size_t>(EARLY ? orow : tl.row0 + lr) * N + n;
            const float* be = bias ? bias + static_cast<size_t>(tl.expert) * N + n : nullptr;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (n + q < N && be != nullptr) v[q] += be[q];
                if (FIRST) v[q] = activate(v[q], activation);
                if (folded) v[q] = fmaf(gate, v[q], 0.f);     // what combine_kernel computes
            }
            if (VEC == 4 && (N & 3) == 0) {               // out rows are then 16-byte aligned (see launch_f32_product)
                if (n < N) *reinterpret_cast<f32x4*>(o) = v;
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (n + q < N) o[q] = v[q];
            }
        }
    }
    __syncthreads();                                      // LDS may be reused
}

// The same product for layers of many rows per expert, where reading the token rows again for every 16 columns bounds the units above
// (64 rows: 40 bytes per clock and CU at the full matrix rate, which is what a CU can pull from its L2).  A unit is one row tile x 32
// columns: two groups of two wavefronts take half of the contraction each, through rings of their own in LDS, and a wavefront of a group
// 16 columns; the rows of a step are in LDS once for both.  Everything is copied straight into LDS a line per eight lanes, in the
// layout that f32_slot describes: 12 KiB per 32 k and group, 24 bytes per clock and CU.  Two blocks fit a CU; blocks are one unit long, and
// the hardware hands them out as CUs fall free.  (With a ring of two stages, three blocks to a CU: 39 -> 43 us on the layer below.)
// Rounding: four chains of sums per half, eight in all, no further from 64 bits than those above (two chains per half were, where those
// have eight: 288 x 1152 2.5 -> 2.7e-7; with four 2.5e-7).
// Rows and columns past the end are copies of the last one and not stored.  K a multiple of 32, everything 16-byte aligned.
constexpr int kWideStages = 3, kWideCols = 32;
template <int TFC>
constexpr int wide_stage_bytes() { return (2 + TFC) * kF32FragFloats * 4; }              // of a group

template <int TFC, bool FIRST, bool FOLDED>
__device__ __forceinline__ void f32_wide_unit(const float* __restrict__ act, const int32_t* __restrict__ rowmap,
                                              const float* __restrict__ w, float* __restrict__ outp, const Tile tl, const int n0,
                                              const int N, const int K, const int activation, const float* __restrict__ bias,
                                              const FoldOut& fold, float* lds) {
    constexpr int kFrags = 2 + TFC, kCopies = 2 * kFrags / 2;      // fragments of a stage; 1-KiB copies of a stage per wavefront of the group
    constexpr int kStage = wide_stage_bytes<TFC>();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const int group = wave >> 1, col = wave & 1;
    const int lrow = lane >> 3, piece = ((lane & 7) ^ lrow) * 4;   // copies: 8 rows x 128 bytes; the row's piece that belongs at the lane's slot
    const int steps = K / kF32Step, half = (steps + 1) >> 1;
    const int s0 = group ? half : 0, n = group ? steps - half : half;
    unsigned char* const ring = reinterpret_cast<unsigned char*>(lds) + group * (kWideStages * kStage);
    const uint32_t ring_at = lds_address(ring);
    // Copy c of the group: half c % 2 of fragment c / 2 (0, 1: weights of the two column blocks); wavefront `col` does c = 2 q + col.
    const float* src[kCopies];
#pragma unroll
    for (int q = 0; q < kCopies; ++q) {
        const int fr = col * 8 + lrow;                     // row of the fragment
        if (q < 2) {
            src[q] = w + (static_cast<size_t>(tl.expert) * N + min(n0 + q * 16 + fr, N - 1)) * K + s0 * kF32Step + piece;
        } else {
            int row = tl.row0 + min((q - 2) * 16 + fr, tl.rows - 1);
            if (rowmap != nullptr) row = rowmap[row];
            src[q] = act + static_cast<size_t>(row) * K + s0 * kF32Step + piece;
        }
    }
    auto copy_stage = [&](int slot) {
#pragma unroll
        for (int q = 0; q < kCopies; ++q) {
            copy16_to_lds(src[q], ring_at + slot * kStage + (2 * q + col) * 1024);
            src[q] += kF32Step;
        }
    };
    f32x4 acc[4][TFC];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int tf = 0; tf < TFC; ++tf) acc[c][tf] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < kWideStages - 1; ++s)
        if (s < n) copy_stage(s);
    int slot = 0;
    for (int s = 0; s < half; ++s) {                       // the second group may have a step less: it only meets the barriers then
        // own copies of step s have landed (those of one later step may be under way), then everybody's
        if (s + 1 < n) __builtin_amdgcn_s_waitcnt(0x0F70 + kCopies);
        else __builtin_amdgcn_s_waitcnt(0x0F70);
        asm volatile("s_barrier" ::: "memory");            // also: step s - 1 has been read by all, its slot is free
        const int free_slot = slot == 0 ? kWideStages - 1 : slot - 1;
        if (s + kWideStages - 1 < n) copy_stage(free_slot);
        if (s < n) {
            const float* st = reinterpret_cast<const float*>(ring + slot * kStage);
            f32x4 wv[2], xv[2][TFC];                       // all reads at once: the second half's are covered by the first half's MFMAs
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int at = f32_slot(r, q * 4 + g);
                wv[q] = *reinterpret_cast<const f32x4*>(st + col * kF32FragFloats + at);
#pragma unroll
                for (int tf = 0; tf < TFC; ++tf) xv[q][tf] = *reinterpret_cast<const f32x4*>(st + (2 + tf) * kF32FragFloats + at);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int tf = 0; tf < TFC; ++tf)
                        acc[j][tf] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[q][j], xv[q][tf][j], acc[j][tf], 0, 0, 0);
            // the reads of this step are done before the next barrier lets its slot be filled
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
        slot = slot + 1 == kWideStages ? 0 : slot + 1;
    }
    __syncthreads();                                       // the operands in LDS give way to the partial sums
    // of its columns, the first group keeps the even row fragments and the second the odd ones
    f32x4* const red = reinterpret_cast<f32x4*>(lds);
#pragma unroll
    for (int tf = 0; tf < TFC; ++tf) {
        acc[0][tf] = (acc[0][tf] + acc[1][tf]) + (acc[2][tf] + acc[3][tf]);
        if ((tf & 1) != group) red[(col * TFC + tf) * 64 + lane] = acc[0][tf];
    }
    __syncthreads();
    const int n1 = n0 + col * 16 + g * 4;
    const float* be = bias ? bias + static_cast<size_t>(tl.expert) * N + n1 : nullptr;
#pragma unroll
    for (int tf = 0; tf < TFC; ++tf) {
        const int lr = tf * 16 + r;
        if ((tf & 1) != group || lr >= tl.rows || n1 >= N) continue;
        const f32x4 other = red[(col * TFC + tf) * 64 + lane];
        f32x4 v = group == 0 ? acc[0][tf] + other : other + acc[0][tf];
        if (be != nullptr) v += *reinterpret_cast<const f32x4*>(be);
        int orow = tl.row0 + lr;
        float gate = 1.f;
        if (FOLDED) {
            orow = fold.tokmap[orow];
            gate = fold.gate[orow];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (FIRST) v[q] = activate(v[q], activation);
            if (FOLDED) v[q] = fmaf(gate, v[q], 0.f);      // what combine_kernel computes
        }
        *reinterpret_cast<f32x4*>(outp + static_cast<size_t>(orow) * N + n1) = v;
    }
}

template <bool FIRST, bool FOLDED>
__global__ __launch_bounds__(256, 2) void ffn_f32_wide_kernel(const float* __restrict__ act, const int32_t* __restrict__ rowmap,
                                                              const float* __restrict__ w, float* __restrict__ outp,
                                                              const Tile* __restrict__ tiles, const int32_t* __restrict__ ntiles_p,
                                                              int N, int K, int activation, const float* __restrict__ bias,
                                                              const FoldOut fold) {
    extern __shared__ __attribute__((aligned(16))) float wide_lds[];
    // Block b of an XCD (b % 8) takes a unit of its eighth of the column groups, as in ffn_f32_kernel: each weight enters one L2 only.
    const int per = ((N + kWideCols - 1) / kWideCols + 7) / 8, u = static_cast<int>(blockIdx.x >> 3);
    const int cg = static_cast<int>(blockIdx.x & 7) * per + u % per, tile = u / per;
    if (tile >= ntiles_p[0] || cg * kWideCols >= N) return;
    const Tile tl = tiles[tile];
    const int n0 = cg * kWideCols;
    switch ((tl.rows + 15) >> 4) {
        case 1: f32_wide_unit<1, FIRST, FOLDED>(act, rowmap, w, outp, tl, n0, N, K, activation, bias, fold, wide_lds); break;
        case 2: f32_wide_unit<2, FIRST, FOLDED>(act, rowmap, w, outp, tl, n0, N, K, activation, bias, fold, wide_lds); break;
        case 3: f32_wide_unit<3, FIRST, FOLDED>(act, rowmap, w, outp, tl, n0, N, K, activation, bias, fold, wide_lds); break;
        default: f32_wide_unit<4, FIRST, FOLDED>(act, rowmap, w, outp, tl, n0, N, K, activation, bias, fold, wide_lds); break;
    }
}
constexpr int kWideLds = 2 * kWideStages * wide_stage_bytes<4>();
static_assert(2 * kWideLds <= static_cast<int>(kLdsPerCu), "two blocks to a CU");

// SORT: the first product of a small layer, whose blocks sort the assignments by expert themselves: such a layer is a chain of short
// kernels, each at its launch, and a dispatch step of its own does nothing but that.  Every block reads the tokens' experts (at
// most kF32SortMax, 4 per thread), ranks them among those of its 64 that name the same expert with one ballot per bit of the
// expert's number, and adds up the groups' histograms; block 0 also writes what the dispatch step would.  The order is the same.
// Whole layers, us, with a dispatch step -> this: 64 tokens, 64 x 256, 8 experts, k = 2 21.1 -> 17.9; 16 tokens, 64 x 256, 4 experts
// 16.6 -> 13.4; 300 tokens, 96 x 384, 8 experts 21.1 -> 17.7; 300 tokens, 256 x 1024, 8 experts 25.2 -> 22.3; 30 tokens, 768 x 3072,
// 4 experts 32.6 -> 29.2.
constexpr int kF32SortMax = 1024, kF32SortExperts = 64, kF32TileRows = 64;
constexpr int kF32SortTiles = kF32SortMax / kF32TileRows + kF32SortExperts;
struct F32Sort {
    const int32_t* idx;
    int32_t* counts;
    int32_t* offsets;
    int32_t* perm;             // may be NULL
    int32_t* inv_perm;
    int32_t* tokmap;
    Tile* tiles;
    int32_t* ntiles;
    int A, E, k;
};
struct F32Lists {
    Tile tiles[kF32SortTiles];
    int32_t token[kF32SortMax];
    int32_t hist[kF32SortMax / 64][kF32SortExperts];         // of 64 assignments each; then their first places
    int32_t ntiles;
};

__device__ __forceinline__ void f32_sort(const F32Sort& p, F32Lists& l) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int A = p.A, E = p.E, groups = (A + 63) >> 6;
    int ex[4], rank[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {                          // group c * 4 + wave
        const int a = c * 256 + static_cast<int>(threadIdx.x);
        ex[c] = a < A ? min(max(p.idx[a], 0), E - 1) : 0;
    }
    for (int i = threadIdx.x; i < groups * kF32SortExperts; i += 256) l.hist[i / kF32SortExperts][i % kF32SortExperts] = 0;
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int grp = c * 4 + wave;
        if (grp >= groups) break;                          // wave-uniform
        uint64_t same = __ballot(grp * 64 + lane < A);
        for (int bit = 1; bit < E; bit <<= 1) {
            const bool mine = (ex[c] & bit) != 0;
            const uint64_t set = __ballot(mine);
            same &= mine ? set : ~set;
        }
        rank[c] = __popcll(same & ((1ull << lane) - 1));
        if (rank[c] == 0 && grp * 64 + lane < A) l.hist[grp][ex[c]] = __popcll(same);
    }
    __syncthreads();
    if (wave == 0) {                                       // lane: expert
        int count = 0;
        for (int q = 0; q < groups; ++q) count += l.hist[q][lane];          // zero from E on
        const int mine = (count + kF32TileRows - 1) / kF32TileRows;
        int row = count, tile = mine;                      // inclusive prefix sums
#pragma unroll
        for (int n = 1; n < 64; n <<= 1) {
            const int r = __shfl_up(row, n), t = __shfl_up(tile, n);
            if (lane >= n) {
                row += r;
                tile += t;
            }
        }
        if (lane == 63) l.ntiles = tile;
        tile -= mine;
        row -= count;
        for (int i = 0; i < mine; ++i)
            l.tiles[tile + i] = Tile{lane, row + i * kF32TileRows, min(kF32TileRows, count - i * kF32TileRows), 0};
        if (blockIdx.x == 0) {
            if (lane < E) {
                p.counts[lane] = count;
                p.offsets[lane] = row;
            }
            if (lane == 0) p.offsets[E] = A;
        }
        for (int q = 0; q < groups; ++q) {
            const int n = l.hist[q][lane];
            l.hist[q][lane] = row;
            row += n;
        }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int a = c * 256 + static_cast<int>(threadIdx.x);
        if (a >= A) break;
        const int at = l.hist[a >> 6][ex[c]] + rank[c], t = a / p.k;
        l.token[at] = t;
        if (blockIdx.x == 0) {
            if (p.perm != nullptr) p.perm[at] = a;
            p.inv_perm[a] = at;
            p.tokmap[at] = t;
        }
    }
    __syncthreads();
    if (blockIdx.x == 0) {                                 // for the second product
        if (threadIdx.x == 0) p.ntiles[0] = l.ntiles;
        if (static_cast<int>(threadIdx.x) < l.ntiles) p.tiles[threadIdx.x] = l.tiles[threadIdx.x];
    }
}
static_assert(kF32SortTiles <= 256, "a thread per tile");

// At least 4 wavefronts per SIMD: the turn through LDS and the start of a unit are covered by the other blocks' MFMAs.  3 with the
// lists of SORT in LDS.
struct F32NoSort {};
template <int VEC, bool FIRST, int CHAINS, bool SORT, int FOLD>
__global__ __launch_bounds__(256, SORT ? 3 : 4) void ffn_f32_kernel(const float* __restrict__ act,
                                                                 const int32_t* __restrict__ rowmap,
                                                                 const float* __restrict__ w, float* __restrict__ outp,
                                                                 const Tile* __restrict__ tiles,
                                                                 const int32_t* __restrict__ ntiles_p, int N, int K,
                                                                 int activation, const float* __restrict__ bias,
                                                                 const FoldOut fold,
                                                                 const std::conditional_t<SORT, F32Sort, F32NoSort> sort) {
    __shared__ __attribute__((aligned(16))) float lds[kF32Waves * 5 * kF32FragFloats];
    if constexpr (SORT) {
        __shared__ F32Lists lists;
        f32_sort(sort, lists);
        tiles = lists.tiles;
        rowmap = lists.token;
        ntiles_p = &lists.ntiles;
    }
    const auto uniform = [](int v) { return SORT ? __builtin_amdgcn_readfirstlane(v) : v; };      // loads from LDS look divergent
    const int ngroups = (N + 15) / 16;
    // Blocks go to the 8 XCDs round-robin, and each XCD has its own L2.  XCD x takes the x-th eighth of the column groups
    // of every tile: each weight enters one L2 only, and the XCDs have equal work whatever the tiles' row counts are.
    // (With runs of whole tiles per XCD the last, partly filled round of units sat on one or two XCDs.)
    const bool sliced = gridDim.x % 8 == 0 && ngroups >= 8;
    const int x = sliced ? static_cast<int>(blockIdx.x & 7) : 0, nx = sliced ? 8 : 1;
    const int g0 = ngroups * x / nx, ng = ngroups * (x + 1) / nx - g0;
    const int units = uniform(ntiles_p[0]) * ng, stride = static_cast<int>(gridDim.x) / nx;
    for (int u = static_cast<int>(blockIdx.x) / nx; u < units; u += stride) {     // block-uniform
        Tile tl = tiles[u / ng];
        if constexpr (SORT) tl = Tile{uniform(tl.expert), uniform(tl.row0), uniform(tl.rows), 0};
        const int n0 = (g0 + u % ng) * 16;
        if constexpr (CHAINS < 4) {
            switch ((tl.rows + 15) >> 4) {                // exact number of row fragments: a fixed number of loads per step
                case 1: f32_unit<1, CHAINS, VEC, FIRST, FOLD>(act, rowmap, w, outp, tl, n0, N, K, activation, bias, fold, lds); break;
                case 2: f32_unit<2, CHAINS, VEC, FIRST, FOLD>(act, rowmap, w, outp, tl, n0, N, K, activation, bias, fold, lds); break;
                case 3: f32_unit<3, CHAINS, VEC, FIRST, FOLD>(act, rowmap, w, outp, tl, n0, N, K, activation, bias, fold, lds); break;
                default: f32_unit<4, CHAINS, VEC, FIRST, FOLD>(act, rowmap, w, outp, tl, n0, N, K, activation, bias, fold, lds); break;
            }
        } else {                                          // four chains of more than two fragments do not fit the registers
            for (int r0 = 0; r0 < tl.rows; r0 += 32) {
                const Tile part{tl.expert, tl.row0 + r0, min(32, tl.rows - r0), 0};
                if (part.rows <= 16)
                    f32_unit<1, CHAINS, VEC, FIRST, FOLD>(act, rowmap, w, outp, part, n0, N, K, activation, bias, fold, lds);
                else
                    f32_unit<2, CHAINS, VEC, FIRST, FOLD>(act, rowmap, w, outp, part, n0, N, K, activation, bias, fold, lds);
            }
        }
    }
}

// CHAINS of a contraction of length K.  Rounding errors of a sum grow with the square of its length: one chain per wavefront
// where the squares of the shares are within 2 % of those of four quarters (1 % in the error itself).
static int f32_chains(int K) {
    long squares = 0;
    for (int w = 0; w < kF32Waves; ++w) {
        const long n = static_cast<long>(f32_first_step(K / kF32Step, w + 1) - f32_first_step(K / kF32Step, w)) * kF32Step +
                       (w == kF32Waves - 1 ? K % kF32Step : 0);
        squares += n * n;
    }
    if (squares * 4 * 100 <= static_cast<long>(K) * K * 102) return 1;
    return K < kF32Waves * kF32Step ? 4 : 2;
}

// the widest load that every row's start allows
static int f32_width(int K, const void* act, const void* w, const void* outp) {
    const uintptr_t bases = reinterpret_cast<uintptr_t>(act) | reinterpret_cast<uintptr_t>(w) | reinterpret_cast<uintptr_t>(outp);
    return K % 4 == 0 && bases % 16 == 0 ? 4 : K % 2 == 0 && bases % 8 == 0 ? 2 : 1;
}

template <int VEC, bool FIRST>
static auto f32_kernel(int K, bool folded) {
    constexpr int kEither = FIRST ? kF32Rows : kF32Either, kFolded = FIRST ? kF32Rows : kF32Folded;
    const int chains = f32_chains(K);
    if (chains == 1) return ffn_f32_kernel<VEC, FIRST, 1, false, kEither>;
    if (chains == 4) return folded ? ffn_f32_kernel<VEC, FIRST, 4, false, kFolded> : ffn_f32_kernel<VEC, FIRST, 4, false, kF32Rows>;
    return folded ? ffn_f32_kernel<VEC, FIRST, 2, false, kFolded> : ffn_f32_kernel<VEC, FIRST, 2, false, kF32Rows>;
}

template <int VEC>
static hipError_t launch_f32(bool first, unsigned grid, const float* act, const int32_t* rowmap, const float* w,
                             float* outp, const Tile* tiles, const int32_t* ntiles, int N, int K, int activation,
                             const float* bias, const FoldOut& fold, hipStream_t st) {
    auto kern = first ? f32_kernel<VEC, true>(K, false) : f32_kernel<VEC, false>(K, fold.out != nullptr);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(256), 0, st, act, rowmap, w, outp, tiles, ntiles, N, K, activation, bias, fold,
                       F32NoSort{});
    return hipGetLastError();
}

// Units of at most `max_tiles` row tiles in a grid that runs them at once: each XCD's eighth of the column groups is rounded up (a grid
// for the plain number of units left a few blocks of some XCDs a second one: 29 groups of 8 tiles, a layer of 20 tokens,
// 464 x 1312, k = 2, 37.1 -> 27.8 us (31.0 with a dispatch step); 500 tokens, 288 x 1152, k = 2, 56.4 -> 50.8).
static long f32_units(long max_tiles, int N) {
    const long ngroups = (N + 15) / 16;
    return ngroups >= 8 ? max_tiles * ((ngroups + 7) / 8) * 8 : (max_tiles * ngroups + 7) / 8 * 8;
}

// Blocks of a product in wide units: one for each, every XCD's eighth of the column groups rounded up.
static long f32_wide_blocks(long max_tiles, int N) { return max_tiles * (((N + kWideCols - 1) / kWideCols + 7) / 8) * 8; }

// Where the wide units are ahead: rows enough per tile to share, and three units for every CU, because a CU with one is bound by the
// latency of its copies.  us, units above -> wide: 500 tokens, 8 experts, 768 x 3072, first product 45.4 -> 39.0 (1440 units at
// most), second 46.0 -> 60.9 (360: not taken); 155 tokens, 14 experts, 544 x 2048 (10 rows per tile: not taken) 42.3 -> 47.4 for the layer;
// 376 tokens, 14 experts, k = 2, 288 x 1024 43.2 -> 41.0.  A launch holds fewer than 2^32 threads: products of more units run in those
// above, whose blocks walk through them.
constexpr long kWideMinRows = 24, kWideMinUnits = 3, kWideThreads = 256, kWideMaxBlocks = 0xffffffffL / kWideThreads;
bool f32_is_wide(long rows, long max_tiles, int N, int K, const void* act, const void* w, const void* outp, const float* bias) {
    const uintptr_t bases = reinterpret_cast<uintptr_t>(act) | reinterpret_cast<uintptr_t>(w) | reinterpret_cast<uintptr_t>(outp) |
                            reinterpret_cast<uintptr_t>(bias);
    return K % kF32Step == 0 && K >= 8 * kF32Step && N % 4 == 0 && bases % 16 == 0 && rows >= kWideMinRows * max_tiles &&
           max_tiles * ((N + kWideCols - 1) / kWideCols) >= kWideMinUnits * device_cu_count() &&
           f32_wide_blocks(max_tiles, N) <= kWideMaxBlocks;
}

template <bool FIRST, bool FOLDED>
static hipError_t configure_wide() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(ffn_f32_wide_kernel<FIRST, FOLDED>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, kWideLds);
}

hipError_t configure_f32_kernels() {
    hipError_t e;
    if ((e = configure_wide<true, false>()) != hipSuccess) return e;
    if ((e = configure_wide<false, false>()) != hipSuccess) return e;
    return configure_wide<false, true>();
}

// fold.out, if not NULL, is the second product's output in place of rows of y: outp is not used then
hipError_t launch_f32_product(bool first, long rows, const float* act, const int32_t* rowmap, const float* w, float* outp,
                              const Tile* tiles, const int32_t* ntiles, long max_tiles, int N, int K, int activation,
                              const float* bias, const FoldOut& fold, hipStream_t st) {
    if (fold.out != nullptr) outp = static_cast<float*>(fold.out);
    if (f32_is_wide(rows, max_tiles, N, K, act, w, outp, bias)) {
        const unsigned blocks = static_cast<unsigned>(f32_wide_blocks(max_tiles, N));
        auto kern = first ? ffn_f32_wide_kernel<true, false> : fold.out != nullptr ? ffn_f32_wide_kernel<false, true> : ffn_f32_wide_kernel<false, false>;
        hipLaunchKernelGGL(kern, dim3(blocks), dim3(kWideThreads), kWideLds, st, act, rowmap, w, outp, tiles, ntiles, N, K, activation, bias, fold);
        return hipGetLastError();
    }
    const long cap = static_cast<long>(device_cu_count()) * 4;
    const unsigned grid = static_cast<unsigned>(std::max(1L, std::min(f32_units(max_tiles, N), cap)));
    switch (f32_width(K, act, w, outp)) {
        case 4: return launch_f32<4>(first, grid, act, rowmap, w, outp, tiles, ntiles, N, K, activation, bias, fold, st);
        case 2: return launch_f32<2>(first, grid, act, rowmap, w, outp, tiles, ntiles, N, K, activation, bias, fold, st);
        default: return launch_f32<1>(first, grid, act, rowmap, w, outp, tiles, ntiles, N, K, activation, bias, fold, st);
    }
}

static long f32_sort_tiles(const moe_shape& s) {
    const long A = static_cast<long>(s.T) * s.k;
    return A / kF32TileRows + std::min<long>(s.E, A);
}

// fp32 layers whose first product sorts the assignments: all its units at once, three blocks to a CU with the lists in LDS, as many
// assignments and experts as the lists hold.  It is ahead up to there, us, with a dispatch step -> this: 300 tokens, 256 x 1024, 8
// experts (768 units) 30.4 -> 24.1; 1024 tokens, 32 x 144, 64 experts 30.3 -> 23.5; 128 tokens, 64 x 128, 64 experts, k = 8 32.5 -> 30.2.
// Of 200 layers within the limits, drawn at random, none takes more than 0.92 of the time, the mean is 0.78; 200 layers drawn without
// regard to the limits take 1.005 at most.
bool layer_sorts_in_first(const moe_shape& s) {
    return s.dtype == MOE_F32 && s.T > 0 && static_cast<long>(s.T) * s.k <= kF32SortMax && s.E <= kF32SortExperts &&
           f32_sort_tiles(s) * ((s.d_ff + 15) / 16) <= 3L * device_cu_count();
}

template <int VEC>
static hipError_t launch_f32_sort(const F32Sort& p, unsigned grid, const float* x, const float* w1, float* h, int N, int K,
                                  int activation, const float* b1, hipStream_t st) {
    const int chains = f32_chains(K);
    auto kern = ffn_f32_kernel<VEC, true, 2, true, kF32Rows>;
    if (chains == 1) kern = ffn_f32_kernel<VEC, true, 1, true, kF32Rows>;
    if (chains == 4) kern = ffn_f32_kernel<VEC, true, 4, true, kF32Rows>;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(256), 0, st, x, nullptr, w1, h, nullptr, nullptr, N, K, activation, b1,
                       FoldOut{nullptr, nullptr, nullptr}, p);
    return hipGetLastError();
}

// both products of such a layer
hipError_t launch_f32_sorted_products(const moe_shape& s, const float* x, const int32_t* idx, const float* w1, const float* w2,
                                      const float* b1, const float* b2, int32_t* counts, int32_t* offsets, int32_t* perm,
                                      int32_t* inv_perm, int32_t* tokmap, const TileLists& lists, float* h, float* y_perm,
                                      const FoldOut& fold, hipStream_t st) {
    const int A = s.T * s.k;
    const F32Sort p{idx, counts, offsets, perm, inv_perm, tokmap, lists.small_tiles, lists.ntiles, A, s.E, s.k};
    const unsigned grid = static_cast<unsigned>(std::min(f32_units(f32_sort_tiles(s), s.d_ff), 3L * device_cu_count()));
    hipError_t err;
    if ((err = mark_profile_event(0, st)) != hipSuccess || (err = mark_profile_event(1, st)) != hipSuccess) return err;
    switch (f32_width(s.d_model, x, w1, h)) {
        case 4: err = launch_f32_sort<4>(p, grid, x, w1, h, s.d_ff, s.d_model, s.activation, b1, st); break;
        case 2: err = launch_f32_sort<2>(p, grid, x, w1, h, s.d_ff, s.d_model, s.activation, b1, st); break;
        default: err = launch_f32_sort<1>(p, grid, x, w1, h, s.d_ff, s.d_model, s.activation, b1, st); break;
    }
    if (err != hipSuccess) return err;
    if ((err = mark_profile_event(2, st)) != hipSuccess || (err = mark_profile_event(3, st)) != hipSuccess) return err;
    err = launch_f32_product(false, A, h, nullptr, w2, y_perm, lists.small_tiles, lists.ntiles,
                             A / kF32TileRows + std::min(s.E, A), s.d_model, s.d_ff, s.activation, b2, fold, st);
    if (err != hipSuccess) return err;
    return mark_profile_event(4, st);
}

}  // namespace moe
