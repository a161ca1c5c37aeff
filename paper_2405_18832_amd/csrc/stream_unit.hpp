#pragma once
#include <type_traits>

#include "tile_schedule.hpp"

namespace moe {

// ---------------------------------------------------------------------------
// bf16 weight-streaming product.
//
//   out[row, n] = sum_k act[row, k] * W_e[n, k]          (FIRST: activation, rounded to bf16)
//
// MFMA 16x16x32: the A operand is a packed 16(n) x 32(k) weight fragment -- one contiguous
// 1 KiB load per wavefront, 16 bytes per lane, straight from HBM into registers -- and the B
// operand is 16 token rows x 32 k of the activations (L2/L1 hits; every wave of a block reads
// the same rows).  A wavefront owns 4 n-blocks (64 output columns) x up to TFMAX*16 token rows
// over one k-slice; the KSPLIT wavefronts that share an output tile add their partial sums in
// LDS in a fixed order.  Blocks are persistent and stride over (tile, n-group) units, whose
// number is only known on the device.
//
// The inner loop is specialised on the exact number of token fragments of the tile (TFC), so
// every k-step issues a fixed number of loads: the compiler can then count outstanding loads
// exactly and keeps PF k-steps in flight across loop iterations (with a data-dependent number
// of loads it drains the queue on every iteration).
// With `rowmap`, row p of the activations is read from act[rowmap[p]] (the token gather of the
// dispatch step folded into the first product); output rows are always in permuted order.
// ---------------------------------------------------------------------------
// tuning constants (overridable at build time)
#ifndef MOE_PF_TF1
#define MOE_PF_TF1 6      // k-steps of loads in flight per wavefront, tiles of <= 16 rows
#endif
#ifndef MOE_PF_TF2
#define MOE_PF_TF2 4      // ... tiles of <= 32 rows
#endif
#ifndef MOE_PF_TF3
#define MOE_PF_TF3 3      // ... tiles of <= 48 rows
#endif
#ifndef MOE_PF_TF4
#define MOE_PF_TF4 3      // ... tiles of <= 64 rows
#endif
#ifndef MOE_PF_NARROW
#define MOE_PF_NARROW 16  // ... when a wavefront owns one column block only (one KiB of weights per step)
#endif
#ifndef MOE_PF_LDS
#define MOE_PF_LDS 6      // k-steps of weight loads in flight when the rows come from LDS
#endif

// s_waitcnt immediate that waits for vmcnt <= n only (n < 64: low four bits in [3:0], the rest in [15:14])
constexpr int vmcnt_imm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }

constexpr size_t kStreamRowLdsMax = 128 * 1024;   // largest row tile kept in LDS by streaming units
constexpr size_t stream_row_lds(int rows, int K) { return static_cast<size_t>(rows) * ((K + 63) / 64) * 128; }     // whole pairs of k-steps

template <int TFC> struct StreamPF;
template <> struct StreamPF<1> { static constexpr int value = MOE_PF_TF1; };
template <> struct StreamPF<2> { static constexpr int value = MOE_PF_TF2; };
template <> struct StreamPF<3> { static constexpr int value = MOE_PF_TF3; };
template <> struct StreamPF<4> { static constexpr int value = MOE_PF_TF4; };

// Token row and gate weight of the lane's rows (row fragment tf, row lane % 16) for a folded second product;
// fetched when a unit starts so that the two dependent loads are long done when the unit's output is stored.
template <int TFC, bool FOLD>
__device__ __forceinline__ void fold_rows(const FoldOut& fold, const Tile tl, int (&ftok)[TFC], float (&fw)[TFC], int tf0 = 0) {
    const int r = lane_of_unit() & 15;
#pragma unroll
    for (int tf = 0; tf < TFC; ++tf) {
        ftok[tf] = 0;
        fw[tf] = 0.f;
        if (FOLD) {
            ftok[tf] = fold.tokmap[tl.row0 + min((tf0 + tf) * 16 + r, tl.rows - 1)];
            fw[tf] = fold.gate[ftok[tf]];
        }
    }
}

// Output of one column group (4 n-blocks) x TFC row fragments of a tile, by one whole wavefront.
template <int TFC, int FIRST, bool FOLD, int GW = 4>
__device__ __forceinline__ void store_group(void* __restrict__ outp, const Tile tl, const int ng, const int nblk,
                                            const int N, const float* __restrict__ be,
                                            const f32x4 (&acc)[GW][TFC], const FoldOut& fold,
                                            const int (&ftok)[TFC], const float (&fw)[TFC]) {
    static_assert(GW >= 2 || !FOLD, "paired stores need pairs of column blocks");
    const int lane = lane_of_unit(), r = lane & 15, g = lane >> 4;
#pragma unroll
    for (int tf = 0; tf < TFC; ++tf) {
        const int lr = tf * 16 + r;
        const bool ok = lr < tl.rows;
        if constexpr (FIRST != 0 && GW >= 2) {
#pragma unroll
            for (int m = 0; m < GW / 2; ++m) {
                const int nb = ng * GW + 2 * m;            // N / 16 is even: the pair exists or not as a whole
                if (nb >= nblk) continue;                  // wave-uniform
                store_h_pair<FIRST, true>(outp, tl.row0 + lr, ok, nb * 16, N, be, acc[2 * m][tf], acc[2 * m + 1][tf]);
            }
        } else if constexpr (FOLD) {                       // the layer output itself
#pragma unroll
            for (int m = 0; m < GW / 2; ++m) {
                const int nb = ng * GW + 2 * m;
                if (nb >= nblk) continue;                  // wave-uniform
                store_folded_pair(static_cast<uint16_t*>(fold.out), ftok[tf], fw[tf], ok, nb * 16, N, be, acc[2 * m][tf], acc[2 * m + 1][tf]);
            }
        } else {
#pragma unroll
            for (int nf = 0; nf < GW; ++nf) {
                const int nb = ng * GW + nf;
                if (ok && nb < nblk)
                    store_out<FIRST, true>(outp, tl.row0 + lr, nb * 16 + g * 4, N, be, acc[nf][tf]);
            }
        }
    }
}

// Output of the wavefront's share of a column group: the pair of n-blocks from nb on, row fragments from tf0 on, as far as the
// tile has rows.
template <int TH, int FIRST, bool FOLD>
__device__ __forceinline__ void store_share(void* __restrict__ outp, const Tile tl, const int nb, const int tf0,
                                            const int nblk, const int N, const float* __restrict__ be, const f32x4 (&own)[2][TH],
                                            const FoldOut& fold, const int (&ftok)[TH], const float (&fw)[TH]) {
    const int lane = lane_of_unit(), r = lane & 15, g = lane >> 4;
    if (nb >= nblk) return;                                // wave-uniform; N / 16 is even: the pair exists or not as a whole
#pragma unroll
    for (int t = 0; t < TH; ++t) {
        const int lr = (tf0 + t) * 16 + r;
        const bool ok = lr < tl.rows;
        if constexpr (FIRST != 0) {
            store_h_pair<FIRST, true>(outp, tl.row0 + lr, ok, nb * 16, N, be, own[0][t], own[1][t]);
        } else if constexpr (FOLD) {
            store_folded_pair(static_cast<uint16_t*>(fold.out), ftok[t], fw[t], ok, nb * 16, N, be, own[0][t], own[1][t]);
        } else if (ok) {
            store_out<FIRST, true>(outp, tl.row0 + lr, nb * 16 + g * 4, N, be, own[0][t]);
            store_out<FIRST, true>(outp, tl.row0 + lr, nb * 16 + 16 + g * 4, N, be, own[1][t]);
        }
    }
}

// Whole loops of a unit (Hooks given: the product kernel, whose wavefronts have 256 registers) issue a step's loads right behind the
// MFMAs that free their registers.  Left to itself the compiler gathers the loads of several steps, which takes up to 350 registers;
// the kernels that have those are as fast either way and keep its order.

// What else a wavefront does at three points of a unit: when its last load is out, when that has arrived, and when all wavefronts of
// the block have got there, before the unit's output is stored.
struct NoHooks {
    __device__ __forceinline__ void loads_out() {}
    __device__ __forceinline__ void loads_done() {}
    __device__ __forceinline__ bool meet() const { return false; }         // whether `met` needs a barrier where the unit has none
    __device__ __forceinline__ void met() {}
};

// One wavefront's share of one unit: 4 n-blocks x TFC token fragments over k-steps [kb0, kb1); `wave`: its number, scalar where registers
// are short (few_first_kernel, which has enough, passes it in a vector register: 35.6 us for a token of 2048 x 8192, k = 2, scalar 35.7).
template <int TFC, int TFMAX, int KSPLIT, int FIRST, bool FOLD, int GW = 4, typename Hooks = NoHooks>
__device__ __forceinline__ void stream_unit(const uint16_t* __restrict__ act,
                                            const int32_t* __restrict__ rowmap,
                                            const uint16_t* __restrict__ wpk, void* __restrict__ outp,
                                            const Tile tl, const int ng, const bool active, const int N,
                                            const int K, const int kb0, const int kb1, f32x4* red,
                                            const bool act_kmajor,
                                            const float* __restrict__ bias, const FoldOut& fold, const int wave,
                                            Hooks&& hooks = {}) {
    constexpr int PF = GW == 4 ? StreamPF<TFC>::value : MOE_PF_NARROW;
    constexpr int NGB = 4 / KSPLIT;
    constexpr bool STEPWISE = !std::is_same_v<std::remove_reference_t<Hooks>, NoHooks>;
    const int lane = lane_of_unit();
    const int r = lane & 15, g = lane >> 4;
    const int ks = KSPLIT == 1 ? 0 : wave % KSPLIT, ngs = wave / KSPLIT;
    const int nblk = N >> 4, kblk = K >> 5;
    // The wavefronts that share a column group each add up and store a share of it: one pair of n-blocks (m) and an equal run of the
    // row fragments.  (As the work of one of them the sums took 192 registers, and its stores all of the unit's end.)
    constexpr bool SHARED = KSPLIT > 1 && GW >= 2;
    constexpr int PAIRS = SHARED ? GW / 2 : 1, RUNS = SHARED ? KSPLIT / PAIRS : 1, TH = (TFC + RUNS - 1) / RUNS;
    const int m = SHARED ? ks % PAIRS : 0, tf0 = SHARED ? (ks / PAIRS) * TH : 0;
    f32x4 acc[GW][TFC];
#pragma unroll
    for (int nf = 0; nf < GW; ++nf)
#pragma unroll
        for (int tf = 0; tf < TFC; ++tf) acc[nf][tf] = f32x4{0.f, 0.f, 0.f, 0.f};

    int ftok[TH];
    float fw[TH];
    fold_rows<TH, FOLD>(fold, tl, ftok, fw, tf0);
    if (active && kb0 < kb1) {
        const uint16_t* wp[GW];
#pragma unroll
        for (int nf = 0; nf < GW; ++nf) {
            const int nb = min(ng * GW + nf, nblk - 1);
            wp[nf] = wpk + (static_cast<size_t>(tl.expert) * nblk + nb) * kblk * 512 + lane * 8;
        }
        const bool km = FIRST == 0 ? true : act_kmajor;     // the second product always reads h
        const uint16_t* ap[TFC];
#pragma unroll
        for (int tf = 0; tf < TFC; ++tf) {
            int row = tl.row0 + min(tf * 16 + r, tl.rows - 1);
            if (rowmap != nullptr) row = rowmap[row];       // gather: permuted position -> token row
            // operand rows are row-major (the caller's x or x_perm) or k-step-major (h, gathered x)
            ap[tf] = km ? act + h_index(row, g * 8, kblk) : act + static_cast<size_t>(row) * K + g * 8;
        }
        const size_t kstride = km ? kStepStride : 32;   // elements per k-step
        bf16x8 a[PF][GW], b[PF][TFC];
        auto issue = [&](int slot, int kb) {
#pragma unroll
            for (int nf = 0; nf < GW; ++nf)
                a[slot][nf] = *reinterpret_cast<const bf16x8*>(wp[nf] + static_cast<size_t>(kb) * 512);
#pragma unroll
            for (int tf = 0; tf < TFC; ++tf) b[slot][tf] = *reinterpret_cast<const bf16x8*>(ap[tf] + kb * kstride);
        };
        auto fma = [&](int slot) {
#pragma unroll
            for (int tf = 0; tf < TFC; ++tf)
#pragma unroll
                for (int nf = 0; nf < GW; ++nf)
                    acc[nf][tf] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[slot][nf], b[slot][tf], acc[nf][tf], 0, 0, 0);
        };
        // prologue: always PF steps of loads (past the end the last step is re-read, never used)
#pragma unroll
        for (int p = 0; p < PF; ++p) issue(p, min(kb0 + p, kb1 - 1));
        int kb = kb0;
        for (; kb + 2 * PF <= kb1; kb += PF) {            // steady state: fixed number of loads per step
#pragma unroll
            for (int p = 0; p < PF; ++p) {
                fma(p);
                if (STEPWISE) __builtin_amdgcn_sched_barrier(0);
                issue(p, kb + p + PF);
                if (STEPWISE) __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (kb + PF < kb1) {                               // one partial round of refills
#pragma unroll
            for (int p = 0; p < PF; ++p) {
                fma(p);
                if (STEPWISE) __builtin_amdgcn_sched_barrier(0);
                issue(p, min(kb + p + PF, kb1 - 1));
                if (STEPWISE) __builtin_amdgcn_sched_barrier(0);
            }
            kb += PF;
        }
#pragma unroll
        for (int p = 0; p < PF; ++p) {                     // drain: no more loads
            if (p == 0) hooks.loads_out();
            if (kb + p < kb1) fma(p);
        }
    } else {
        hooks.loads_out();
    }
    hooks.loads_done();

    // LDS only: a bare barrier after the LDS accesses have completed.  (__syncthreads() also waits for every outstanding
    // global store, i.e. for the previous unit's output rows: a store latency per unit.)
    const float* be = bias ? bias + static_cast<size_t>(tl.expert) * N : nullptr;
    if constexpr (SHARED) {
        // the share of wavefront o from the KSPLIT - 1 others: fragment (i, t) from the q-th of them at
        // ((o * (KSPLIT - 1) + q) * 2 * TH + i * TH + t) * 64 + lane
        f32x4* const mine = red + static_cast<size_t>(ngs) * (KSPLIT * (KSPLIT - 1) * 2 * TH) * 64 + lane;
        f32x4 own[2][TH];
#pragma unroll
        for (int o = 0; o < KSPLIT; ++o) {
            const int h0 = (o / PAIRS) * TH;
            f32x4* const to = mine + (o * (KSPLIT - 1) + (ks < o ? ks : ks - 1)) * (2 * TH * 64);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int t = 0; t < TH; ++t) {
                    if (h0 + t >= TFC) continue;
                    if (o == ks) own[i][t] = acc[2 * (o % PAIRS) + i][h0 + t];              // wave-uniform
                    else if (active) to[(i * TH + t) * 64] = acc[2 * (o % PAIRS) + i][h0 + t];
                }
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        hooks.met();
        if (active && tf0 < TFC) {                         // wave-uniform
            const f32x4* const from = mine + ks * (KSPLIT - 1) * (2 * TH * 64);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int t = 0; t < TH; ++t) {             // in the order of the contraction
                    f32x4 part[KSPLIT - 1];
#pragma unroll
                    for (int q = 0; q < KSPLIT - 1; ++q) part[q] = from[(q * 2 * TH + i * TH + t) * 64];
                    f32x4 sum = ks == 0 ? own[i][t] : part[0];
#pragma unroll
                    for (int s = 1; s < KSPLIT; ++s) {
                        const f32x4 lower = part[s - 1];
                        sum += s == ks ? own[i][t] : s < ks ? part[s < KSPLIT - 1 ? s : s - 1] : lower;
                    }
                    own[i][t] = sum;
                }
            store_share<TH, FIRST, FOLD>(outp, tl, ng * GW + 2 * m, tf0, nblk, N, be, own, fold, ftok, fw);
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");       // `red` may be reused
    } else if constexpr (KSPLIT > 1) {                     // one n-block: the first wavefront's
        if (active && ks > 0) {
            f32x4* dst = red + static_cast<size_t>((ks - 1) * NGB + ngs) * GW * TFMAX * 64 + lane;
#pragma unroll
            for (int nf = 0; nf < GW; ++nf)
#pragma unroll
                for (int tf = 0; tf < TFC; ++tf) dst[(nf * TFMAX + tf) * 64] = acc[nf][tf];
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (active && ks == 0) {
#pragma unroll
            for (int s = 1; s < KSPLIT; ++s) {
                const f32x4* src = red + static_cast<size_t>((s - 1) * NGB + ngs) * GW * TFMAX * 64 + lane;
#pragma unroll
                for (int nf = 0; nf < GW; ++nf)
#pragma unroll
                    for (int tf = 0; tf < TFC; ++tf) acc[nf][tf] += src[(nf * TFMAX + tf) * 64];
            }
            store_group<TFC, FIRST, FOLD, GW>(outp, tl, ng, nblk, N, be, acc, fold, ftok, fw);
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    } else if (active) {
        store_group<TFC, FIRST, FOLD, GW>(outp, tl, ng, nblk, N, be, acc, fold, ftok, fw);
    }
}

// The same unit when all four wavefronts of the block share the tile's rows over the same k range
// (KSPLIT = 1: the block covers four column groups): the rows are copied once per block into LDS
// instead of being fetched by every wavefront at every k-step.  That takes the
// row operand out of the vector-memory queue that the weights stream through (one quarter of the
// requests, issued once, asynchronously) and out of the registers that hold loads in flight.
// `tok_lds` holds, for every row fragment, ceil(K / 64) pairs of k-steps of 2 KiB each: rows of the blocked layout as two MFMA
// fragments of 1 KiB, plain rows as 16 lines of 128 bytes whose 16-byte pieces are permuted by the row's number.
template <int TFC, int FIRST, bool FOLD, typename Hooks = NoHooks>
__device__ __forceinline__ void stream_unit_lds(const uint16_t* __restrict__ act,
                                                const int32_t* __restrict__ rowmap,
                                                const uint16_t* __restrict__ wpk, void* __restrict__ outp,
                                                const Tile tl, const int ng, const bool active, const int N,
                                                const int K, const bool act_kmajor,
                                                const float* __restrict__ bias, unsigned char* tok_lds,
                                                const FoldOut& fold, const int wave,
                                                Hooks&& hooks = {}) {
    constexpr int PF = MOE_PF_LDS;
    constexpr bool STEPWISE = !std::is_same_v<std::remove_reference_t<Hooks>, NoHooks>;
    const int lane = lane_of_unit();
    const int r = lane & 15, g = lane >> 4;
    const int nblk = N >> 4, kblk = K >> 5;
    f32x4 acc[4][TFC];
#pragma unroll
    for (int nf = 0; nf < 4; ++nf)
#pragma unroll
        for (int tf = 0; tf < TFC; ++tf) acc[nf][tf] = f32x4{0.f, 0.f, 0.f, 0.f};

    int ftok[TFC];
    float fw[TFC];
    fold_rows<TFC, FOLD>(fold, tl, ftok, fw);
    // The lane's rows in a copy: of a fragment whose rows are 64 bytes apart (the blocked layout) row lane % 16, k-group lane / 16;
    // of plain rows row lane / 8 of either half of the fragment and one of the eight 16-byte pieces of a line, two k-steps.
    int rows_of[TFC][2];
#pragma unroll
    for (int tf = 0; tf < TFC; ++tf)
#pragma unroll
        for (int i = 0; i < 2; ++i) {                      // fetched before the barrier, whose wait hides them
            if (act_kmajor && i == 1) continue;
            rows_of[tf][i] = tl.row0 + min(tf * 16 + (act_kmajor ? r : i * 8 + (lane >> 3)), tl.rows - 1);
            if (rowmap != nullptr) rows_of[tf][i] = rowmap[rows_of[tf][i]];
        }
    // every wavefront has finished reading the previous unit's rows
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const uint32_t lds0 = lds_address(tok_lds);
    const int pairs = (kblk + 1) >> 1;
    if (act_kmajor) {                                      // wavefront w copies the fragments (tf, kb) with kb = w, w + 4, ...
#pragma unroll
        for (int tf = 0; tf < TFC; ++tf) {
            const uint16_t* ap = act + h_index(rows_of[tf][0], g * 8, kblk);
            for (int kb = wave; kb < kblk; kb += 4)
                copy16_to_lds(ap + static_cast<size_t>(kb) * kStepStride, lds0 + (tf * 2 * pairs + kb) * 1024);
        }
    } else {
        // Pairs of k-steps, in lines: one line of every row per eight lanes (as fragments, 16 consecutive lanes touch 16 rows and half of
        // each line, four times the accesses).  Piece p of row r lies at r * 128 + 16 * (p ^ (r & 7)) of its pair, so that reads of
        // eight rows touch different banks.
        const int piece = (lane & 7) ^ (lane >> 3);
#pragma unroll
        for (int tf = 0; tf < TFC; ++tf)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const uint16_t* ap = act + static_cast<size_t>(rows_of[tf][i]) * K;
                for (int kp = wave; kp < pairs; kp += 4)   // the last pair may be half a one: its other pieces are never read
                    copy16_to_lds(ap + min(kp * 64 + piece * 8, K - 8), lds0 + ((tf * pairs + kp) * 2 + i) * 1024);
            }
    }

    const uint16_t* wp[4];
#pragma unroll
    for (int nf = 0; nf < 4; ++nf) {
        const int nb = min(ng * 4 + nf, nblk - 1);
        wp[nf] = wpk + (static_cast<size_t>(tl.expert) * nblk + nb) * kblk * 512 + lane * 8;
    }
    bf16x8 a[PF][4];
    auto issue = [&](int slot, int kb) {
#pragma unroll
        for (int nf = 0; nf < 4; ++nf)
            a[slot][nf] = *reinterpret_cast<const bf16x8*>(wp[nf] + static_cast<size_t>(kb) * 512);
    };
    if (active) {
#pragma unroll
        for (int p = 0; p < PF; ++p) issue(p, min(p, kblk - 1));   // past the end: re-read, never used
    }
    // The row copies were issued before the weight loads, and loads complete in order: they have landed
    // once at most the weight loads are outstanding ... for every wavefront.
    if (active) __builtin_amdgcn_s_waitcnt(vmcnt_imm(PF * 4));
    else __builtin_amdgcn_s_waitcnt(0x0F70);
    asm volatile("s_barrier" ::: "memory");

    if (active) {
        // where the lane's operand of an even k-step lies in the pair, and how far the odd one's is from there
        const int even = act_kmajor ? lane * 16 : r * 128 + ((g ^ (r & 7)) << 4);
        const int odd = act_kmajor ? even + 1024 : even ^ 64;
        auto fma = [&](int slot, int kb) {
            bf16x8 b[TFC];
            const unsigned char* bl = tok_lds + (kb >> 1) * 2048 + ((kb & 1) ? odd : even);
#pragma unroll
            for (int tf = 0; tf < TFC; ++tf) b[tf] = *reinterpret_cast<const bf16x8*>(bl + tf * pairs * 2048);
#pragma unroll
            for (int tf = 0; tf < TFC; ++tf)
#pragma unroll
                for (int nf = 0; nf < 4; ++nf)
                    acc[nf][tf] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[slot][nf], b[tf], acc[nf][tf], 0, 0, 0);
        };
        int kb = 0;
        for (; kb + 2 * PF <= kblk; kb += PF) {
#pragma unroll
            for (int p = 0; p < PF; ++p) {
                fma(p, kb + p);
                if (STEPWISE) __builtin_amdgcn_sched_barrier(0);
                issue(p, kb + p + PF);
                if (STEPWISE) __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (kb + PF < kblk) {
#pragma unroll
            for (int p = 0; p < PF; ++p) {
                fma(p, kb + p);
                if (STEPWISE) __builtin_amdgcn_sched_barrier(0);
                issue(p, min(kb + p + PF, kblk - 1));
                if (STEPWISE) __builtin_amdgcn_sched_barrier(0);
            }
            kb += PF;
        }
        hooks.loads_out();
#pragma unroll
        for (int p = 0; p < PF; ++p)
            if (kb + p < kblk) fma(p, kb + p);
    } else {
        hooks.loads_out();
    }
    hooks.loads_done();
    if (hooks.meet()) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");       // block-uniform
    hooks.met();
    if (active) {
        const float* be = bias ? bias + static_cast<size_t>(tl.expert) * N : nullptr;
        store_group<TFC, FIRST, FOLD>(outp, tl, ng, nblk, N, be, acc, fold, ftok, fw);
    }
}

}  // namespace moe
