#pragma once
#include "tile_schedule.hpp"

namespace moe {

// ---------------------------------------------------------------------------
// bf16 weight-streaming product.
//
//   out[row, n] = sum_k act[row, k] * W_e[n, k]          (FIRST: relu, rounded to bf16)
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

constexpr size_t kStreamRowLdsMax = 128 * 1024;   // largest row tile kept in LDS by the streaming kernel

template <int TFC> struct StreamPF;
template <> struct StreamPF<1> { static constexpr int value = MOE_PF_TF1; };
template <> struct StreamPF<2> { static constexpr int value = MOE_PF_TF2; };
template <> struct StreamPF<3> { static constexpr int value = MOE_PF_TF3; };
template <> struct StreamPF<4> { static constexpr int value = MOE_PF_TF4; };

// Token row and gate weight of the lane's rows (row fragment tf, row lane % 16) for a folded second product;
// fetched when a unit starts so that the two dependent loads are long done when the unit's output is stored.
template <int TFC, bool FOLD>
__device__ __forceinline__ void fold_rows(const FoldOut& fold, const Tile tl, int (&ftok)[TFC], float (&fw)[TFC]) {
    const int r = threadIdx.x & 15;
#pragma unroll
    for (int tf = 0; tf < TFC; ++tf) {
        ftok[tf] = 0;
        fw[tf] = 0.f;
        if (FOLD) {
            ftok[tf] = fold.tokmap[tl.row0 + min(tf * 16 + r, tl.rows - 1)];
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
    static_assert(GW == 4 || !FOLD, "paired stores need groups of 4 column blocks");
    const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
#pragma unroll
    for (int tf = 0; tf < TFC; ++tf) {
        const int lr = tf * 16 + r;
        const bool ok = lr < tl.rows;
        if constexpr (FIRST != 0 && GW == 4) {
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const int nb = ng * 4 + 2 * m;             // N / 16 is even: the pair exists or not as a whole
                if (nb >= nblk) continue;                  // wave-uniform
                store_h_pair<FIRST, true>(outp, tl.row0 + lr, ok, nb * 16, N, be, acc[2 * m][tf], acc[2 * m + 1][tf]);
            }
        } else if constexpr (FOLD && GW == 4) {            // the layer output itself
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const int nb = ng * 4 + 2 * m;
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

// One wavefront's share of one unit: 4 n-blocks x TFC token fragments over k-steps [kb0, kb1).
template <int TFC, int TFMAX, int KSPLIT, int FIRST, bool FOLD, int GW = 4>
__device__ __forceinline__ void stream_unit(const uint16_t* __restrict__ act,
                                            const int32_t* __restrict__ rowmap,
                                            const uint16_t* __restrict__ wpk, void* __restrict__ outp,
                                            const Tile tl, const int ng, const bool active, const int N,
                                            const int K, const int kb0, const int kb1, f32x4* red,
                                            const bool act_kmajor,
                                            const float* __restrict__ bias, const FoldOut& fold) {
    constexpr int PF = GW == 4 ? StreamPF<TFC>::value : MOE_PF_NARROW;
    constexpr int NGB = 4 / KSPLIT;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int r = lane & 15, g = lane >> 4;
    const int ks = wave % KSPLIT, ngs = wave / KSPLIT;
    const int nblk = N >> 4, kblk = K >> 5;
    f32x4 acc[GW][TFC];
#pragma unroll
    for (int nf = 0; nf < GW; ++nf)
#pragma unroll
        for (int tf = 0; tf < TFC; ++tf) acc[nf][tf] = f32x4{0.f, 0.f, 0.f, 0.f};

    int ftok[TFC];
    float fw[TFC];
    fold_rows<TFC, FOLD>(fold, tl, ftok, fw);
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
                issue(p, kb + p + PF);
            }
        }
        if (kb + PF < kb1) {                               // one partial round of refills
#pragma unroll
            for (int p = 0; p < PF; ++p) {
                fma(p);
                issue(p, min(kb + p + PF, kb1 - 1));
            }
            kb += PF;
        }
#pragma unroll
        for (int p = 0; p < PF; ++p)                       // drain: no more loads
            if (kb + p < kb1) fma(p);
    }

    if (KSPLIT > 1) {
        if (active && ks > 0) {
            f32x4* dst = red + (static_cast<size_t>((ks - 1) * NGB + ngs) * GW * TFMAX) * 64 + lane;
#pragma unroll
            for (int nf = 0; nf < GW; ++nf)
#pragma unroll
                for (int tf = 0; tf < TFC; ++tf) dst[(nf * TFMAX + tf) * 64] = acc[nf][tf];
        }
        // LDS only: a bare barrier after the LDS writes have completed.  (__syncthreads() also waits for
        // every outstanding global store, i.e. for the previous unit's output rows: a store latency per unit.)
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (active && ks == 0) {
#pragma unroll
            for (int s = 1; s < KSPLIT; ++s) {
                const f32x4* src = red + (static_cast<size_t>((s - 1) * NGB + ngs) * GW * TFMAX) * 64 + lane;
#pragma unroll
                for (int nf = 0; nf < GW; ++nf)
#pragma unroll
                    for (int tf = 0; tf < TFC; ++tf) acc[nf][tf] += src[(nf * TFMAX + tf) * 64];
            }
        }
    }
    if (active && ks == 0) {
        const float* be = bias ? bias + static_cast<size_t>(tl.expert) * N : nullptr;
        store_group<TFC, FIRST, FOLD, GW>(outp, tl, ng, nblk, N, be, acc, fold, ftok, fw);
    }
    if (KSPLIT > 1) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // `red` may be reused
}

}  // namespace moe
