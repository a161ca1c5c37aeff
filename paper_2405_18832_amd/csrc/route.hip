// Gating and routing: logits = x . w_gate^T (+ bias), softmax over experts, top-k with
// lowest-index tie-break, gate weights, per-expert token histogram, prefix sums and the
// top-H hot mask (paper Section 2.1 for the gating network, Section 3.3 for the token
// counts and the hot set).
//
// Two kernels.  route_bf16_kernel / route_f32_kernel: one block per chunk of tokens computes the chunk's
// logits into LDS, picks each token's experts there and leaves the chunk's per-expert
// histogram in the workspace.  dispatch_kernel: one block turns the chunk histograms
// into counts, prefix sums, the hot mask and the expert tile lists, while the others place the
// chunks' assignments.  Nothing is ordered through atomics on global memory, so every output
// is the same on every run.
#include <algorithm>
#include <type_traits>

#include "tile_schedule.hpp"
#include "topk.hpp"

namespace moe {

// Floats per token row of the logits in LDS: whole groups of 16 * NF experts (the accumulate step writes
// full fragments) plus 4, which keeps the rows 16-byte aligned and moves consecutive rows to different banks.
__host__ __device__ inline int route_row_stride(int E, int NF) { return (E + 16 * NF - 1) / (16 * NF) * (16 * NF) + 4; }

// ---------------------------------------------------------------------------
// Routing of a chunk of tokens by one block: logits into LDS, softmax and top-k there, and the chunk's histogram to
// chunk_hist[chunk * E + e].
//
// route_bf16_kernel<TF, NF, STAGES, KSPLIT>: chunk = 16 * TF tokens, 4 wavefronts, experts 16 * NF at a time.  MFMA 16x16x32
// with gate rows as the A operand and token rows as the B operand (a lane ends up with 4 consecutive experts of one token);
// a wavefront owns NF / 4 fragments of experts for all the chunk's tokens.  Rows of both operands go through a ring of LDS stages, 64 k
// = one 128-byte line of every row per stage, copied by eight consecutive lanes each.  (Loaded straight into operand form,
// 16 consecutive lanes touch 16 different rows: 64 cache accesses per load instruction instead of 16, which bounded the
// kernel; neither more loads in flight nor more wavefronts changed it, nor do more stages than four.)  The 16-byte pieces of
// a row are permuted by its row number, so that the rows a read touches at once lie in different banks.  The contraction runs
// in four chains per accumulator, which are added at the end.
// KSPLIT = 4: every wavefront takes all the experts for a quarter of the contraction, through a ring of its own (no barriers),
// and the quarters are added in LDS in order.
// DIRECT: x and w_gate are 16-byte aligned and the copies go straight into LDS.  Otherwise (a view into a larger buffer) they
// go through registers: ordinary loads take any alignment.  They are issued four stages ahead and written to LDS two stages
// ahead (5003 tokens x 2048 x 128 experts, with dispatch: 23.4 us aligned, 28.1 at an odd element, 44 when each was waited for at
// once; with the loads in operand form 49 and 130).
// Dynamic LDS: the ring or rings, then logits [16 * TF][route_row_stride(E, NF)] floats, then the histogram [E] ints.
// ---------------------------------------------------------------------------
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
constexpr int kRouteWaves = 4;
template <int TF, int NF, int STAGES, int KSPLIT>
struct RouteRing {
    static constexpr int kWaves = kRouteWaves / KSPLIT;                // wavefronts that share a ring
    static constexpr int kRows = (16 * (TF + NF) + 8 * kWaves - 1) / (8 * kWaves) * (8 * kWaves);     // whole copies for each
    static constexpr int kStageBytes = kRows * 128;
    static constexpr int kCopies = kRows / (8 * kWaves);               // per wavefront and stage, 8 rows each
    static constexpr int kRingBytes = STAGES * kStageBytes;
    static constexpr int kBytes = KSPLIT * kRingBytes;
    // s_waitcnt operand that lets all but two stages' worth of a wavefront's copies be in flight (vmcnt: bits 3:0 and 15:14)
    static constexpr int kInFlight = (STAGES - 2) * kCopies;
    static constexpr int kWait = 0x0F70 | (kInFlight & 15) | (kInFlight >> 4) << 14;
};

template <int TF, int NF, int STAGES, int KSPLIT, bool DIRECT>
__global__ __launch_bounds__(kRouteWaves * 64) void route_bf16_kernel(const uint16_t* __restrict__ x,
                                                                      const uint16_t* __restrict__ wg,
                                                                      const float* __restrict__ bias,
                                                                      int32_t* __restrict__ topk_idx,
                                                                      float* __restrict__ topk_w, float* __restrict__ margin,
                                                                      int32_t* __restrict__ chunk_hist, int T, int d, int E,
                                                                      int k, int renorm) {
    using Ring = RouteRing<TF, NF, STAGES, KSPLIT>;
    constexpr int TOK = 16 * TF, NW = kRouteWaves, NT = NW * 64, RW = Ring::kWaves, FPW = NF / RW, S = STAGES, P = Ring::kCopies;
    static_assert(NF % RW == 0, "whole fragments of experts per wavefront");
    extern __shared__ __attribute__((aligned(16))) unsigned char route_lds[];
    const int Ep = route_row_stride(E, NF);
    float* L = reinterpret_cast<float*>(route_lds + Ring::kBytes);
    int32_t* hist = reinterpret_cast<int32_t*>(L + TOK * Ep);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int r = lane & 15, g = lane >> 4;
    const int t0 = blockIdx.x * TOK;
    for (int e = threadIdx.x; e < E; e += NT) hist[e] = 0;

    // the ring's stages of the contraction: all of them, or this wavefront's share
    static_assert(KSPLIT == 1 || RW == 1, "one ring, or one per wavefront");
    const int rw = KSPLIT == 1 ? wave : 0, part = KSPLIT == 1 ? 0 : wave;
    const int per_ring = (((d >> 5) + 1) / 2 + KSPLIT - 1) / KSPLIT;
    const int j0 = part * per_ring, ksteps = (d >> 5) - 2 * j0, nstages = min((ksteps + 1) >> 1, per_ring);     // <= 0: none
    unsigned char* ring = route_lds + part * Ring::kRingBytes;
    const uint32_t ring0 = lds_address(ring);
    // copies: this wavefront's p-th takes the rows 8 * (rw + RW * p) ... + 7 of a stage, tokens first
    const int piece = (lane & 7) ^ (lane >> 3);
    for (int ec = 0; ec < E; ec += 16 * NF) {
        const uint16_t* src[P];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int row = 8 * (rw + RW * p) + (lane >> 3);
            src[p] = (row < TOK ? x + static_cast<size_t>(min(t0 + row, T - 1)) * d
                                : wg + static_cast<size_t>(min(ec + row - TOK, E - 1)) * d) + j0 * 64;
        }
        // this lane's 16 bytes of stage j by the p-th copy.  A last stage of one 32-k step: its second half is read again from
        // the first, and not used
        auto from = [&](int j, int p) { return src[p] + j * 64 + ((2 * j + 1 < ksteps) ? piece : (piece & 3)) * 8; };
        auto stage_in = [&](int j) {                       // DIRECT
            const uint32_t base = ring0 + (j % S) * Ring::kStageBytes;
#pragma unroll
            for (int p = 0; p < P; ++p) copy16_to_lds(from(j, p), base + (rw + RW * p) * 1024);
        };
        // otherwise through registers: loaded four steps ahead, written two steps ahead
        uint4 held[2][DIRECT ? 1 : P];
        auto load_stage = [&](int j, auto& v) {            // past the end: the last stage again, which is not used
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const u32x4_any u = *reinterpret_cast<const u32x4_any*>(from(min(j, nstages - 1), p));
                v[p] = uint4{u[0], u[1], u[2], u[3]};
            }
        };
        auto write_stage = [&](int j, const auto& v) {
#pragma unroll
            for (int p = 0; p < P; ++p)
                *reinterpret_cast<uint4*>(ring + (j % S) * Ring::kStageBytes + (rw + RW * p) * 1024 + lane * 16) = v[p];
        };
        f32x4 acc[4][FPW][TF];                             // [chain]
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int nf = 0; nf < FPW; ++nf)
#pragma unroll
                for (int tf = 0; tf < TF; ++tf) acc[c][nf][tf] = f32x4{0.f, 0.f, 0.f, 0.f};
        // the last stages of a previous group of experts have been read
        if (ec > 0) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if constexpr (DIRECT) {
#pragma unroll
            for (int j = 0; j < S - 1; ++j)
                if (j < nstages) stage_in(j);
        } else if (nstages > 0) {
            load_stage(0, held[0]);
            load_stage(1, held[1]);
            write_stage(0, held[0]);
            load_stage(2, held[0]);
            write_stage(1, held[1]);
            load_stage(3, held[1]);
        }
        f32x4 first[FPW];                                  // what the sums start from: the bias
#pragma unroll
        for (int nf = 0; nf < FPW; ++nf) {
            first[nf] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (bias != nullptr) {
#pragma unroll
                for (int i = 0; i < 4; ++i) first[nf][i] = bias[min(ec + (rw * FPW + nf) * 16 + g * 4 + i, E - 1)];
            }
        }
        auto step = [&](int j, auto parity) {
            constexpr int C = 2 * decltype(parity)::value;
            // Stage j has landed for every wavefront, and nobody reads stage j - 1 any more: the reads are waited for here,
            // because nothing else keeps the matrix instructions that consume them in front of the barrier.
            if constexpr (DIRECT) {
                if (j + S - 2 < nstages) __builtin_amdgcn_s_waitcnt(Ring::kWait);
                else __builtin_amdgcn_s_waitcnt(0x0F70);
            }
            if constexpr (RW > 1) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if constexpr (DIRECT) {
                if (j + S - 1 < nstages) stage_in(j + S - 1);
            } else {
                write_stage(j + 2, held[C / 2]);
                load_stage(j + 4, held[C / 2]);
            }
            const unsigned char* st = ring + (j % S) * Ring::kStageBytes;
            const int halves = 2 * j + 1 < ksteps ? 2 : 1;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (h == 1 && halves == 1) break;          // uniform
                const int at = r * 128 + (((h * 4 + g) ^ (r & 7)) << 4);
                bf16x8 a[FPW], b[TF];
#pragma unroll
                for (int nf = 0; nf < FPW; ++nf)
                    a[nf] = *reinterpret_cast<const bf16x8*>(st + (TOK + (rw * FPW + nf) * 16) * 128 + at);
#pragma unroll
                for (int tf = 0; tf < TF; ++tf) b[tf] = *reinterpret_cast<const bf16x8*>(st + tf * 16 * 128 + at);
#pragma unroll
                for (int nf = 0; nf < FPW; ++nf)
#pragma unroll
                    for (int tf = 0; tf < TF; ++tf)
                        acc[C + h][nf][tf] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[nf], b[tf], acc[C + h][nf][tf], 0, 0, 0);
            }
        };
        int j = 0;
        for (; j + 1 < nstages; j += 2) {
            step(j, std::integral_constant<int, 0>{});
            step(j + 1, std::integral_constant<int, 1>{});
        }
        if (j < nstages) step(j, std::integral_constant<int, 0>{});
        // The compiler does not see that the branch around the second half of a last stage leads from a matrix instruction
        // straight to the reads of its result, and leaves out the wait states these need (d = 32 gave wrong logits).
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_nop 7\n\ts_nop 7");
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < KSPLIT; ++q) {                 // shares of the contraction in order
            if (part == q) {
#pragma unroll
                for (int nf = 0; nf < FPW; ++nf)
#pragma unroll
                    for (int tf = 0; tf < TF; ++tf) {
                        f32x4* p = reinterpret_cast<f32x4*>(L + (tf * 16 + r) * Ep + ec + (rw * FPW + nf) * 16 + g * 4);
                        *p = ((q == 0 ? first[nf] : *p) + acc[0][nf][tf]) + acc[1][nf][tf] + (acc[2][nf][tf] + acc[3][nf][tf]);
                    }
            }
            if (q + 1 < KSPLIT) __syncthreads();
        }
    }
    __syncthreads();

    // top-k: 4 tokens per wavefront and pass
    const int grp = lane >> 4, sub = lane & 15;
#pragma unroll 1
    for (int tl = wave * 4 + grp; tl < TOK; tl += NW * 4) {
        const int t = t0 + tl;
        const bool live = t < T;
        const size_t o = static_cast<size_t>(live ? t : 0) * k;
        topk_from_lds(L + tl * Ep, E, k, renorm, sub, live, topk_idx + o, topk_w + o,
                      margin ? margin + (live ? t : 0) : nullptr, hist);
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += NT) chunk_hist[static_cast<size_t>(blockIdx.x) * E + e] = hist[e];
}

// fp32: 16 tokens, 16 experts at a time with the fp32 matrix instruction, 16 k per step (operands as in ffn_f32.hip); the
// wavefronts split the contraction and meet in LDS in wave order.  Dynamic LDS: logits, then the histogram, as above.
__global__ __launch_bounds__(kRouteWaves * 64) void route_f32_kernel(const float* __restrict__ x, const float* __restrict__ wg,
                                                                     const float* __restrict__ bias,
                                                                     int32_t* __restrict__ topk_idx,
                                                                     float* __restrict__ topk_w, float* __restrict__ margin,
                                                                     int32_t* __restrict__ chunk_hist, int T, int d, int E,
                                                                     int k, int renorm) {
    constexpr int TOK = 16, NW = kRouteWaves, NT = NW * 64;
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const int Ep = route_row_stride(E, 1);
    float* L = lds;
    int32_t* hist = reinterpret_cast<int32_t*>(lds + TOK * Ep);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int t0 = blockIdx.x * TOK;
    for (int e = threadIdx.x; e < E; e += NT) hist[e] = 0;

    const int r = lane & 15, g = lane >> 4;
    const float* xr = x + static_cast<size_t>(min(t0 + r, T - 1)) * d + g * 4;
    const int steps = d >> 4, per = (steps + NW - 1) / NW;
    const int s0 = min(steps, wave * per), s1 = min(steps, s0 + per);
    const bool aligned = d % 4 == 0 && ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(wg)) & 15) == 0;
    for (int ec = 0; ec < E; ec += 16) {
        const float* wr = wg + static_cast<size_t>(min(ec + r, E - 1)) * d + g * 4;
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
        auto fma = [&](const f32x4 a, const f32x4 b) {
#pragma unroll
            for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b[j], acc, 0, 0, 0);
        };
        auto walk = [&](auto vec) {
            constexpr int PF = 8;
            for (int s = s0; s < s1; s += PF) {
                f32x4 a[PF], b[PF];
#pragma unroll
                for (int p = 0; p < PF; ++p) {
                    const int k0 = min(s + p, s1 - 1) * 16;          // past the end: re-read, not used
                    a[p] = load_k4<decltype(vec)::value>(wr + k0);
                    b[p] = load_k4<decltype(vec)::value>(xr + k0);
                }
#pragma unroll
                for (int p = 0; p < PF; ++p)
                    if (s + p < s1) fma(a[p], b[p]);
            }
        };
        if (aligned) walk(std::integral_constant<int, 4>{});
        else walk(std::integral_constant<int, 1>{});
        if ((d & 15) != 0 && wave == NW - 1)
            fma(load_k4_tail(wr + steps * 16, (d & 15) - g * 4), load_k4_tail(xr + steps * 16, (d & 15) - g * 4));
        for (int w = 0; w < NW; ++w) {
            if (wave == w) {
                f32x4* p = reinterpret_cast<f32x4*>(L + r * Ep + ec + g * 4);
                f32x4 sofar = f32x4{0.f, 0.f, 0.f, 0.f};
                if (w > 0) {
                    sofar = *p;
                } else if (bias != nullptr) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) sofar[i] = bias[min(ec + g * 4 + i, E - 1)];
                }
                *p = acc + sofar;
            }
            __syncthreads();
        }
    }

    // top-k: 4 tokens per wavefront and pass
    const int grp = lane >> 4, sub = lane & 15;
#pragma unroll 1
    for (int tl = wave * 4 + grp; tl < TOK; tl += NW * 4) {
        const int t = t0 + tl;
        const bool live = t < T;
        const size_t o = static_cast<size_t>(live ? t : 0) * k;
        topk_from_lds(L + tl * Ep, E, k, renorm, sub, live, topk_idx + o, topk_w + o,
                      margin ? margin + (live ? t : 0) : nullptr, hist);
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += NT) chunk_hist[static_cast<size_t>(blockIdx.x) * E + e] = hist[e];
}

// ---------------------------------------------------------------------------
// From the chunk histograms [nchunks][E] of the assignments to counts, offsets, hot mask, tile lists and places.
// ---------------------------------------------------------------------------
constexpr int kMaxWaves = 16;           // wavefronts of a block of 1024 threads

// Per expert, the sum of its histogram over all chunks (total) and over the chunks before cfirst (before), by a block
// of 1024 threads; thread e < E returns with expert e's.  Threads that take consecutive experts of one chunk read
// contiguously: the block is cut into ngrp = 1024 / Ew groups of Ew threads (Ew = E rounded up to whole wavefronts),
// group q adds up the chunks [q * seg, (q + 1) * seg) 16 loads at a time, and the group sums meet in LDS (`groups`,
// 2048 ints).
__device__ __forceinline__ void sum_chunks(const int32_t* __restrict__ chunk_hist, int nchunks, int E, int cfirst,
                                           int32_t* groups, int& total, int& before) {
    const int Ew = min(1024, (E + 63) & ~63), ngrp = 1024 / Ew;
    const int q = threadIdx.x / Ew, ex = threadIdx.x - q * Ew;
    const bool have = q < ngrp && ex < E;                  // threads past ngrp * Ew (none when Ew divides 1024)
    const int seg = (nchunks + ngrp - 1) / ngrp;
    const int c_begin = min(q * seg, nchunks), c_end = min(c_begin + seg, nchunks);
    const int32_t* col = chunk_hist + (have ? ex : 0);
    int sum = 0, low = 0;
    for (int c0 = c_begin; c0 < c_end; c0 += 16) {
        int v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = (have && c0 + i < c_end) ? col[static_cast<size_t>(c0 + i) * E] : 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            sum += v[i];
            low += c0 + i < cfirst ? v[i] : 0;
        }
    }
    if (have) {
        groups[q * Ew + ex] = sum;
        groups[1024 + q * Ew + ex] = low;
    }
    __syncthreads();
    total = before = 0;
    const int e = threadIdx.x;
    if (e < E) {
        for (int o = 0; o < ngrp; ++o) {
            total += groups[o * Ew + e];
            before += groups[1024 + o * Ew + e];
        }
    }
}

// counts, offsets, hot mask and tile lists from the token counts, by a block of 1024 threads, thread e owning expert e
// with `mine` tokens.  `cnt` (2 * MOE_MAX_E ints) and `scan` (kScanInts) are LDS scratch.  Any output pointer may be NULL.
// `mask_copy`: a second place for the hot mask (the caller's output buffer, which later kernels of the call must not depend
// on: the caller may write to it as soon as the call has returned).  Returns the expert's first row.
__device__ __forceinline__ int finalize_outputs(int mine, int E, int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
                                                int H, uint8_t* __restrict__ hot_mask, uint8_t* __restrict__ mask_copy,
                                                const uint8_t* __restrict__ mask_in, const TileLists lists, int want_tiles,
                                                int32_t* cnt, int32_t* scan) {
    const int e = threadIdx.x;
    bool on = e < E;
    if (H >= 0) {                                          // uniform: rank by count, ties by lowest index
        // The ranks are counted by the whole block, group q of Ew threads comparing with its share of the experts (one
        // thread per expert reads E counts one after the other: 3 us of a step at 128 experts).
        const int Ew = min(1024, (E + 63) & ~63), ngrp = 1024 / Ew;
        const int q = threadIdx.x / Ew, ex = threadIdx.x - q * Ew;
        if (e < E) cnt[e] = mine;
        __syncthreads();
        if (q < ngrp && ex < E) {
            const int my = cnt[ex], per = (E + ngrp - 1) / ngrp;
            int rank = 0;
            for (int o = q * per; o < min(E, (q + 1) * per); ++o) rank += (cnt[o] > my || (cnt[o] == my && o < ex)) ? 1 : 0;
            cnt[MOE_MAX_E + q * Ew + ex] = rank;
        }
        __syncthreads();
        if (e < E) {
            int rank = 0;
            for (int o = 0; o < ngrp; ++o) rank += cnt[MOE_MAX_E + o * Ew + e];
            on = rank < H;
            if (hot_mask) hot_mask[e] = on ? 1 : 0;
            if (mask_copy) mask_copy[e] = on ? 1 : 0;
        }
    } else if (mask_in != nullptr && e < E) {
        on = mask_in[e] != 0;
    }
    int row0, rows, at_min = 0, joined = 0;
    if (want_tiles && lists.big_min > 0) {                 // uniform
        const int v[3] = {mine, on ? big_tiles_at_min(mine, lists) : 0, on ? half_tiles_joined(mine, lists) : 0};
        int incl[3], total[3];
        block_scan(v, incl, total, scan, (E + 63) >> 6);
        row0 = incl[0] - mine;
        rows = total[0];
        at_min = total[1];
        joined = total[2];
    } else {
        const int v[1] = {mine};
        int incl[1], total[1];
        block_scan(v, incl, total, scan, (E + 63) >> 6);
        row0 = incl[0] - mine;
        rows = total[0];
    }
    if (e < E) {
        if (counts) counts[e] = mine;
        if (offsets) offsets[e] = row0;
    }
    if (e == 0 && offsets) offsets[E] = rows;
    if (want_tiles) emit_tiles(e, E, row0, on ? mine : 0, at_min, joined, lists, scan + 48);     // uniform: a kernel argument
    return row0;
}

__device__ __forceinline__ int expert_bits(int E) {
    int b = 0;
    while ((1 << b) < E) ++b;
    return b;
}

// One launch for the whole step: with `finalize`, block 0 writes the outputs of finalize_outputs, and every other block
// places the assignments of PW chunks, one wavefront each (PW = 0: nothing is placed).  Every block adds the histograms
// up by itself: at most kDispatchMaxHist ints from L2, less than a second launch and the trip of the sums through
// memory (4096 tokens, 128 experts: 12.4 + 4.8 us as two launches, 9.2 us).
// `offsets_in` != NULL: the caller's offsets instead of the counts' prefix sums.
// Dynamic LDS: PW * E ints, the next free slot of every expert per wavefront.
template <int PW>
__global__ __launch_bounds__(1024) void dispatch_kernel(const int32_t* __restrict__ chunk_hist, int nchunks, int E,
                                                        const int32_t* __restrict__ offsets_in, int finalize,
                                                        int32_t* __restrict__ counts, int32_t* __restrict__ offsets, int H,
                                                        uint8_t* __restrict__ hot_mask, uint8_t* __restrict__ mask_copy,
                                                        const uint8_t* __restrict__ mask_in, const TileLists lists,
                                                        const int want_tiles, const PlaceArgs place) {
    extern __shared__ int32_t next_all[];
    __shared__ int32_t groups[2048];
    __shared__ int32_t scan[kScanInts];
    const int e = threadIdx.x;
    int total, before;
    if (finalize && blockIdx.x == 0) {
        sum_chunks(chunk_hist, nchunks, E, 0, groups, total, before);
        __syncthreads();                                   // `groups` becomes `cnt`
        finalize_outputs(total, E, counts, offsets, H, hot_mask, mask_copy, mask_in, lists, want_tiles, groups, scan);
        return;
    }
    if constexpr (PW > 0) {
        const int wave = threadIdx.x >> 6;
        const int cfirst = (static_cast<int>(blockIdx.x) - (finalize ? 1 : 0)) * PW;
        const int c = cfirst + wave;
        const bool mine = wave < PW && c < nchunks;        // wave-uniform
        ChunkExperts first{};
        if (mine) first = chunk_experts(place.idx, place.A, place.chunk, c);
        int own[PW];                                       // the block's chunks, expert e
#pragma unroll
        for (int w = 0; w < PW; ++w)
            own[w] = (e < E && cfirst + w < nchunks) ? chunk_hist[static_cast<size_t>(cfirst + w) * E + e] : 0;
        sum_chunks(chunk_hist, nchunks, E, cfirst, groups, total, before);
        int at = 0;
        if (offsets_in != nullptr) {
            if (e < E) at = offsets_in[e];
        } else {
            const int v[1] = {total};
            int incl[1], all[1];
            block_scan(v, incl, all, scan, (E + 63) >> 6);
            at = incl[0] - total;
        }
        at += before;
#pragma unroll
        for (int w = 0; w < PW; ++w) {
            if (e < E) next_all[w * E + e] = at;
            at += own[w];
        }
        __syncthreads();
        if (mine)
            place_chunk(place.idx, first, next_all + wave * E, place.perm, place.inv_perm, place.tokmap, place.A, E, place.k,
                        expert_bits(E), place.chunk, c);
    }
}

// The same for histograms too large to be read by every block: one block writes the outputs and turns the histograms
// into slot bases in place (per expert, exclusive prefix sums over the chunks), then perm_place_kernel places.
__global__ __launch_bounds__(1024) void scan_finalize_kernel(int32_t* __restrict__ chunk_hist, int nchunks, int E,
                                                             int finalize, int32_t* __restrict__ counts,
                                                             int32_t* __restrict__ offsets, int H,
                                                             uint8_t* __restrict__ hot_mask, uint8_t* __restrict__ mask_copy,
                                                             const uint8_t* __restrict__ mask_in, const TileLists lists,
                                                             const int want_tiles) {
    __shared__ int32_t groups[2048];
    __shared__ int32_t scan[kScanInts];
    int total, before;
    sum_chunks(chunk_hist, nchunks, E, 0, groups, total, before);
    __syncthreads();
    {
        const int Ew = min(1024, (E + 63) & ~63), ngrp = 1024 / Ew;      // the groups of sum_chunks
        const int q = threadIdx.x / Ew, ex = threadIdx.x - q * Ew;
        const int seg = (nchunks + ngrp - 1) / ngrp;
        const int c_begin = min(q * seg, nchunks), c_end = min(c_begin + seg, nchunks);
        if (q < ngrp && ex < E) {
            int carry = 0;
            for (int o = 0; o < q; ++o) carry += groups[o * Ew + ex];
            int32_t* col = chunk_hist + ex;
            for (int c0 = c_begin; c0 < c_end; c0 += 16) {
                int v[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) v[i] = c0 + i < c_end ? col[static_cast<size_t>(c0 + i) * E] : 0;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    if (c0 + i < c_end) col[static_cast<size_t>(c0 + i) * E] = carry;
                    carry += v[i];
                }
            }
        }
    }
    __syncthreads();
    if (finalize) finalize_outputs(total, E, counts, offsets, H, hot_mask, mask_copy, mask_in, lists, want_tiles, groups, scan);
}

// places one chunk per wavefront from the slot bases that scan_finalize_kernel left
__global__ __launch_bounds__(256) void perm_place_kernel(const int32_t* __restrict__ offsets,
                                                         const int32_t* __restrict__ chunk_base, int E, int nchunks,
                                                         const PlaceArgs place) {
    __shared__ int32_t next_all[4][MOE_MAX_E];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int c = blockIdx.x * 4 + wave;
    if (c >= nchunks) return;                   // no block-wide barrier below: waves are independent
    int32_t* next = next_all[wave];
    const ChunkExperts first = chunk_experts(place.idx, place.A, place.chunk, c);
    for (int e = lane; e < E; e += 64) next[e] = offsets[e] + chunk_base[static_cast<size_t>(c) * E + e];
    __builtin_amdgcn_wave_barrier();
    place_chunk(place.idx, first, next, place.perm, place.inv_perm, place.tokmap, place.A, E, place.k, expert_bits(E),
                place.chunk, c);
}

// Hot-set size from the counts (Section 3.3, Eq. 6) and the top-H mask.  One block, thread e owns
// expert e.  The real-valued H is formed in double precision with individually rounded operations
// (no fused multiply-add), so that it is the same number a plain double evaluation gives.
__global__ __launch_bounds__(1024) void select_hot_kernel(const int32_t* __restrict__ counts, int E, double alpha,
                                                          double bw_a, double bw_b, int32_t* __restrict__ H_out,
                                                          uint8_t* __restrict__ hot_mask) {
    __shared__ int32_t cnt[MOE_MAX_E];
    __shared__ int32_t active;
    const int e = threadIdx.x;
    if (e == 0) active = 0;
    const int mine = e < E ? counts[e] : 0;
    cnt[e] = mine;
    __syncthreads();
    if (e < E && mine > 0) atomicAdd(&active, 1);
    __syncthreads();
    const double share = __ddiv_rn(__dmul_rn(alpha, bw_a), __dadd_rn(bw_a, bw_b));
    const double h = floor(__dadd_rn(__dmul_rn(share, static_cast<double>(active)), 0.5));
    const int H = h >= static_cast<double>(E) ? E : (h <= 0.0 ? 0 : static_cast<int>(h));
    if (e == 0 && H_out != nullptr) *H_out = H;
    if (e < E && hot_mask != nullptr) {
        int rank = 0;
        for (int o = 0; o < E; ++o) rank += (cnt[o] > mine || (cnt[o] == mine && o < e)) ? 1 : 0;
        hot_mask[e] = rank < H ? 1 : 0;
    }
}

hipError_t launch_select_hot(int E, const int32_t* counts, double alpha, double bw_a, double bw_b, int32_t* H_out,
                             uint8_t* hot_mask, hipStream_t st) {
    hipLaunchKernelGGL(select_hot_kernel, dim3(1), dim3(1024), 0, st, counts, E, alpha, bw_a, bw_b, H_out, hot_mask);
    return hipGetLastError();
}

__global__ void mask_out_kernel(const uint8_t* __restrict__ src, uint8_t* __restrict__ dst, int E) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < E) dst[e] = src ? (src[e] ? 1 : 0) : 1;
}

hipError_t launch_mask_out(const uint8_t* mask_or_null, uint8_t* dst, int E, hipStream_t st) {
    hipLaunchKernelGGL(mask_out_kernel, dim3((E + 255) / 256), dim3(256), 0, st, mask_or_null, dst, E);
    return hipGetLastError();
}

// Tokens per routing block and fragments of experts taken at a time, from the shape alone.  More tokens per block read the
// gate matrix fewer times, as long as the chip is one round of blocks: with 313 blocks of 16 tokens on 256 CUs, 5003 tokens
// took 42 us, with 157 of 32 tokens 31 us (128 experts, d = 2048, an earlier form of the kernel).
// Two fragments (up to 32 experts) mean that the wavefronts split the contraction, each with a ring of its own: side by side
// in one ring, two or three of them would work on experts that do not exist, and every stage waits for the block.  That pays
// from d = 1024 on (16 experts, tokens x d, with dispatch: 1000 x 2048 14.9 -> 11.2 us, 1000 x 4096 21.4 -> 13.2, 8300 x 2048 22.7 ->
// 18.9, 8300 x 768 15.9 -> 16.1); past 64 tokens per CU two blocks of 64 tokens share a CU and hide it (20000 x 2048 38 against 28 us).
struct RouteCfg { int tok, nf; };
static RouteCfg route_cfg(const moe_shape& s) {
    RouteCfg c{16, 1};
    if (s.dtype != MOE_BF16) return c;
    const int cus = device_cu_count();
    c.nf = s.E > 64 ? 8 : (s.E > 32 || s.d_model < 1024 || s.T > 64 * cus ? 4 : 2);
    if (route_is_split(s)) return c;                       // the split path works in chunks of 16 tokens
    if (s.T > 32 * cus && s.E <= 128) c.tok = 64;
    else if (s.T > 16 * cus && s.E <= 256) c.tok = 32;
    return c;
}

int route_chunk_tokens(const moe_shape& s) { return route_cfg(s).tok; }

// Most dynamic LDS a routing kernel asks for: four rings of three stages of 96 rows (144 KiB) next to the logits of 64 tokens
// x 32 experts, or one of four stages of 160 rows (80 KiB) next to those of 16 tokens x 1024 experts; and the histogram.
constexpr size_t kRouteLdsMax = kLdsPerCu;

template <typename ST>
using RouteKernel = void (*)(const ST*, const ST*, const float*, int32_t*, float*, float*, int32_t*, int, int, int, int, int);

template <typename ST>
static hipError_t launch_route_kernel(RouteKernel<ST> kern, int tok, int nf, size_t ring, const moe_shape& s, const void* x,
                                      const void* w_gate, const float* bias, int32_t* idx, float* gate, float* margin,
                                      int32_t* chunk_hist, hipStream_t st) {
    const unsigned grid = static_cast<unsigned>((s.T + tok - 1) / tok);
    const size_t lds = ring + static_cast<size_t>(tok) * route_row_stride(s.E, nf) * 4 + static_cast<size_t>(s.E) * 4;
    if (lds > kRouteLdsMax) return hipErrorInvalidValue;     // cannot happen for E <= MOE_MAX_E (see kRouteLdsMax)
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kRouteWaves * 64), lds, st, static_cast<const ST*>(x),
                       static_cast<const ST*>(w_gate), bias, idx, gate, margin, chunk_hist, s.T, s.d_model, s.E, s.k,
                       s.renormalize);
    return hipGetLastError();
}

template <int TF, int NF, int STAGES, int KSPLIT>
static hipError_t launch_route_bf16(const moe_shape& s, const void* x, const void* w_gate, const float* bias, int32_t* idx,
                                    float* gate, float* margin, int32_t* chunk_hist, hipStream_t st) {
    // whole rows are multiples of 64 bytes
    const bool aligned = ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(w_gate)) & 15) == 0;
    auto kern = aligned ? route_bf16_kernel<TF, NF, STAGES, KSPLIT, true> : route_bf16_kernel<TF, NF, STAGES, KSPLIT, false>;
    return launch_route_kernel<uint16_t>(kern, 16 * TF, NF, RouteRing<TF, NF, STAGES, KSPLIT>::kBytes, s, x, w_gate, bias, idx,
                                         gate, margin, chunk_hist, st);
}

template <typename Kernel>
static hipError_t configure_route(Kernel kern) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                               static_cast<int>(kRouteLdsMax));
}

template <int TF, int NF, int STAGES, int KSPLIT>
static hipError_t configure_route_bf16() {
    const hipError_t e = configure_route(route_bf16_kernel<TF, NF, STAGES, KSPLIT, true>);
    return e != hipSuccess ? e : configure_route(route_bf16_kernel<TF, NF, STAGES, KSPLIT, false>);
}

// Few tokens (a decode step): the gate product is one skinny GEMM whose cost is reading the gate weights, and
// one block per 16 tokens would leave that to one or two CUs.  gate_partial_kernel cuts it into
// (16 experts) x (1 / kGateSplit of the contraction) x (16 tokens) pieces, one wavefront each, which leave fp32
// partial logits in the workspace; route_topk_kernel adds the slices in order (plus the bias) and does the
// softmax / top-k / chunk histogram per 16 tokens as route_bf16_kernel does.
__global__ __launch_bounds__(64) void gate_partial_kernel(const uint16_t* __restrict__ x,
                                                          const uint16_t* __restrict__ wg,
                                                          float* __restrict__ part, int T, int d, int E, int Tpad) {
    const int lane = threadIdx.x, r = lane & 15, g = lane >> 4;
    const int nb = blockIdx.x, ks = blockIdx.y, tf = blockIdx.z;
    const int ksteps = d >> 5;
    const int per = (ksteps + kGateSplit - 1) / kGateSplit;
    const int kb0 = min(ksteps, ks * per), kb1 = min(ksteps, kb0 + per);
    const uint16_t* xr = x + static_cast<size_t>(min(tf * 16 + r, T - 1)) * d + g * 8;
    const uint16_t* wr = wg + static_cast<size_t>(min(nb * 16 + r, E - 1)) * d + g * 8;
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    constexpr int PF = 8;
    for (int kb = kb0; kb < kb1; kb += PF) {
        bf16x8 a[PF], b[PF];
#pragma unroll
        for (int p = 0; p < PF; ++p) {
            const int kk = min(kb + p, kb1 - 1);            // past the end: re-read, not used
            a[p] = *reinterpret_cast<const bf16x8*>(wr + kk * 32);
            b[p] = *reinterpret_cast<const bf16x8*>(xr + kk * 32);
        }
#pragma unroll
        for (int p = 0; p < PF; ++p)
            if (kb + p < kb1) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[p], b[p], acc, 0, 0, 0);
    }
    // lane (r, g): token tf * 16 + r, experts nb * 16 + 4 g + 0..3
    const int t = tf * 16 + r;
    float* dst = part + (static_cast<size_t>(ks) * Tpad + t) * E;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int e = nb * 16 + g * 4 + i;
        if (t < T && e < E) dst[e] = acc[i];               // rows of padding are not read
    }
}

__global__ __launch_bounds__(256) void route_topk_kernel(const float* __restrict__ part,
                                                         const float* __restrict__ bias,
                                                         int32_t* __restrict__ topk_idx, float* __restrict__ topk_w,
                                                         float* __restrict__ margin,
                                                         int32_t* __restrict__ chunk_hist, int T, int E, int k,
                                                         int renorm, int Tpad) {
    extern __shared__ float lds[];
    const int Ep = E + 1;
    float* L = lds;
    int32_t* hist = reinterpret_cast<int32_t*>(lds + 16 * Ep);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int t0 = blockIdx.x * 16;
    for (int e = threadIdx.x; e < E; e += 256) hist[e] = 0;
    // 4 logits per thread and pass: their 4 * kGateSplit partial sums are loaded before any is added (a wait
    // per logit otherwise: this kernel is two blocks of pure latency on the decode path).  Only the rows of tokens that exist
    // have been written.
    const int logits = min(16, T - t0) * E;
    for (int i0 = threadIdx.x; i0 < logits; i0 += 4 * 256) {
        float p[4][kGateSplit];
        float b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = min(i0 + u * 256, logits - 1);   // past the end: re-read, not stored
            const int tl = i / E, e = i - tl * E, t = t0 + tl;
            b[u] = bias ? bias[e] : 0.f;
#pragma unroll
            for (int ks = 0; ks < kGateSplit; ++ks) p[u][ks] = part[(static_cast<size_t>(ks) * Tpad + t) * E + e];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * 256;
            if (i >= logits) break;
            const int tl = i / E, e = i - tl * E;
            float s = b[u];
#pragma unroll
            for (int ks = 0; ks < kGateSplit; ++ks) s += p[u][ks];      // fixed order
            L[tl * Ep + e] = s;
        }
    }
    __syncthreads();
    const int grp = lane >> 4, sub = lane & 15;
    const int tl = wave * 4 + grp;                     // 4 wavefronts x 4 tokens
    const int t = t0 + tl;
    const bool live = t < T;
    const size_t o = static_cast<size_t>(live ? t : 0) * k;
    topk_from_lds(L + tl * Ep, E, k, renorm, sub, live, topk_idx + o, topk_w + o,
                  margin ? margin + (live ? t : 0) : nullptr, hist);
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += 256) chunk_hist[static_cast<size_t>(blockIdx.x) * E + e] = hist[e];
}

// route_topk_kernel and dispatch_kernel in one block of 1024 threads, for layers of at most 64 tokens and
// 256 experts (decoder steps): the 16 wavefronts take 4 tokens each, the four 16-token chunks keep their
// histograms and their experts in LDS, and the block goes straight on to the prefix sums, tile lists and the
// placement.  One launch less on a path that is a chain of short kernels, and no trip through memory between its steps
// (with histograms and experts read back from memory the kernel took 10.2 us at one token).
// Dynamic LDS: logits [64][E + 1] floats, then histograms [4][E] ints, then experts [64 * k] ints.
constexpr int kTopkFinalizeMaxE = 256;
__global__ __launch_bounds__(1024) void route_topk_finalize_kernel(const float* __restrict__ part,
                                                                   const float* __restrict__ bias,
                                                                   int32_t* __restrict__ topk_idx,
                                                                   float* __restrict__ topk_w,
                                                                   float* __restrict__ margin, int T, int E, int k,
                                                                   int renorm, int Tpad, int32_t* __restrict__ counts,
                                                                   int32_t* __restrict__ offsets, int H,
                                                                   uint8_t* __restrict__ hot_mask,
                                                                   uint8_t* __restrict__ mask_copy,
                                                                   const uint8_t* __restrict__ mask_in,
                                                                   const TileLists lists, const int want_tiles,
                                                                   const PlaceArgs place) {
    extern __shared__ float lds[];
    const int Ep = E + 1;
    float* L = lds;
    int32_t* hist = reinterpret_cast<int32_t*>(lds + 64 * Ep);
    int32_t* experts = hist + 4 * E;
    __shared__ int32_t cnt[2 * MOE_MAX_E];
    __shared__ int32_t scan[kScanInts];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int nchunks = Tpad >> 4;                         // <= 4
    for (int i = threadIdx.x; i < 4 * E; i += 1024) hist[i] = 0;
    // 4 logits per thread and pass, their 4 * kGateSplit partial sums loaded before any is added (of the T tokens only:
    // at one token the 16 padded rows were 64 KB for a single CU)
    for (int i0 = threadIdx.x; i0 < T * E; i0 += 4 * 1024) {
        float p[4][kGateSplit];
        float b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = min(i0 + u * 1024, T * E - 1);      // past the end: re-read, not stored
            const int tl = i / E, e = i - tl * E;
            b[u] = bias ? bias[e] : 0.f;
#pragma unroll
            for (int ks = 0; ks < kGateSplit; ++ks) p[u][ks] = part[(static_cast<size_t>(ks) * Tpad + tl) * E + e];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * 1024;
            if (i >= T * E) break;
            const int tl = i / E, e = i - tl * E;
            float sum = b[u];
#pragma unroll
            for (int ks = 0; ks < kGateSplit; ++ks) sum += p[u][ks];      // fixed order
            L[tl * Ep + e] = sum;
        }
    }
    __syncthreads();
    const int grp = lane >> 4, sub = lane & 15;
    const int tl = wave * 4 + grp;                         // 16 wavefronts x 4 tokens
    if (wave * 4 < Tpad) {                                 // wave-uniform: Tpad is a multiple of 16
        const bool live = tl < T;
        const size_t o = static_cast<size_t>(live ? tl : 0) * k;
        topk_from_lds(L + tl * Ep, E, k, renorm, sub, live, topk_idx + o, topk_w + o,
                      margin ? margin + (live ? tl : 0) : nullptr, hist + (tl >> 4) * E, experts + o);
    }
    __syncthreads();
    const int e = threadIdx.x;
    int mine = 0;
    if (e < E)
        for (int c = 0; c < nchunks; ++c) mine += hist[c * E + e];
    int at = finalize_outputs(mine, E, counts, offsets, H, hot_mask, mask_copy, mask_in, lists, want_tiles, cnt, scan);
    if (place.idx == nullptr) return;                      // uniform
    if (e < E) {                                           // histograms -> the chunks' first free slots
        for (int c = 0; c < nchunks; ++c) {
            const int n = hist[c * E + e];
            hist[c * E + e] = at;
            at += n;
        }
    }
    __syncthreads();
    if (wave < nchunks)
        place_chunk(experts, chunk_experts(experts, place.A, place.chunk, wave), hist + wave * E, place.perm, place.inv_perm,
                    place.tokmap, place.A, E, place.k, expert_bits(E), place.chunk, wave);
}

constexpr size_t kTopkFinalizeLdsMax = static_cast<size_t>(64) * (kTopkFinalizeMaxE + 1) * 4 + 4 * kTopkFinalizeMaxE * 4 + 64 * MOE_MAX_K * 4;

hipError_t configure_route_kernels(int) {
    hipError_t e;
    if ((e = configure_route(route_f32_kernel)) != hipSuccess) return e;
    if ((e = configure_route_bf16<1, 4, 4, 1>()) != hipSuccess) return e;
    if ((e = configure_route_bf16<2, 4, 4, 1>()) != hipSuccess) return e;
    if ((e = configure_route_bf16<4, 4, 4, 1>()) != hipSuccess) return e;
    if ((e = configure_route_bf16<4, 4, 3, 1>()) != hipSuccess) return e;
    if ((e = configure_route_bf16<1, 2, 4, 4>()) != hipSuccess) return e;
    if ((e = configure_route_bf16<2, 2, 4, 4>()) != hipSuccess) return e;
    if ((e = configure_route_bf16<4, 2, 3, 4>()) != hipSuccess) return e;
    if ((e = configure_route_bf16<1, 8, 4, 1>()) != hipSuccess) return e;
    if ((e = configure_route_bf16<2, 8, 4, 1>()) != hipSuccess) return e;
    if ((e = configure_route_bf16<4, 8, 4, 1>()) != hipSuccess) return e;
    if ((e = configure_route(route_topk_kernel)) != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void*>(route_topk_finalize_kernel),
                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kTopkFinalizeLdsMax));
}

hipError_t launch_gate_partial(const moe_shape& s, const void* x, const void* w_gate, float* part, hipStream_t st) {
    const int tfs = (s.T + 15) / 16, Tpad = tfs * 16, nbs = (s.E + 15) / 16;
    hipLaunchKernelGGL(gate_partial_kernel, dim3(nbs, kGateSplit, tfs), dim3(64), 0, st, static_cast<const uint16_t*>(x),
                       static_cast<const uint16_t*>(w_gate), part, s.T, s.d_model, s.E, Tpad);
    return hipGetLastError();
}

static hipError_t launch_route_small(const moe_shape& s, const void* x, const void* w_gate, const float* bias,
                                     int32_t* idx, float* gate, float* margin, int32_t* chunk_hist, float* part,
                                     hipStream_t st) {
    const int tfs = (s.T + 15) / 16, Tpad = tfs * 16;
    hipError_t err = launch_gate_partial(s, x, w_gate, part, st);
    if (err != hipSuccess) return err;
    const size_t lds = static_cast<size_t>(16) * (s.E + 1) * 4 + static_cast<size_t>(s.E) * 4;   // <= 70 KiB
    hipLaunchKernelGGL(route_topk_kernel, dim3(tfs), dim3(256), lds, st, part, bias, idx, gate, margin, chunk_hist, s.T,
                       s.E, s.k, s.renormalize, Tpad);
    return hipGetLastError();
}

hipError_t launch_route_fused(const moe_shape& s, const void* x, const void* w_gate, const float* bias,
                              int32_t* idx, float* gate, float* margin, int32_t* chunk_hist, float* gate_part_ws,
                              hipStream_t st) {
    if (s.dtype != MOE_BF16)
        return launch_route_kernel<float>(route_f32_kernel, 16, 1, 0, s, x, w_gate, bias, idx, gate, margin, chunk_hist, st);
    if (route_is_split(s) && gate_part_ws != nullptr)
        return launch_route_small(s, x, w_gate, bias, idx, gate, margin, chunk_hist, gate_part_ws, st);
    const RouteCfg c = route_cfg(s);
    switch (c.tok + c.nf) {
        case 64 + 8: return launch_route_bf16<4, 8, 4, 1>(s, x, w_gate, bias, idx, gate, margin, chunk_hist, st);
        case 32 + 8: return launch_route_bf16<2, 8, 4, 1>(s, x, w_gate, bias, idx, gate, margin, chunk_hist, st);
        case 16 + 8: return launch_route_bf16<1, 8, 4, 1>(s, x, w_gate, bias, idx, gate, margin, chunk_hist, st);
        case 64 + 2: return launch_route_bf16<4, 2, 3, 4>(s, x, w_gate, bias, idx, gate, margin, chunk_hist, st);
        case 32 + 2: return launch_route_bf16<2, 2, 4, 4>(s, x, w_gate, bias, idx, gate, margin, chunk_hist, st);
        case 16 + 2: return launch_route_bf16<1, 2, 4, 4>(s, x, w_gate, bias, idx, gate, margin, chunk_hist, st);
        case 64 + 4:
            // more than a round of blocks: three stages, so that two blocks fit a CU (8 experts, 20000 x 768 26.5 -> 19.0 us); up to
            // a round, four (8300 x 768 16.5 -> 15.9)
            if (s.T > 64 * device_cu_count())
                return launch_route_bf16<4, 4, 3, 1>(s, x, w_gate, bias, idx, gate, margin, chunk_hist, st);
            return launch_route_bf16<4, 4, 4, 1>(s, x, w_gate, bias, idx, gate, margin, chunk_hist, st);
        case 32 + 4: return launch_route_bf16<2, 4, 4, 1>(s, x, w_gate, bias, idx, gate, margin, chunk_hist, st);
        default: return launch_route_bf16<1, 4, 4, 1>(s, x, w_gate, bias, idx, gate, margin, chunk_hist, st);
    }
}

// Histograms of up to this many ints are added up by every block of dispatch_kernel; larger ones would cost the blocks
// more than the second launch does.
constexpr long kDispatchMaxHist = 64 * 1024;
constexpr int kDispatchMaxChunks = 1024;      // few experts: a chunk's row is short, and its loads wait for one another

template <int PW>
static hipError_t launch_dispatch_pw(const int32_t* chunk_hist, int nchunks, int E, const int32_t* offsets_in, bool finalize,
                                     int32_t* counts, int32_t* offsets, int H, uint8_t* hot_mask, uint8_t* mask_copy,
                                     const uint8_t* mask_in, const TileLists& lists, bool want_tiles, const PlaceArgs& place,
                                     hipStream_t st) {
    const unsigned blocks = (PW > 0 ? static_cast<unsigned>((nchunks + PW - 1) / std::max(PW, 1)) : 0u) + (finalize ? 1 : 0);
    hipLaunchKernelGGL(dispatch_kernel<PW>, dim3(blocks), dim3(1024), static_cast<size_t>(PW) * E * 4, st, chunk_hist, nchunks,
                       E, offsets_in, finalize ? 1 : 0, counts, offsets, H, hot_mask, mask_copy, mask_in, lists, want_tiles ? 1 : 0,
                       place);
    return hipGetLastError();
}

// chunk histograms -> counts, offsets, hot mask, tile lists (`finalize`) and places (place.idx != NULL); with offsets_in
// the places start from the caller's offsets.  Overwrites chunk_hist where it is large.
static hipError_t launch_dispatch(int32_t* chunk_hist, int nchunks, int E, const int32_t* offsets_in, bool finalize,
                                  int32_t* counts, int32_t* offsets, int H, uint8_t* hot_mask, uint8_t* mask_copy,
                                  const uint8_t* mask_in, const TileLists* lists, const PlaceArgs* place, hipStream_t st) {
    const TileLists none{nullptr, nullptr, nullptr, nullptr, nullptr, 16, 0, 0, 0, 0, 0, 1, false};
    const PlaceArgs no_place{nullptr, nullptr, nullptr, nullptr, 0, 1, 1};
    const TileLists& tl = lists ? *lists : none;
    const bool tiles = lists != nullptr;
    if (place == nullptr || nchunks == 0)
        return launch_dispatch_pw<0>(chunk_hist, nchunks, E, nullptr, true, counts, offsets, H, hot_mask, mask_copy, mask_in, tl,
                                     tiles, no_place, st);
    if (static_cast<long>(nchunks) * E <= kDispatchMaxHist && nchunks <= kDispatchMaxChunks) {
        if (E <= 256)
            return launch_dispatch_pw<16>(chunk_hist, nchunks, E, offsets_in, finalize, counts, offsets, H, hot_mask, mask_copy,
                                          mask_in, tl, tiles, *place, st);
        return launch_dispatch_pw<4>(chunk_hist, nchunks, E, offsets_in, finalize, counts, offsets, H, hot_mask, mask_copy, mask_in,
                                     tl, tiles, *place, st);
    }
    hipLaunchKernelGGL(scan_finalize_kernel, dim3(1), dim3(1024), 0, st, chunk_hist, nchunks, E, finalize ? 1 : 0, counts,
                       offsets, H, hot_mask, mask_copy, mask_in, tl, tiles ? 1 : 0);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(perm_place_kernel, dim3((nchunks + 3) / 4), dim3(256), 0, st, finalize ? offsets : offsets_in, chunk_hist,
                       E, nchunks, *place);
    return hipGetLastError();
}

hipError_t launch_place(int32_t* chunk_hist, int nchunks, int E, const int32_t* offsets, const PlaceArgs& place,
                        hipStream_t st) {
    return launch_dispatch(chunk_hist, nchunks, E, offsets, false, nullptr, nullptr, -1, nullptr, nullptr, nullptr, nullptr, &place,
                           st);
}

// routing followed by the finalize step; one kernel does both for decoder-sized layers
hipError_t launch_route_finalize(const moe_shape& s, const void* x, const void* w_gate, const float* bias,
                                 int32_t* idx, float* gate, float* margin, int32_t* hist_ws, float* gate_part_ws,
                                 int32_t* counts, int32_t* offsets, int H, uint8_t* hot_mask, uint8_t* mask_copy,
                                 const uint8_t* mask_in, const TileLists* lists, const PlaceArgs* place, hipStream_t st) {
    int nchunks = 0;
    if (s.T > 0) {
        const int tok = route_chunk_tokens(s);
        nchunks = (s.T + tok - 1) / tok;
        if (route_is_split(s) && gate_part_ws != nullptr && s.E <= kTopkFinalizeMaxE) {
            const int Tpad = (s.T + 15) / 16 * 16;
            hipError_t err = launch_gate_partial(s, x, w_gate, gate_part_ws, st);
            if (err != hipSuccess) return err;
            // at most kTopkFinalizeLdsMax: the limit configure_route_kernels has raised this kernel to
            const size_t lds = static_cast<size_t>(64) * (s.E + 1) * 4 + static_cast<size_t>(4) * s.E * 4 + static_cast<size_t>(64) * s.k * 4;
            const TileLists none{nullptr, nullptr, nullptr, nullptr, nullptr, 16, 0, 0, 0, 0, 0, 1, false};
            const PlaceArgs no_place{nullptr, nullptr, nullptr, nullptr, 0, 1, 1};
            hipLaunchKernelGGL(route_topk_finalize_kernel, dim3(1), dim3(1024), lds, st, gate_part_ws, bias, idx, gate,
                               margin, s.T, s.E, s.k, s.renormalize, Tpad, counts, offsets, H, hot_mask, mask_copy,
                               mask_in, lists ? *lists : none, lists ? 1 : 0, place ? *place : no_place);
            return hipGetLastError();
        }
        hipError_t err = launch_route_fused(s, x, w_gate, bias, idx, gate, margin, hist_ws, gate_part_ws, st);
        if (err != hipSuccess) return err;
    }
    return launch_dispatch(hist_ws, nchunks, s.E, nullptr, true, counts, offsets, H, hot_mask, mask_copy, mask_in, lists, place, st);
}

hipError_t launch_route(const moe_shape& s, const void* x, const void* w_gate, const float* bias,
                        int32_t* idx, float* gate, float* margin, int32_t* counts,
                        int32_t* offsets, int32_t H, uint8_t* hot_mask, int32_t* hist_ws, float* gate_part_ws,
                        hipStream_t st) {
    return launch_route_finalize(s, x, w_gate, bias, idx, gate, margin, hist_ws, gate_part_ws, counts, offsets, H, hot_mask,
                                 nullptr, nullptr, nullptr, nullptr, st);
}

}  // namespace moe
