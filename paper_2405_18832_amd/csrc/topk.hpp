// Softmax and top-k of token rows whose logits lie in LDS, used by the routing kernels and by the first product of layers of
// few tokens.
#pragma once
#include "common.hpp"

namespace moe {

#ifdef __HIPCC__
static_assert(MOE_MAX_K + 1 <= 16, "a token's winners sit in the 16 lanes of its group");

// Value of the lane n places away inside the lane's row of 16 (a DPP row rotation, no LDS traffic).  Four
// steps with n = 8, 4, 2, 1 leave every lane of the row with the reduction over the row; for sums the
// operand pairs are those of the xor butterfly (after a step with n the values have period n in the row).
template <int N>
__device__ __forceinline__ float row_rot(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + N, 0xF, 0xF, false));
}
template <int N>
__device__ __forceinline__ int row_rot(int v) {
    return __builtin_amdgcn_update_dpp(0, v, 0x120 + N, 0xF, 0xF, false);
}

// ---------------------------------------------------------------------------
// top-k of one token from its logits row in LDS, by a group of 16 lanes (4 tokens per wave).
// k rounds (k + 1 when the margin is wanted) of a (value, index) arg-max; on equal values the
// lower index wins, in the lane-local scan and in every exchange, so the order is "descending
// logit, ties by lowest expert index".  A winner is retired by setting its logit to -inf.
// ---------------------------------------------------------------------------
// V > 0: the row has at most 16 * V experts and the lane keeps its V logits (experts sub, sub + 16, ...) in
// registers for all rounds; V == 0: any E, the row is read from LDS in every round and a winner is retired by
// overwriting its logit there.  (Every LDS read in the per-round loops is a round trip the next compare waits
// for: with the row in registers the top-k of a 64-token chunk of 128 experts takes a third of the time.)
template <int V>
__device__ __forceinline__ void topk_row(float* __restrict__ row, int E, int k, int renorm, int sub, bool live,
                                         int32_t* __restrict__ idx_out, float* __restrict__ w_out,
                                         float* __restrict__ margin_out, int32_t* __restrict__ hist,
                                         int32_t* __restrict__ idx_lds) {
    const float NEG = -__builtin_huge_valf();
    float sel_v = NEG;                    // lane j of the group keeps the winner of round j
    int sel_i = 0;
    const int rounds = min(k + (margin_out != nullptr ? 1 : 0), E);   // the margin needs one more winner
    float vmax = 0.f, denom = 1.f;
    float v[V > 0 ? V : 1];
    if constexpr (V > 0) {
#pragma unroll
        for (int q = 0; q < V; ++q) v[q] = (sub + 16 * q < E) ? row[sub + 16 * q] : NEG;
    }
#pragma unroll 1
    for (int j = 0; j < rounds; ++j) {
        float bv = NEG;
        int bi = 0x7fffffff;
        if constexpr (V > 0) {
#pragma unroll
            for (int q = 0; q < V; ++q) {
                const int e = sub + 16 * q;
                if (e < E && (v[q] > bv || bi == 0x7fffffff)) { bv = v[q]; bi = e; }
            }
        } else {
            for (int e = sub; e < E; e += 16) {
                const float x = row[e];
                if (x > bv || bi == 0x7fffffff) { bv = x; bi = e; }
            }
        }
        auto better = [&](float ov, int oi) {
            if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
        };
        better(row_rot<8>(bv), row_rot<8>(bi));
        better(row_rot<4>(bv), row_rot<4>(bi));
        better(row_rot<2>(bv), row_rot<2>(bi));
        better(row_rot<1>(bv), row_rot<1>(bi));
        bi = min(bi, E - 1);          // NaN logits must not produce an out-of-range expert
        if constexpr (V == 0) {       // lanes that hold a NaN see another winner: the first lane's counts, which retires it below
            bv = __shfl(bv, 0, 16);
            bi = __shfl(bi, 0, 16);
        }
        if (j == 0) {
            vmax = bv;
            float part = 0.f;
            if constexpr (V > 0) {
#pragma unroll
                for (int q = 0; q < V; ++q)
                    if (sub + 16 * q < E) part += expf(v[q] - vmax);
            } else {
                for (int e = sub; e < E; e += 16) part += expf(row[e] - vmax);
            }
            part += row_rot<8>(part);
            part += row_rot<4>(part);
            part += row_rot<2>(part);
            part += row_rot<1>(part);
            denom = part;
        }
        if (sub == j) { sel_v = bv; sel_i = bi; }
        if constexpr (V > 0) {
#pragma unroll
            for (int q = 0; q < V; ++q)
                if (sub + 16 * q == bi) v[q] = NEG;
        } else {
            if (sub == 0) row[bi] = NEG;
            __builtin_amdgcn_wave_barrier();
        }
    }
    // Lane j finishes winner j: one exponential and one division each, side by side (one lane doing all k of them, unrolled
    // to MOE_MAX_K, was most of the kernel's code, which a short kernel fetches cold).
    const float p = expf(sel_v - vmax) / denom;
    float psum = 0.f;
    if (renorm) {
#pragma unroll 1
        for (int j = 0; j < k; ++j) psum += __shfl(p, j, 16);          // in slot order
    }
    if (live && sub < k) {
        idx_out[sub] = sel_i;
        if (idx_lds != nullptr) idx_lds[sub] = sel_i;
        w_out[sub] = renorm ? p / psum : p;
        atomicAdd(&hist[sel_i], 1);                                    // LDS, integer: order does not matter
    }
    if (margin_out != nullptr) {                                       // uniform
        const float next = __shfl_down(sel_v, 1, 16);
        float m = sub + 1 < rounds ? sel_v - next : __builtin_huge_valf();
        m = fminf(m, row_rot<8>(m));
        m = fminf(m, row_rot<4>(m));
        m = fminf(m, row_rot<2>(m));
        m = fminf(m, row_rot<1>(m));
        if (live && sub == 0) *margin_out = m;
    }
}

// called by whole wavefronts; E is uniform
__device__ __forceinline__ void topk_from_lds(float* __restrict__ row, int E, int k, int renorm, int sub,
                                              bool live, int32_t* __restrict__ idx_out,
                                              float* __restrict__ w_out, float* __restrict__ margin_out,
                                              int32_t* __restrict__ hist, int32_t* __restrict__ idx_lds = nullptr) {
    if (E <= 64) topk_row<4>(row, E, k, renorm, sub, live, idx_out, w_out, margin_out, hist, idx_lds);
    else if (E <= 128) topk_row<8>(row, E, k, renorm, sub, live, idx_out, w_out, margin_out, hist, idx_lds);
    else if (E <= 256) topk_row<16>(row, E, k, renorm, sub, live, idx_out, w_out, margin_out, hist, idx_lds);
    else topk_row<0>(row, E, k, renorm, sub, live, idx_out, w_out, margin_out, hist, idx_lds);
}
#endif

}  // namespace moe
