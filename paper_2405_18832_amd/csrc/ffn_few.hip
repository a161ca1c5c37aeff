// Layers of few tokens (decoder steps of one or a few sentences; layer_is_few): routing, both products and the combine in three
// launches instead of five.  Such a step is a chain of short kernels around two streams of weights; a launch that moves almost
// nothing costs its own latency and about 1.7 us between the kernels.
//
//   gate_partial_kernel (route.hip)   partial logits
//   few_first_kernel                  every block works out the routing of all the tokens for itself (logits, softmax, top-k: the
//                                     same arithmetic on the same values), then streams its share of the first product
//   few_second_kernel                 a block owns 8 output columns of all experts and adds up the tokens' outputs itself
//
// One token, 128 experts, k = 2, 2048 x 8192: 36.4 -> 32.9 us a step; k = 1, 768 x 3072: 23.1 -> 14.2 us.
#include <algorithm>

#include "stream_unit.hpp"
#include "topk.hpp"

namespace moe {

constexpr int kFewTokens = 8;
constexpr int kFewAssignments = 20;     // at most a lane each
constexpr int kFewExperts = 256;        // a thread each in few_first_kernel
constexpr int kFewRows = 8;             // rows of a tile: an expert has more only if a token (of NaN logits) names it twice

// The assignments in expert order: tiles of up to kFewRows rows, the place of every assignment, the token of every place.
struct FewLists {
    Tile tiles[kFewAssignments];
    int place[kFewAssignments];
    int token[kFewAssignments];
    int ntiles;
};

// Called by one whole wavefront; lane a < A holds the expert of assignment a.
__device__ __forceinline__ void few_lists(int e, int A, int k, FewLists* l) {
    const int a = threadIdx.x & 63;
    int less = 0, before = 0, same = 0;
    for (int b = 0; b < A; ++b) {
        const int eb = __builtin_amdgcn_readlane(e, b);
        less += eb < e ? 1 : 0;
        same += eb == e ? 1 : 0;
        before += (eb == e && b < a) ? 1 : 0;
    }
    const bool first = a < A && before % kFewRows == 0;
    const uint64_t firsts = __ballot(first);
    int t = 0;
    for (uint64_t m = firsts; m != 0; m &= m - 1) {        // wave-uniform
        const int b = __builtin_ctzll(m), eb = __builtin_amdgcn_readlane(e, b);
        t += (eb < e || (eb == e && b < a)) ? 1 : 0;
    }
    if (first) l->tiles[t] = Tile{e, less + before, min(kFewRows, same - before), 0};
    if (a < A) {
        l->place[a] = less + before;
        l->token[less + before] = a / k;
    }
    if (a == 0) l->ntiles = __popcll(firsts);
}

struct FewRoute {
    const float* part;         // [kGateSplit][Tpad][E] partial logits
    const float* bias;
    int32_t* idx;
    float* gate;
    int32_t* counts;
    int32_t* offsets;
    int32_t* perm;             // may be NULL
    int32_t* inv_perm;
    int32_t* tokmap;
    int T, E, k, renorm, Tpad;
};

// First product.  A unit is 64 columns of a tile, or 16 where those are fewer than the CUs; the four wavefronts split the
// contraction.  Block 0 writes the routing's outputs and takes the last unit of a round: one that is there only where the grid is
// all the blocks that fit (without it 511 blocks share 512 units, or 1024, and wait for one or two of them: layers of 4 tokens,
// k = 1, 2048 x 8192, 54.6 -> 52.7 us; k = 2, 1024 x 4096, 34.6 -> 33.5).
template <int FIRST>
__global__ __launch_bounds__(256, 2) void few_first_kernel(const FewRoute p, const uint16_t* __restrict__ x,
                                                        const uint16_t* __restrict__ w1, uint16_t* __restrict__ h,
                                                        const float* __restrict__ b1, int N, int K, int cus) {
    __shared__ f32x4 red[3 * 4 * 64];
    __shared__ float logits[kFewTokens * (kFewExperts + 1)];
    __shared__ int32_t hist[kFewExperts];
    __shared__ int32_t experts[kFewAssignments];
    __shared__ float weights[kFewAssignments];
    __shared__ FewLists lists;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int T = p.T, E = p.E, k = p.k, A = T * k, Ep = E + 1;
    hist[threadIdx.x] = 0;
    // four logits per thread and pass, their partial sums loaded before any is added
    for (int i0 = threadIdx.x; i0 < T * E; i0 += 4 * 256) {
        float v[4][kGateSplit], b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = min(i0 + u * 256, T * E - 1);    // past the end: re-read, not stored
            const int t = i / E, e = i - t * E;
            b[u] = p.bias ? p.bias[e] : 0.f;
#pragma unroll
            for (int ks = 0; ks < kGateSplit; ++ks) v[u][ks] = p.part[(static_cast<size_t>(ks) * p.Tpad + t) * E + e];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * 256;
            if (i >= T * E) break;
            const int t = i / E, e = i - t * E;
            float sum = b[u];
#pragma unroll
            for (int ks = 0; ks < kGateSplit; ++ks) sum += v[u][ks];          // fixed order
            logits[t * Ep + e] = sum;
        }
    }
    __syncthreads();
    if (wave * 4 < T) {                                    // wave-uniform: 16 lanes per token
        const int t = wave * 4 + (lane >> 4);
        const bool live = t < T;
        const int o = live ? t * k : 0;
        topk_from_lds(logits + t * Ep, E, k, p.renorm, lane & 15, live, experts + o, weights + o, nullptr, hist);
    }
    __syncthreads();
    if (wave == 0) few_lists(lane < A ? experts[lane] : 0x7fffffff, A, k, &lists);
    __syncthreads();

    if (blockIdx.x == 0) {                                   // the routing's outputs
        const int e = threadIdx.x;
        int before = 0;
        for (int a = 0; a < A; ++a) before += experts[a] < e ? 1 : 0;
        if (e < E) {
            p.counts[e] = hist[e];
            p.offsets[e] = before;
        }
        if (e == 0) p.offsets[E] = A;
        if (e < A) {
            const int at = lists.place[e];
            p.idx[e] = experts[e];
            p.gate[e] = weights[e];
            if (p.perm != nullptr) p.perm[at] = e;
            p.inv_perm[e] = at;
            p.tokmap[at] = e / k;
        }
    }
    const int nblk = N >> 4, kblk = K >> 5, ngroups = (nblk + 3) >> 2;
    const int kb0 = kblk * wave / 4, kb1 = kblk * (wave + 1) / 4;
    const int grid = static_cast<int>(gridDim.x), first = blockIdx.x == 0 ? grid - 1 : static_cast<int>(blockIdx.x) - 1;
    const FoldOut none{nullptr, nullptr, nullptr};
    if (lists.ntiles * ngroups >= cus) {                   // uniform
        for (int u = first; u < lists.ntiles * ngroups; u += grid)
            stream_unit<1, 1, 4, FIRST, false, 4>(x, lists.token, w1, h, lists.tiles[u / ngroups], u % ngroups, true, N, K, kb0, kb1,
                                                  red, false, b1, none, wave);
    } else {
        for (int u = first; u < lists.ntiles * nblk; u += grid)
            stream_unit<1, 1, 4, FIRST, false, 1>(x, lists.token, w1, h, lists.tiles[u / nblk], u % nblk, true, N, K, kb0, kb1, red,
                                                  false, b1, none, wave);
    }
}

// Second product and combine.  A block owns 8 columns, half of a packed fragment, so that a 2048-wide layer has a block for every
// CU (128 blocks of 16 columns would be bound by the 35 GB/s that one CU pulls in).  One load takes that half of two consecutive
// k-steps: operand rows 0 - 7 are the columns at the first of them, rows 8 - 15 the same columns at the second, and the other
// operand's 16 columns are the tile's 8 rows at the one and at the other; the products wanted are the two diagonal quarters.
// The eight wavefronts split the contraction and walk through all the tiles without a barrier; their sums of every row meet in
// LDS at the end.
constexpr int kFewWaves = 8;
constexpr int kFewAhead = 8;            // KiB of weights in flight per wavefront
__global__ __launch_bounds__(kFewWaves * 64) void few_second_kernel(const uint16_t* __restrict__ h, const uint16_t* __restrict__ w2,
                                                                    const int32_t* __restrict__ idx,
                                                                    const float* __restrict__ gate,
                                                                    const float* __restrict__ b2, uint16_t* __restrict__ out,
                                                                    int T, int E, int k, int N, int K) {
    __shared__ FewLists lists;
    // [wavefront][row][k-step of a pair][column]; written 16 bytes at a time
    __shared__ __attribute__((aligned(16))) float sums[kFewWaves][kFewAssignments][2][8];
    static_assert(__alignof__(sums) >= alignof(f32x4), "stored as f32x4");
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const int A = T * k, nblk = N >> 4, kblk = K >> 5;
    __shared__ int32_t experts[kFewAssignments];
    __shared__ float weights[kFewAssignments];
    if (wave == 0) {
        const int e = lane < A ? min(max(idx[lane], 0), E - 1) : 0x7fffffff;
        if (lane < A) {
            experts[lane] = e;
            weights[lane] = gate[lane];
        }
        few_lists(e, A, k, &lists);
    }
    __syncthreads();
    const int ntiles = __builtin_amdgcn_readfirstlane(lists.ntiles);

    const int pairs = (kblk + 1) >> 1;                     // pairs of k-steps; the second of the last one may not exist
    const int p0 = pairs * wave / kFewWaves, per = pairs * (wave + 1) / kFewWaves - p0;
    const int nb = blockIdx.x >> 1, half = blockIdx.x & 1, sub = r & 7, odd = r >> 3;
    const int total = ntiles * per;
    // load position: pair `ip` of tile `it`
    int it = 0, ip = 0;
    const uint16_t *wp, *hp;
    auto point_at = [&](int t) {
        const int expert = __builtin_amdgcn_readfirstlane(lists.tiles[t].expert);
        const int row = lists.tiles[t].row0 + min(sub, lists.tiles[t].rows - 1);
        wp = w2 + (static_cast<size_t>(expert) * nblk + nb) * kblk * 512 + (g * 16 + half * 8 + sub) * 8;
        hp = h + static_cast<size_t>(row) * 32 + g * 8;    // few rows: all in the first row block
    };
    bf16x8 a[kFewAhead], b[kFewAhead];
    auto issue = [&](int slot) {
        const int kb = 2 * (p0 + ip) + odd, at = min(kb, kblk - 1);
        a[slot] = *reinterpret_cast<const bf16x8*>(wp + static_cast<size_t>(at) * 512);
        b[slot] = *reinterpret_cast<const bf16x8*>(hp + static_cast<size_t>(at) * kStepStride);
        if (ip + 1 < per) {
            ++ip;
        } else if (it + 1 < ntiles) {                      // past the end the last pair is read again, not used
            ip = 0;
            point_at(++it);
        }
    };
    if (per > 0) {
        point_at(0);
#pragma unroll
        for (int s = 0; s < kFewAhead; ++s) issue(s);
        int t = 0, left = per;
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int q0 = 0; q0 < total; q0 += kFewAhead) {
#pragma unroll
            for (int s = 0; s < kFewAhead; ++s) {
                if (q0 + s >= total) break;                // wave-uniform
                const bool cut = (kblk & 1) != 0 && p0 + per == pairs && left == 1;      // uniform: a pair without its second step
                bf16x8 va = a[s], vb = b[s];
                if (cut && odd != 0) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) va[i] = vb[i] = 0.f;
                }
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, vb, acc, 0, 0, 0);
                issue(s);
                if (--left == 0) {                         // lane (r, g) holds operand rows 4g ... 4g + 3 of operand column r
                    const int row = lists.tiles[t].row0 + sub;
                    if (odd == g >> 1 && sub < lists.tiles[t].rows)
                        *reinterpret_cast<f32x4*>(&sums[wave][row][odd][(g & 1) * 4]) = acc;
                    acc = f32x4{0.f, 0.f, 0.f, 0.f};
                    left = per;
                    ++t;
                }
            }
        }
    }
    __syncthreads();
    // wavefronts without a pair have left nothing (short contractions)
    for (int i = threadIdx.x; i < T * 8; i += kFewWaves * 64) {
        const int t = i >> 3, c = i & 7, n = blockIdx.x * 8 + c;
        float o = 0.f;
        for (int j = 0; j < k; ++j) {                      // in slot order
            const int at = lists.place[t * k + j];
            float y = 0.f;
#pragma unroll
            for (int w = 0; w < kFewWaves; ++w)
                if (pairs * (w + 1) / kFewWaves > pairs * w / kFewWaves) y += sums[w][at][0][c] + sums[w][at][1][c];
            if (b2 != nullptr) y += b2[static_cast<size_t>(experts[t * k + j]) * N + n];
            o = fmaf(weights[t * k + j], y, o);
        }
        out[static_cast<size_t>(t) * N + n] = f32_to_bf16(o);
    }
}

// units of the first product if all tiles are of different experts
struct FewUnits {
    long count;
    int columns;
};
static FewUnits few_units(const moe_shape& s, int tiles, int cus) {
    const long wide = static_cast<long>(tiles) * ((s.d_ff / 16 + 3) / 4);
    if (wide >= cus) return {wide, 64};
    return {static_cast<long>(tiles) * (s.d_ff / 16), 16};
}

// Layers that this is faster for than the general path.  It saves two launches, or three (k > 1), 5 to 9 us.  What it may lose, from
// the 35 GB/s that a CU pulls in and the 5.5 TB/s of the chip:
//  - a block of the second product streams 8 columns of every tile, however few blocks d_model gives; the general path's units are
//    over the whole chip.  Up to 2.8 us of it are no matter.  Blocks that share a CU (d_model above 8 per CU) are worth it up to 4 us;
//  - the first product's units, where there are many and a little more than a whole number per CU;
//  - tiles are one after the other in the second product.
// And the first product has to be less than one and a half rounds of units with a whole contraction per wavefront: past that the
// general path streams as fast or faster (from two rounds on with its rows in LDS).
// us, general and this, taken: 1 token, 2048 x 8192, k = 2 36.4 and 32.9; 1 token, 1024 x 4096 23.7 and 14.8; 4 tokens, 2048 x 8192, k = 2
// 97.3 and 93.7; 8 tokens, 768 x 3072 28.5 and 26.6.  Not taken: 8 tokens, 512 x 2048, k = 2 25.4 and 27.5; 8 tokens, 256 x 1024, k = 8
// 38.0 and 60.7; 5 tokens, 256 x 8192, k = 2 33.5 and 52.2; 3 tokens, 4096 x 16384 152 and 169.  Of 1100 layers of 64 to 8192
// columns drawn at random after the line was set, none takes more than 1.015 of the general path's time (half a microsecond).
bool layer_is_few(const moe_shape& s) {
    if (s.dtype != MOE_BF16 || s.T < 1 || s.T > kFewTokens || s.T * s.k > kFewAssignments || s.E > kFewExperts) return false;
    const int cus = device_cu_count(), tiles = std::min(s.T * s.k, s.E);
    if (2L * tiles * ((s.d_ff / 64 + 3) / 4) >= 3L * cus) return false;
    constexpr double kCuRate = 35e3, kChipRate = 5.5e6;    // bytes per us
    const double block = tiles * 16.0 * s.d_ff / kCuRate;
    if (block <= 2.8) return true;
    if (s.d_model > 8 * cus) return block <= 4.;
    double loss = block - tiles * 2.0 * s.d_model * s.d_ff / kChipRate;
    const FewUnits u = few_units(s, tiles, cus);
    const double uneven = ((u.count + cus - 1) / cus - static_cast<double>(u.count) / cus) * u.columns * 2.0 * s.d_model / kCuRate;
    if (tiles > 6 && uneven >= 2.) loss += tiles > 8 ? uneven : uneven / 2;
    if (tiles > 8) loss += 0.1 * (tiles - 8);
    return loss <= 4.4;
}

hipError_t launch_few_products(const moe_shape& s, const void* x, const float* gate_bias, const float* gate_part, const void* w1,
                               const void* w2, const float* b1, const float* b2, int32_t* idx, float* gate, int32_t* counts,
                               int32_t* offsets, int32_t* perm, int32_t* inv_perm, int32_t* tokmap, void* h, void* out,
                               hipStream_t st) {
    const int Tpad = (s.T + 15) / 16 * 16, cus = device_cu_count();
    const FewRoute p{gate_part, gate_bias, idx, gate, counts, offsets, perm, inv_perm, tokmap, s.T, s.E, s.k, s.renormalize, Tpad};
    const FewUnits units = few_units(s, std::min(s.T * s.k, s.E), cus);
    const unsigned grid = static_cast<unsigned>(std::min(units.count + 1, 2L * cus));     // two blocks fit a CU
    hipError_t err;
    if ((err = mark_profile_event(0, st)) != hipSuccess || (err = mark_profile_event(1, st)) != hipSuccess) return err;
    auto first = s.activation == MOE_ACT_GELU ? few_first_kernel<kFirstGelu> : few_first_kernel<kFirstRelu>;
    hipLaunchKernelGGL(first, dim3(grid), dim3(256), 0, st, p, static_cast<const uint16_t*>(x), static_cast<const uint16_t*>(w1),
                       static_cast<uint16_t*>(h), b1, s.d_ff, s.d_model, cus);
    if ((err = hipGetLastError()) != hipSuccess) return err;
    if ((err = mark_profile_event(2, st)) != hipSuccess || (err = mark_profile_event(3, st)) != hipSuccess) return err;
    hipLaunchKernelGGL(few_second_kernel, dim3(static_cast<unsigned>(s.d_model / 8)), dim3(kFewWaves * 64), 0, st,
                       static_cast<const uint16_t*>(h), static_cast<const uint16_t*>(w2), idx, gate, b2,
                       static_cast<uint16_t*>(out), s.T, s.E, s.k, s.d_model, s.d_ff);
    if ((err = hipGetLastError()) != hipSuccess) return err;
    return mark_profile_event(4, st);
}

}  // namespace moe
