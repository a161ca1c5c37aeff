// Expert FFNs as a grouped product over variable token counts:
//   y_perm[rows of e] = relu(x_perm[rows of e] . W1_e^T) . W2_e^T        for every active expert e
// (paper Section 2.1: an expert is two linear layers with an activation between; Sections 3.1
// and 3.4: each is C = A x B, the first with a trailing ReLU).  The paper's observation that
// most experts receive very few tokens, so that their cost is reading their parameters
// (Section 2.2), is what shapes the kernel below: it streams every active expert's weights
// exactly once at full memory bandwidth while the few token rows ride along as the other MFMA
// operand.
#include <algorithm>

#include "stream_unit.hpp"

namespace moe {

// ---------------------------------------------------------------------------
// weight packing: [E][N][K] row-major  ->  [E][N/16][K/32] fragments of 64 lanes x 8 elements.
// One thread per 16-byte piece of the destination.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void pack_bf16_kernel(const uint4* __restrict__ src,
                                                        uint4* __restrict__ dst, int N, int K,
                                                        size_t total) {
    const size_t c = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (c >= total) return;
    const size_t per_expert = static_cast<size_t>(N) * K / 8;
    const size_t e = c / per_expert, ce = c % per_expert;
    const int kblk = K / 32;
    const size_t frag = ce / 64;
    const int l = static_cast<int>(ce % 64);
    const int nb = static_cast<int>(frag / kblk), kb = static_cast<int>(frag % kblk);
    const int n = nb * 16 + (l & 15), kk = kb * 32 + (l >> 4) * 8;
    dst[c] = src[(e * N + n) * (K / 8) + kk / 8];
}

__global__ __launch_bounds__(256) void copy_u32_kernel(const uint32_t* __restrict__ src,
                                                       uint32_t* __restrict__ dst, size_t total) {
    const size_t c = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (c < total) dst[c] = src[c];
}

hipError_t launch_pack(const moe_shape& s, int which, const void* src, void* dst, hipStream_t st) {
    const int N = which == 1 ? s.d_ff : s.d_model, K = which == 1 ? s.d_model : s.d_ff;
    if (s.dtype == MOE_BF16) {
        const size_t total = static_cast<size_t>(s.E) * N * K / 8;
        hipLaunchKernelGGL(pack_bf16_kernel, dim3(static_cast<unsigned>((total + 255) / 256)), dim3(256), 0,
                           st, static_cast<const uint4*>(src), static_cast<uint4*>(dst), N, K, total);
    } else {
        const size_t total = static_cast<size_t>(s.E) * N * K;
        hipLaunchKernelGGL(copy_u32_kernel, dim3(static_cast<unsigned>((total + 255) / 256)), dim3(256), 0,
                           st, static_cast<const uint32_t*>(src), static_cast<uint32_t*>(dst), total);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// tile lists from caller-supplied offsets (the stand-alone expert-FFN call): every active,
// masked-in expert's row segment cut into row tiles.  One block, one thread per expert.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void build_tiles_kernel(const int32_t* __restrict__ offsets,
                                                           const uint8_t* __restrict__ mask, int E, int A,
                                                           const TileLists lists) {
    __shared__ int32_t scan[kScanInts];
    const int e = threadIdx.x;
    int row0 = 0, m = 0;
    bool bad = false;
    if (e < E) {
        row0 = offsets[e];
        m = offsets[e + 1] - row0;
        bad = row0 < 0 || m < 0 || row0 + m > A;
        if (mask != nullptr && mask[e] == 0) m = 0;
    }
    // Offsets that are not prefix sums (a negative count anywhere, a segment outside [0, A]): run nothing at all.
    // With every count >= 0 the segments are disjoint and their sum is at most A, which is what the capacity of
    // the tile lists assumes.
    if (__syncthreads_or(bad ? 1 : 0)) m = 0;
    const int v[2] = {big_tiles_at_min(m, lists), half_tiles_joined(m, lists)};
    int incl[2], total[2];
    block_scan(v, incl, total, scan, (E + 63) >> 6);
    emit_tiles(e, E, row0, m, total[0], total[1], lists, scan + 48);
}

template <int TFMAX, int KSPLIT, int FIRST, bool FOLD>
__global__ __launch_bounds__(256) void ffn_stream_kernel(const uint16_t* __restrict__ act,
                                                         const int32_t* __restrict__ rowmap,
                                                         const uint16_t* __restrict__ wpk,
                                                         void* __restrict__ outp,
                                                         const Tile* __restrict__ tiles,
                                                         const int32_t* __restrict__ ntiles_p, int N,
                                                         int K, int balance,
                                                         int act_kmajor, int rows_in_lds,
                                                         const float* __restrict__ bias, const FoldOut fold) {
    extern __shared__ __attribute__((aligned(16))) unsigned char tok_lds[];
    constexpr int NGB = 4 / KSPLIT;   // n-groups (of 64 columns) per block
    __shared__ f32x4 red[KSPLIT > 1 ? (KSPLIT - 1) * NGB * 4 * TFMAX * 64 : 1];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ks = wave % KSPLIT, ngs = wave / KSPLIT;
    const int nblk = N >> 4, kblk = K >> 5;
    const int ngroups = (nblk + 3) >> 2;
    const int ngchunks = (ngroups + NGB - 1) / NGB;
    const int kb_per = (kblk + KSPLIT - 1) / KSPLIT;
    const int kb0 = min(kblk, ks * kb_per), kb1 = min(kblk, kb0 + kb_per);
    const int nbu = ntiles_p[0] * ngchunks;
    int stride = gridDim.x;
    if (balance) {
        // Units are equal-sized, so a grid that does not divide them ends with a round of few blocks and
        // little data in flight.  Use only as many blocks as make every block run the same number of
        // units (the others exit): the memory system sees a constant number of streams to the end.
        const int rounds = (nbu + stride - 1) / stride;
        if (rounds > 0) stride = (nbu + rounds - 1) / rounds;
        if (static_cast<int>(blockIdx.x) >= stride) return;
    }
    // Blocks go to the 8 XCDs round-robin and each XCD has its own L2: give the blocks of one XCD
    // consecutive units, i.e. the column groups of the same tile, so that the tile's activation rows are
    // fetched into that L2 once instead of into all eight.
    const int pb = (stride % 8 == 0) ? static_cast<int>(blockIdx.x & 7) * (stride >> 3) + static_cast<int>(blockIdx.x >> 3)
                                     : static_cast<int>(blockIdx.x);
    for (int base = 0; base < nbu; base += stride) {
        const int bu = base + pb;
        if (bu >= nbu) break;                             // block-uniform
        const Tile tl = tiles[bu / ngchunks];
        const int ng = (bu % ngchunks) * NGB + ngs;
        const bool active = ng < ngroups;                 // wave-uniform
        const int tfc = (tl.rows + 15) >> 4;              // token fragments in use: block-uniform
        if (KSPLIT == 1 && rows_in_lds) {
            const bool km = act_kmajor != 0;
            if (TFMAX >= 4 && tfc == 4)
                stream_unit_lds<4, FIRST, FOLD>(act, rowmap, wpk, outp, tl, ng, active, N, K, km, bias, tok_lds, fold, wave);
            else if (TFMAX >= 4 && tfc == 3)
                stream_unit_lds<3, FIRST, FOLD>(act, rowmap, wpk, outp, tl, ng, active, N, K, km, bias, tok_lds, fold, wave);
            else if (TFMAX >= 2 && tfc == 2)
                stream_unit_lds<2, FIRST, FOLD>(act, rowmap, wpk, outp, tl, ng, active, N, K, km, bias, tok_lds, fold, wave);
            else
                stream_unit_lds<1, FIRST, FOLD>(act, rowmap, wpk, outp, tl, ng, active, N, K, km, bias, tok_lds, fold, wave);
            continue;
        }
        if (TFMAX >= 4 && tfc == 4)
            stream_unit<4, TFMAX, KSPLIT, FIRST, FOLD>(act, rowmap, wpk, outp, tl, ng, active, N, K, kb0, kb1, red, act_kmajor != 0, bias, fold, wave);
        else if (TFMAX >= 4 && tfc == 3)
            stream_unit<3, TFMAX, KSPLIT, FIRST, FOLD>(act, rowmap, wpk, outp, tl, ng, active, N, K, kb0, kb1, red, act_kmajor != 0, bias, fold, wave);
        else if (TFMAX >= 2 && tfc == 2)
            stream_unit<2, TFMAX, KSPLIT, FIRST, FOLD>(act, rowmap, wpk, outp, tl, ng, active, N, K, kb0, kb1, red, act_kmajor != 0, bias, fold, wave);
        else
            stream_unit<1, TFMAX, KSPLIT, FIRST, FOLD>(act, rowmap, wpk, outp, tl, ng, active, N, K, kb0, kb1, red, act_kmajor != 0, bias, fold, wave);
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// per device, written once by configure_ffn_kernels (under the set-up lock) before any launch reads them
static int g_cus[kMaxDevices] = {0};

int device_cu_count() {
    const int n = g_cus[current_device_index()];
    return n > 0 ? n : 256;
}

// resident blocks per CU that the registers of a weight-streaming kernel allow, per device
template <int TFMAX, int KSPLIT, int FIRST, bool FOLD>
struct StreamKernelInfo {
    static int per_cu[kMaxDevices];
};
template <int TFMAX, int KSPLIT, int FIRST, bool FOLD>
int StreamKernelInfo<TFMAX, KSPLIT, FIRST, FOLD>::per_cu[kMaxDevices] = {0};

// Second product of a layer of at most 16 tokens when its experts are so few that groups of 64 columns leave
// most CUs without a unit (one token with two experts, 2048 columns: 64 units): a unit is one 16-column block, the
// four wavefronts of a block split the contraction as usual and keep 16 KiB-steps of weights in flight each.  Layers of few
// tokens without a mask go to ffn_few.hip instead where that is faster; what comes here has a mask, is called step by step, or has
// more tokens, experts or bytes per column than pay there.
__global__ __launch_bounds__(256) void ffn_stream_narrow_kernel(const uint16_t* __restrict__ act,
                                                                const uint16_t* __restrict__ wpk,
                                                                void* __restrict__ outp,
                                                                const Tile* __restrict__ tiles,
                                                                const int32_t* __restrict__ ntiles_p, int N, int K,
                                                                const float* __restrict__ bias) {
    __shared__ f32x4 red[3 * 64];
    const int ks = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nblk = N >> 4, kblk = K >> 5;
    const int kb_per = (kblk + 3) / 4;
    const int kb0 = min(kblk, ks * kb_per), kb1 = min(kblk, kb0 + kb_per);
    const int nbu = ntiles_p[0] * nblk;
    // as in ffn_stream_kernel: every block that runs gets the same number of units, and the blocks of an XCD
    // take consecutive units
    int stride = gridDim.x;
    const int rounds = (nbu + stride - 1) / stride;
    if (rounds > 0) stride = (nbu + rounds - 1) / rounds;
    if (static_cast<int>(blockIdx.x) >= stride) return;
    const int pb = (stride % 8 == 0) ? static_cast<int>(blockIdx.x & 7) * (stride >> 3) + static_cast<int>(blockIdx.x >> 3)
                                     : static_cast<int>(blockIdx.x);
    const FoldOut none{nullptr, nullptr, nullptr};
    for (int base = 0; base < nbu; base += stride) {
        const int bu = base + pb;
        if (bu >= nbu) break;                             // block-uniform
        stream_unit<1, 1, 4, 0, false, 1>(act, nullptr, wpk, outp, tiles[bu / nblk], bu % nblk, true, N, K, kb0, kb1, red,
                                          true, bias, none, ks);
    }
}

template <int TFMAX, int KSPLIT, int FIRST, bool FOLD>
static hipError_t launch_stream(const uint16_t* act, const int32_t* rowmap, const uint16_t* wpk, void* outp,
                                const Tile* tiles, const int32_t* ntiles, int N, int K, long max_units,
                                bool act_kmajor, const float* bias, const FoldOut& fold, hipStream_t st) {
    auto kern = ffn_stream_kernel<TFMAX, KSPLIT, FIRST, FOLD>;
    // Tiles of more than 16 rows run as one block per CU, though the registers allow three, the smallest as two.  Layers, us, two blocks ->
    // one: 2048 x 8192, 128 experts, k = 2, 20, 40 and 127 tokens 423, 687, 1229 -> 411, 672, 1206; 1024 x 4096, 128 experts 82.0, 120.0,
    // 254.8 -> 74.0, 121.7, 247.4; 768 x 3072, 64 experts 44.2, 71.5, 115.6 -> 44.1, 73.6, 109.4; 8 experts (less than a round) the same.
    const int per_cu = std::max(1, std::min(TFMAX == 1 ? 2 : 1, StreamKernelInfo<TFMAX, KSPLIT, FIRST, FOLD>::per_cu[current_device_index()]));
    // KSPLIT = 1: the tile's rows (16 * TFMAX x K, bf16) go through LDS when they fit (the kernel's dynamic-LDS
    // limit was raised by configure_ffn_kernels)
    const size_t row_bytes = stream_row_lds(16 * TFMAX, K);
    const bool rows_in_lds = KSPLIT == 1 && row_bytes <= kStreamRowLdsMax;
    const size_t lds = rows_in_lds ? row_bytes : 0;
    // resident blocks per CU: what registers allow, and what the row tiles in LDS leave room for
    int blocks_per_cu = per_cu;
    if (lds > 0) blocks_per_cu = std::max(1, std::min(per_cu, static_cast<int>(kLdsPerCu / lds)));
    long grid = static_cast<long>(device_cu_count()) * blocks_per_cu;
    if (grid > max_units) grid = max_units;
    if (grid < 1) grid = 1;
    // decode-sized tiles (many units per block): balanced grid; larger tiles: every block stays busy
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(grid)), dim3(256), lds, st, act, rowmap, wpk, outp, tiles,
                       ntiles, N, K, TFMAX <= 2 ? 1 : 0, act_kmajor ? 1 : 0, rows_in_lds ? 1 : 0, bias, fold);
    return hipGetLastError();
}

template <int TFMAX, int FIRST, bool FOLD>
static hipError_t launch_stream_kf(int ksplit, const uint16_t* act, const int32_t* rowmap, const uint16_t* wpk,
                                   void* outp, const Tile* tiles, const int32_t* ntiles, int N, int K,
                                   long max_tiles, bool act_kmajor, const float* bias, const FoldOut& fold, hipStream_t st) {
    const long ngroups = (N / 16 + 3) / 4;
    if (ksplit == 4)
        return launch_stream<TFMAX, 4, FIRST, FOLD>(act, rowmap, wpk, outp, tiles, ntiles, N, K, max_tiles * ngroups,
                                                    act_kmajor, bias, fold, st);
    if (ksplit == 2)
        return launch_stream<TFMAX, 2, FIRST, FOLD>(act, rowmap, wpk, outp, tiles, ntiles, N, K,
                                                    max_tiles * ((ngroups + 1) / 2), act_kmajor, bias, fold, st);
    return launch_stream<TFMAX, 1, FIRST, FOLD>(act, rowmap, wpk, outp, tiles, ntiles, N, K,
                                                max_tiles * ((ngroups + 3) / 4), act_kmajor, bias, fold, st);
}

// the folded form exists for the second product only
template <int TFMAX, int FIRST>
static hipError_t launch_stream_k(int ksplit, const uint16_t* act, const int32_t* rowmap, const uint16_t* wpk,
                                  void* outp, const Tile* tiles, const int32_t* ntiles, int N, int K,
                                  long max_tiles, bool act_kmajor, const float* bias, const FoldOut& fold, hipStream_t st) {
    if constexpr (FIRST == 0) {
        if (fold.out != nullptr)
            return launch_stream_kf<TFMAX, 0, true>(ksplit, act, rowmap, wpk, outp, tiles, ntiles, N, K, max_tiles,
                                                    act_kmajor, bias, fold, st);
    }
    return launch_stream_kf<TFMAX, FIRST, false>(ksplit, act, rowmap, wpk, outp, tiles, ntiles, N, K, max_tiles,
                                                 act_kmajor, bias, fold, st);
}

template <int TFMAX, int KSPLIT, int FIRST, bool FOLD>
static hipError_t configure_stream(int dev) {
    auto kern = ffn_stream_kernel<TFMAX, KSPLIT, FIRST, FOLD>;
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kern, 256, 0) != hipSuccess || n <= 0) n = 1;
    StreamKernelInfo<TFMAX, KSPLIT, FIRST, FOLD>::per_cu[dev] = n;
    if (KSPLIT == 1)
        return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   static_cast<int>(kStreamRowLdsMax));
    return hipSuccess;
}

template <int TFMAX, int KSPLIT>
static hipError_t configure_stream_products(int dev) {
    hipError_t e;
    if ((e = configure_stream<TFMAX, KSPLIT, kFirstRelu, false>(dev)) != hipSuccess) return e;
    if ((e = configure_stream<TFMAX, KSPLIT, kFirstGelu, false>(dev)) != hipSuccess) return e;
    if ((e = configure_stream<TFMAX, KSPLIT, 0, false>(dev)) != hipSuccess) return e;
    return configure_stream<TFMAX, KSPLIT, 0, true>(dev);
}

template <int TFMAX>
static hipError_t configure_stream_splits(int dev) {
    hipError_t e;
    if ((e = configure_stream_products<TFMAX, 1>(dev)) != hipSuccess) return e;
    if ((e = configure_stream_products<TFMAX, 2>(dev)) != hipSuccess) return e;
    return configure_stream_products<TFMAX, 4>(dev);
}

hipError_t configure_ffn_kernels(int dev) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    g_cus[dev] = n;
    hipError_t e;
    if ((e = configure_stream_splits<1>(dev)) != hipSuccess) return e;
    if ((e = configure_stream_splits<2>(dev)) != hipSuccess) return e;
    return configure_stream_splits<4>(dev);
}

// Split K (k-steps of 32) over up to 4 wavefronts.  Decode-sized tiles want many short units
// (>= 16 steps each) for an even spread over the chip; tiles with several row fragments carry more
// per-unit work and keep >= 24 steps per wavefront.  Decode-sized tiles whose rows fit into LDS do not
// split at all when that still leaves two units for every CU (`tiles_expected`: about how many tiles there
// will be): a wavefront then streams its whole contraction in one go, with the rows read from LDS
// (measured on the decode preset, first product: 285 -> 257 us).
#ifndef MOE_KS4_MIN_STEPS
#define MOE_KS4_MIN_STEPS 96
#endif
#ifndef MOE_KS2_MIN_STEPS
#define MOE_KS2_MIN_STEPS 32     // (48 before: with 32 the first product of a d_model = 1024 layer with few small
#endif                           // experts spreads over twice the blocks: 21.7 -> 16.0 us on the Switch-large preset)
static int pick_ksplit(int K, int N, int tfmax, long tiles_expected) {
    const int steps = K / 32;
    if (tfmax <= 2) {
        const bool rows_fit = stream_row_lds(16 * tfmax, K) <= kStreamRowLdsMax;
        const long units_unsplit = tiles_expected * ((N / 64 + 3) / 4);
        if (rows_fit && units_unsplit >= 2L * device_cu_count()) return 1;
    }
    const int s4 = tfmax <= 2 ? 64 : MOE_KS4_MIN_STEPS, s2 = tfmax <= 2 ? 32 : MOE_KS2_MIN_STEPS;
    if (steps >= s4) return 4;
    if (steps >= s2) return 2;
    return 1;
}

// events recorded around the two products when a caller asked for them (profiling aid)
static hipEvent_t g_profile_events[5] = {nullptr, nullptr, nullptr, nullptr, nullptr};

void set_profile_events(const hipEvent_t* ev) {
    for (int i = 0; i < 5; ++i) g_profile_events[i] = ev ? ev[i] : nullptr;
}

hipError_t mark_profile_event(int i, hipStream_t st) {
    return g_profile_events[i] ? hipEventRecord(g_profile_events[i], st) : hipSuccess;
}

// token fragments per tile: an expert holds at most T rows (a token picks an expert at most once)
static int ffn_tfmax(const moe_shape& s) { return s.T <= 16 ? 1 : (s.T <= 32 ? 2 : 4); }

int ffn_tile_rows(const moe_shape& s) { return 16 * ffn_tfmax(s); }

TileLists ffn_tile_lists(const moe_shape& s, Tile* small_ws, Tile* big_ws, Tile* half_ws, int32_t* ntiles_ws,
                         float* partials_ws) {
    TileLists l;
    l.small_tiles = small_ws;
    l.big_tiles = big_ws;
    l.half_tiles = half_ws;
    l.ntiles = ntiles_ws;
    l.small_rows = ffn_tile_rows(s);
    // a large expert needs kBigMinRows rows, and an expert holds at most T rows
    l.big_min = (s.dtype == MOE_BF16 && s.T >= kBigMinRows) ? kBigMinRows : 0;
    l.partials = l.big_min > 0 ? partials_ws : nullptr;
    l.join_tiles = l.big_min > 0 ? tiled_join_tiles(s) : 0;
    l.d_model = s.d_model;
    l.d_ff = s.d_ff;
    l.cus = tile_product_grid();
    l.gelu = s.activation == MOE_ACT_GELU;
    l.join_half_tiles = tile_product_grid() / ((std::max(s.d_model, s.d_ff) + FineUnits::kCols - 1) / FineUnits::kCols);
    return l;
}

// row tiles of one full round of big units in the product with the fewer column tiles
int tiled_join_tiles(const moe_shape& s) {
    const int narrow = s.d_model < s.d_ff ? s.d_model : s.d_ff;
    const int col_tiles = (narrow + 255) / 256;
    return (tile_product_grid() + col_tiles - 1) / col_tiles;
}

// the two grouped products over existing tile lists
// The extra pass over the token rows pays once the layer is large (measured: a gain from 4 M elements of
// gathered rows on, a small loss at 1.5 M, where the launch costs more than the better-shaped loads save).
#ifndef MOE_GATHER_MIN_MELEMS
#define MOE_GATHER_MIN_MELEMS 4      // gathered elements (T * k * d_model), in units of 2^20, from which the pass pays
#endif
bool layer_gathers_kmajor(const moe_shape& s) {
    return s.dtype == MOE_BF16 && s.T >= kBigMinRows &&
           static_cast<long>(s.T) * s.k * s.d_model >= (static_cast<long>(MOE_GATHER_MIN_MELEMS) << 20);
}

hipError_t launch_expert_products(const moe_shape& s, const void* act, const int32_t* rowmap, bool act_kmajor,
                                  const void* w1, const void* w2, const float* b1, const float* b2, float* y_perm,
                                  void* h_ws, const TileLists& lists, const FoldOut& fold, hipStream_t st) {
    const int A = s.T * s.k, E = s.E, d = s.d_model, f = s.d_ff;
    const int tile_rows = lists.small_rows;
    const Tile* tiles = lists.small_tiles;
    const int32_t* ntiles = lists.ntiles;
    const long max_tiles = A / tile_rows + (E < A ? E : A);
    const bool big = lists.big_min > 0;
    hipError_t err;
    if ((err = mark_profile_event(0, st)) != hipSuccess) return err;

    if (s.dtype == MOE_F32) {
        if ((err = mark_profile_event(1, st)) != hipSuccess) return err;
        err = launch_f32_product(true, A, static_cast<const float*>(act), rowmap, static_cast<const float*>(w1),
                                 static_cast<float*>(h_ws), tiles, ntiles, max_tiles, f, d, s.activation, b1,
                                 FoldOut{nullptr, nullptr, nullptr}, st);
        if (err != hipSuccess) return err;
        if ((err = mark_profile_event(2, st)) != hipSuccess || (err = mark_profile_event(3, st)) != hipSuccess) return err;
        err = launch_f32_product(false, A, static_cast<const float*>(h_ws), nullptr, static_cast<const float*>(w2), y_perm,
                                 tiles, ntiles, max_tiles, d, f, s.activation, b2, fold, st);
        if (err != hipSuccess) return err;
        return mark_profile_event(4, st);
    }

    const uint16_t* xp = static_cast<const uint16_t*>(act);
    const uint16_t* p1 = static_cast<const uint16_t*>(w1);
    const uint16_t* p2 = static_cast<const uint16_t*>(w2);
    uint16_t* h = static_cast<uint16_t*>(h_ws);
    const long tiles_expected = A < E ? A : E;      // every assignment on its own expert, at most E of them
    const int ks1 = pick_ksplit(d, f, ffn_tfmax(s), tiles_expected), ks2 = pick_ksplit(f, d, ffn_tfmax(s), tiles_expected);
    if (big) {                                             // one kernel per product for large and small experts
        const FoldOut none{nullptr, nullptr, nullptr};
        for (const bool first : {true, false}) {
            auto run = [&](int kinds) {
                return first ? launch_tiled_product(true, ks1, xp, rowmap, p1, h, lists, f, d, act_kmajor, s.activation, b1, none, kinds, st)
                             : launch_tiled_product(false, ks2, h, nullptr, p2, y_perm, lists, d, f, true, s.activation, b2, fold, kinds, st);
            };
            const int apart = first ? 1 : 3;               // the event between the two kinds of units: a launch each
            if (g_profile_events[apart] != nullptr) {
                if ((err = run(kTiledUnits)) != hipSuccess || (err = mark_profile_event(apart, st)) != hipSuccess) return err;
                err = run(kStreamUnits);
            } else {
                err = run(kTiledUnits | kStreamUnits);
            }
            if (err != hipSuccess || (err = mark_profile_event(apart + 1, st)) != hipSuccess) return err;
        }
        return hipSuccess;
    }
    if ((err = mark_profile_event(1, st)) != hipSuccess) return err;
    const bool gelu = s.activation == MOE_ACT_GELU;
    switch (ffn_tfmax(s) * 2 + (gelu ? 1 : 0)) {
        case 2: err = launch_stream_k<1, kFirstRelu>(ks1, xp, rowmap, p1, h, tiles, ntiles, f, d, max_tiles, act_kmajor, b1, FoldOut{nullptr, nullptr, nullptr}, st); break;
        case 3: err = launch_stream_k<1, kFirstGelu>(ks1, xp, rowmap, p1, h, tiles, ntiles, f, d, max_tiles, act_kmajor, b1, FoldOut{nullptr, nullptr, nullptr}, st); break;
        case 4: err = launch_stream_k<2, kFirstRelu>(ks1, xp, rowmap, p1, h, tiles, ntiles, f, d, max_tiles, act_kmajor, b1, FoldOut{nullptr, nullptr, nullptr}, st); break;
        case 5: err = launch_stream_k<2, kFirstGelu>(ks1, xp, rowmap, p1, h, tiles, ntiles, f, d, max_tiles, act_kmajor, b1, FoldOut{nullptr, nullptr, nullptr}, st); break;
        case 8: err = launch_stream_k<4, kFirstRelu>(ks1, xp, rowmap, p1, h, tiles, ntiles, f, d, max_tiles, act_kmajor, b1, FoldOut{nullptr, nullptr, nullptr}, st); break;
        default: err = launch_stream_k<4, kFirstGelu>(ks1, xp, rowmap, p1, h, tiles, ntiles, f, d, max_tiles, act_kmajor, b1, FoldOut{nullptr, nullptr, nullptr}, st); break;
    }
    if (err != hipSuccess) return err;
    if ((err = mark_profile_event(2, st)) != hipSuccess) return err;
    if ((err = mark_profile_event(3, st)) != hipSuccess) return err;
    // few tokens and few experts: units of one column block, so that every CU has one
    const bool narrow = ffn_tfmax(s) == 1 && ks2 == 4 && fold.out == nullptr &&
                        tiles_expected * ((d / 16 + 3) / 4) < device_cu_count();
    if (narrow) {
        long grid = max_tiles * (d / 16);
        if (grid > device_cu_count()) grid = device_cu_count();
        hipLaunchKernelGGL(ffn_stream_narrow_kernel, dim3(static_cast<unsigned>(grid < 1 ? 1 : grid)), dim3(256), 0, st, h, p2,
                           static_cast<void*>(y_perm), tiles, ntiles, d, f, b2);
        if ((err = hipGetLastError()) != hipSuccess) return err;
        return mark_profile_event(4, st);
    }
    switch (ffn_tfmax(s)) {
        case 1: err = launch_stream_k<1, 0>(ks2, h, nullptr, p2, y_perm, tiles, ntiles, d, f, max_tiles, true, b2, fold, st); break;
        case 2: err = launch_stream_k<2, 0>(ks2, h, nullptr, p2, y_perm, tiles, ntiles, d, f, max_tiles, true, b2, fold, st); break;
        default: err = launch_stream_k<4, 0>(ks2, h, nullptr, p2, y_perm, tiles, ntiles, d, f, max_tiles, true, b2, fold, st); break;
    }
    if (err != hipSuccess) return err;
    return mark_profile_event(4, st);
}

hipError_t launch_expert_ffn(const moe_shape& s, const void* x_perm, const void* w1, const void* w2,
                             const float* b1, const float* b2,
                             const int32_t* offsets, const uint8_t* mask, float* y_perm, void* h_ws,
                             Tile* tiles_ws, Tile* tiles_big_ws, Tile* tiles_half_ws, int32_t* ntiles_ws, float* partials_ws,
                             void* x_kmajor_ws, hipStream_t st) {
    const TileLists lists = ffn_tile_lists(s, tiles_ws, tiles_big_ws, tiles_half_ws, ntiles_ws, partials_ws);
    hipLaunchKernelGGL(build_tiles_kernel, dim3(1), dim3(1024), 0, st, offsets, mask, s.E, s.T * s.k, lists);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    if (layer_gathers_kmajor(s)) {      // large layer: re-lay the permuted rows k-step-major first
        err = launch_gather_kmajor(s, x_perm, nullptr, x_kmajor_ws, st);
        if (err != hipSuccess) return err;
        return launch_expert_products(s, x_kmajor_ws, nullptr, true, w1, w2, b1, b2, y_perm, h_ws, lists,
                                      FoldOut{nullptr, nullptr, nullptr}, st);
    }
    return launch_expert_products(s, x_perm, nullptr, false, w1, w2, b1, b2, y_perm, h_ws, lists,
                                  FoldOut{nullptr, nullptr, nullptr}, st);
}

}  // namespace moe
