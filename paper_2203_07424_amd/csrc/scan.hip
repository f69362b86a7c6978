// S0: pooling lengths -> bag offsets (exclusive scan), staged in LDS.
//
// The sparse input gives, per (table, sample), how many ids follow (the pooling
// factor varies per lookup, Fig. 2(c)); the gather needs where each bag starts.
// One launch over at most a few hundred thousand int32: a block scans a tile of
// 2048 in LDS, publishes its sum in a word of device memory that carries its own
// "valid" bit (no fence: the word is all that is handed on, and the pooling launch
// clears it) and polls the words of the tiles before it.  Bound by that hand-over, a round trip to memory: 80 tiles
// with Bottom-FC riding along 11.2 us against 5.5 + 9.6 in two launches (40 tables x
// 4096 170.9 -> 166.7 us per forward), 52 tiles alone 8.4 against 4.6 + 5.4 (103.8
// -> 102.3), 480 tiles with Bottom-FC 26.6 against 6.3 + 20.
// Measured and dropped: two launches, tile sums first (what this replaced); tile
// totals reduced by each pooling wave (+28 us of pooling); a last-block-done
// ticket in front of the offsets (its device-scope fences cost more than a launch).
#include <algorithm>
#include "gemm_split_body.h"
#include "mlp_chain_body.h"
#include "scan_body.h"

namespace rec {

namespace {

using namespace scan;

__global__ __launch_bounds__(64) void clear_err_kernel(ErrRecord *err)
{
    if (threadIdx.x == 0) {
        err->first_bad_len = ~0ull;
        err->first_bad_idx = ~0ull;
        err->flags = 0u;
    }
}

__global__ __launch_bounds__(256) void clear_tile_words_kernel(unsigned long long *words, int n)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) words[i] = 0;
}

// The scan alone: blocks [0, tiles) write the offsets, the blocks
// behind them do a concatenation model's dense copy.
__global__ __launch_bounds__(SCAN_THREADS) void scan_tile_offsets(
    const int32_t *__restrict__ len, int32_t *__restrict__ offsets, unsigned long long *words, long long nnz, int n,
    int tiles, int polls, int extra, ErrRecord *err, const ConcatDense job)
{
    __shared__ ScanShared sh;
    if ((int)blockIdx.x < tiles)
        scan_offsets_tile(len, n, nnz, TileLink{words, tiles, polls}, offsets, err, blockIdx.x, sh);
    else
        concat_dense_block<SCAN_THREADS>(job, blockIdx.x - tiles, extra);
}

// The same with a stack of fully connected layers riding along: blocks of
// chain::CH_THREADS threads; behind the scan's and the copy's blocks come
// chain_grid_x blocks that each take 32 samples through the stack.
// A scan block uses its first SCAN_THREADS threads; the waves of the others end
// at once (a barrier counts only the waves of a group that have not ended).
template <int MAXC>
__global__ __launch_bounds__(chain::CH_THREADS, chain::waves_per_simd<MAXC>()) void scan_offsets_ride_kernel(
    const int32_t *__restrict__ len, int32_t *__restrict__ offsets, unsigned long long *words, long long nnz, int n,
    int tiles, int polls, int extra, int chain_grid_x, ErrRecord *err, const ConcatDense job, const ChainArgs<1> a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int b = blockIdx.x;
    if (b < tiles) {
        __shared__ ScanShared sh;
        if (threadIdx.x < SCAN_THREADS) scan_offsets_tile(len, n, nnz, TileLink{words, tiles, polls}, offsets, err, b, sh);
    } else if (b < tiles + extra) {
        concat_dense_block<chain::CH_THREADS>(job, b - tiles, extra);
    } else {
        chain::touch_args<64 + sizeof(job) + sizeof(a)>();
        const int bx = b - tiles - extra, share = chain::touch_share(chain_grid_x);
        chain::mlp_chain_block<true, 1, MAXC>(a, smem, bx, 0, (bx >> 3) % share, share);
    }
}

// The same with the first layer of a stack that does not ride as a whole, in the tiles of
// its own launch: it starts at once instead of behind scan and pooling, whose few blocks
// leave the chip idle.  1536-1024 beside 10 tables x 900 samples 42.5 -> 36.9 us per forward,
// 500-256 beside 10 x 3000 51.5 -> 45.9; one 64-64 layer of a concatenation model, 26 x 4096
// 104.8 -> 97.9.  Layers that take 128 x 128 tiles: fc_big_behind_scan_kernel.
template <int TM, int TN, int WK>
__global__ __launch_bounds__(64 * WK, TM * TN >= 8 ? 2 : 4) void scan_offsets_layer_kernel(
    const int32_t *__restrict__ len, int32_t *__restrict__ offsets, unsigned long long *words, long long nnz, int n,
    int tiles, int polls, int extra, ErrRecord *err, const ConcatDense job, const split::Rider a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int b = blockIdx.x;
    if (b < tiles) {
        __shared__ ScanShared sh;
        if (threadIdx.x < SCAN_THREADS) scan_offsets_tile(len, n, nnz, TileLink{words, tiles, polls}, offsets, err, b, sh);
    } else if (b < tiles + extra) {
        concat_dense_block<64 * WK>(job, b - tiles, extra);
    } else {
        split::split_block<TM, TN, 1, WK, split::IN_F32, split::OUT_EITHER>(a.p, a.g, smem, b - tiles - extra);
    }
}

template <int TM, int TN, int WK>
hipError_t launch_beside(const ScanBlocks &b, int extra, const ConcatDense &job, const FcProblem &layer, void *z, int ldz,
                         int z_cols, hipStream_t s)
{
    const split::Rider a = split::rider_of(layer, TM, TN, z, ldz, z_cols);
    hipLaunchKernelGGL((scan_offsets_layer_kernel<TM, TN, WK>), dim3(b.tiles + extra + 8 * a.p.per_xcd), dim3(64 * WK),
                       (split::split_lds_bytes<TM, TN, 1, WK>()), s, b.lengths, b.offsets, b.words, b.nnz, b.n, b.tiles,
                       b.polls, extra, b.err, job, a);
    return hipGetLastError();
}

template <int TM, int TN, int WK>
hipError_t grant_layer_lds()
{
    return grant_lds(scan_offsets_layer_kernel<TM, TN, WK>, split::split_lds_bytes<TM, TN, 1, WK>());
}

}  // namespace

hipError_t launch_clear_err(ErrRecord *err, hipStream_t s)
{
    hipLaunchKernelGGL(clear_err_kernel, dim3(1), dim3(64), 0, s, err);
    return hipGetLastError();
}

hipError_t launch_clear_tile_words(unsigned long long *words, int n, hipStream_t s)
{
    hipLaunchKernelGGL(clear_tile_words_kernel, dim3(std::min((n + 255) / 256, 256)), dim3(256), 0, s, words, n);
    return hipGetLastError();
}

hipError_t scan_prepare()
{
    constexpr size_t most = chain::chain_lds_bytes<1>(CHAIN_MAX_WIDTH + chain::CH_LDS_PAD);
    hipError_t e = grant_lds(scan_offsets_ride_kernel<1>, most);
    if (e == hipSuccess) e = grant_lds(scan_offsets_ride_kernel<4>, most);
    if (e == hipSuccess) e = grant_layer_lds<2, 2, 8>();
    if (e == hipSuccess) e = grant_layer_lds<2, 4, 8>();
    if (e == hipSuccess) e = grant_layer_lds<3, 4, 8>();
    if (e == hipSuccess) e = grant_layer_lds<4, 4, 4>();
    if (e == hipSuccess) e = grant_layer_lds<5, 4, 8>();
    return e;
}

// With a stack riding along the launch lasts as long as the stack, so for a few
// tiles its scan blocks have the time to add up the earlier lengths themselves.
int scan_linked_words(int n, bool with_rider)
{
    const int tiles = (n + SCAN_TILE - 1) / SCAN_TILE;
    return tiles > (with_rider ? 8 : 1) ? tiles - 1 : 0;
}

hipError_t launch_scan(const int32_t *lengths, int n, long long nnz, int32_t *offsets,
                       unsigned long long *tile_words, ErrRecord *err, const ConcatDense &job,
                       const ChainProblem *rider, hipStream_t s, int polls)
{
    if (n <= 0) return hipSuccess;
    const int tiles = (n + SCAN_TILE - 1) / SCAN_TILE;
    const int extra = concat_dense_blocks(job, SCAN_THREADS / 64);
    const bool has_rider = rider && rider->M > 0;
    unsigned long long *words = scan_linked_words(n, has_rider) > 0 ? tile_words : nullptr;
    if (has_rider) {
        if (!rider->a_f32 || rider->groups != 1) return hipErrorInvalidValue;
        ChainProblem a;
        const hipError_t e = chain_finalize(*rider, a);
        if (e != hipSuccess) return e;
        const int chain_grid_x = (a.M + 31) / 32;
        auto k = chain::narrow_run(a) ? scan_offsets_ride_kernel<1> : scan_offsets_ride_kernel<4>;
        hipLaunchKernelGGL(k, dim3(tiles + extra + chain_grid_x), dim3(chain::CH_THREADS),
                           chain::chain_lds_bytes<1>(a.ld_lds), s, lengths, offsets, words, nnz, n, tiles, polls, extra,
                           chain_grid_x, err, job, one_stack(a));
        return hipGetLastError();
    }
    hipLaunchKernelGGL(scan_tile_offsets, dim3(tiles + extra), dim3(SCAN_THREADS), 0, s, lengths, offsets, words, nnz, n,
                       tiles, polls, extra, err, job);
    return hipGetLastError();
}

bool scan_layer_rides(const FcProblem &a, const void *z)
{
    return fc_split_rides(a) || (!z && fc_big_rides(a, a.num_cus));
}

hipError_t launch_scan_beside_layer(const int32_t *lengths, int n, long long nnz, int32_t *offsets,
                                    unsigned long long *tile_words, ErrRecord *err, const ConcatDense &job,
                                    const FcProblem &layer, void *z, int ldz, int z_cols, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    if (!scan_layer_rides(layer, z) || (z && ldz % 4 != 0)) return hipErrorInvalidValue;
    const ScanBlocks b{lengths, offsets, scan_linked_words(n, true) > 0 ? tile_words : nullptr, nnz, n,
                       (n + SCAN_TILE - 1) / SCAN_TILE, SCAN_LINK_POLLS, err};
    if (!fc_split_rides(layer)) return job.x0 ? hipErrorInvalidValue : launch_fc_big_behind_scan(layer, b, s);
    const int extra = concat_dense_blocks(job, SCAN_THREADS / 64);
    const FcTile t = fc_split_tile(layer);
    switch (t.tm * 100 + t.tn * 10 + t.wk) {
    case 118: return launch_beside<1, 1, 8>(b, extra, job, layer, z, ldz, z_cols, s);
    case 128: return launch_beside<1, 2, 8>(b, extra, job, layer, z, ldz, z_cols, s);
    case 224: return launch_beside<2, 2, 4>(b, extra, job, layer, z, ldz, z_cols, s);
    case 228: return launch_beside<2, 2, 8>(b, extra, job, layer, z, ldz, z_cols, s);
    case 244: return launch_beside<2, 4, 4>(b, extra, job, layer, z, ldz, z_cols, s);
    case 248: return launch_beside<2, 4, 8>(b, extra, job, layer, z, ldz, z_cols, s);
    case 348: return launch_beside<3, 4, 8>(b, extra, job, layer, z, ldz, z_cols, s);
    case 444: return launch_beside<4, 4, 4>(b, extra, job, layer, z, ldz, z_cols, s);
    case 548: return launch_beside<5, 4, 8>(b, extra, job, layer, z, ldz, z_cols, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace rec
