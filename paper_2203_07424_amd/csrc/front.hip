// S0 and S1 in one launch, with Bottom-FC (S2) riding along: everything up to the
// pooled vectors, for small batches.
//
// Pooling needs where its bags start, which is why the scan runs before it.  But a
// block of pooling waves takes neighbouring bags, so it needs one sum, that of all
// earlier lengths, and a few thousand lengths are added up by its threads with a
// few loads each, all in flight together: about as long as reading the offsets
// the scan would have left, and a launch less in front of it.  The offsets
// themselves are still written, by the scan's own blocks, for inspection and for its checks.
//
// front_kernel (pooled dot model, Bottom-FC of narrow layers): blocks of 8 waves;
// first those of the scan, then those of Bottom-FC, then pooling, one bag a wave.
// front_fc_kernel (pooled dot model, any other Bottom-FC or none): instead of the stack
// its first layer alone, which needs nothing but the input, in the blocks its own
// launch would have (csrc/gemm_split.hip): 2560-1024-256-32 beside 10 tables, 1 sample
// 25.0 -> 20.3 us per forward, 64 26.9 -> 21.4, 300 37.2 -> 28.7, 700 46.3 -> 38.4;
// 500-256-64, 400 samples 24.6 -> 18.1.
// front_short_kernel (concatenation model, bags of a few ids, Bottom-FC none or one
// layer): blocks of 4 waves; the scan's, those that narrow the dense part (or that
// layer's, which write its columns of the Predict-FC input rows too), then pooling.
// 64-64 in front of four towers, 26 tables x 300 42.6 -> 32.5 us, x 1 28.3 -> 17.3.
//
// The pooling waves of front_kernel get the registers Bottom-FC's need: 122, and 16 of them share a compute unit, or 64
// in the light form, and all 32 do (front_takes_light()).  LONG_BAGS is its limit in the form with 122, beyond which some shapes
// lose against two launches (us per forward, two launches / one: 8 tables x 800 samples 15.7 / 12.8, 40 x 160 26.9 / 23.2,
// 10 x 700 22.2 / 20.2; 10 x 800 22.9 / 23.2); LIGHT_BAGS, below, that of the light one.
//
// front_fc_kernel's pooling blocks get the registers and the LDS of the layer's tile: tiles of up to 32 rows,
// between 68 and 123 registers.  Its limit is LONG_BAGS as well: below, the layer beside the scan alone (csrc/scan.hip) is the
// longer forward in most shapes and near the line as often the shorter one (beside pooling / beside the scan: 30 x 200,
// 2560 -> 1024 36.0 / 38.3; 14 x 500, 600 -> 512 with 8 ids 27.1 / 25.5, with 60 31.3 / 31.6); beyond it that is the
// shorter (12 000 bags: 50.5 / 49.7, 57.9 as three launches; 14 000 and more 59.8 / 52.2, 41.6 / 24.8).
//
// front_short_kernel, up to SHORT_FORM_BAGS: 26 tables x 300 samples 47.4 -> 44.8 us, x 16 36.7 -> 34.0, even at 16 380 bags,
// where adding up the lengths takes as long as the launches it saves.
#include <algorithm>

#include "gemm_split_body.h"
#include "mlp_chain_body.h"
#include "pool_body.h"
#include "scan_body.h"

namespace rec {

namespace {

using namespace scan;
using namespace pool;
using split::Rider;

constexpr int LONG_BAGS = 7 * SCAN_TILE / 2;
// With the light form of a whole Bottom-FC: us per forward, two launches / one, 10 tables of 80 fp32 rows x 1024
// samples 31.1 / 27.7, 40 of 80 fp16 rows x 256 30.6 / 25.9, 13 x 966 of 10 ids 18.0 / 15.4 (12 558 bags), 14 x 949 of 42
// 29.9 / 26.3 (13 286).  Each block of eight bags reads all earlier lengths, so beyond it shapes lose: 12 x 1276 24.1 /
// 25.0 (15 312), 5 x 3155 26.6 / 28.0 (15 775), 40 x 800 43.2 / 52.7.  In front of one to three tables Bottom-FC's
// blocks are so many that the line lies lower (8 ids, fp32 and fp16 rows: 1 x 12 300 29.4 / 28.2 and 26.7 / 26.3, 1 x 13 000 29.5 / 29.2 and 26.8 /
// 27.4, 1 x 14 300 29.8 / 30.5 and 27.3 / 28.8, 2 x 7150 23.4 / 23.9 and 21.4 / 22.4; but 4 x 3575 21.0 / 20.5, 8 x 1787 18.8 / 18.3).
constexpr int LIGHT_BAGS = 7 * SCAN_TILE, LIGHT_BAGS_FEW = 25 * SCAN_TILE / 4;
constexpr int MANY_LOADS = 7, MANY_BAGS = 13 * SCAN_TILE / 2;  // loads of a thread, and beyond which bags
constexpr int LIGHT_INPUT = 512;  // inputs of such a stack at most: four blocks a compute unit by its LDS

// Sum over max(len, 0) of lengths [0, n) by all threads of the block; s_w: a word
// per wave.
template <int THREADS, int U>
__device__ inline long long sum_before(const int32_t *__restrict__ len, int n, long long *s_w)
{
    const long long sum = wave_sum(part_of_sum<THREADS, U>(len, n));
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = sum;
    __syncthreads();
    long long all = 0;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) all += s_w[w];
    return all;
}

// Block `b` of the pooling blocks, WAVES bags a block, one a wave.
template <int WAVES, int LPR, bool HALF, bool STREAM, int U = SUM_LOADS>
__device__ inline void pool_from_lengths(const int32_t *__restrict__ len, const TableDesc *__restrict__ tables,
                                         const int32_t *__restrict__ indices, long long nnz, int n, int b, int per,
                                         const BagTable &div, int T, float one, ErrRecord *err, const PoolOut &out)
{
    // XCD x takes an eighth of the table-major bag list (see pool_kernel).
    const int first = ((b & 7) * per + (b >> 3)) * WAVES;
    if (first >= n) return;
    __shared__ long long s_w[WAVES];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), bag = first + wave;
    int own[WAVES];  // the block's lengths, requested with the others
#pragma unroll
    for (int i = 0; i < WAVES; ++i) own[i] = max(len[min(first + i, n - 1)], 0);
    long long start = sum_before<WAVES * 64, U>(len, first, s_w);
    if (bag >= n) return;
    long long end = start;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) {
        start += i < wave ? own[i] : 0;
        end += i <= wave ? own[i] : 0;
    }
    const int t = div.of(bag);
    pool_bag<LPR, HALF, false, STREAM, true>(tables, indices, out, 0, T, bag - t * (int)div.B, t, (int)min(start, nnz),
                                             (int)min(end, nnz), one, err);
}

// LIGHT: Bottom-FC within 64 registers, so that 32 pooling waves share a compute unit.  U: loads of a thread for the
// earlier lengths; SUM_LOADS take 12 288 of them in one trip, and seven pay from where many blocks have more (us per
// forward, six / seven, 8 tables of 8 ids x 1787 samples 19.6 / 18.9, x 1625 18.1 / 18.4, x 1375 17.3 / 17.4; both in one
// kernel, chosen at run time, cost those 0.2 us that need no seventh).
template <int LPR, bool HALF, bool STREAM, bool LIGHT, int U = SUM_LOADS>
__global__ __launch_bounds__(chain::CH_THREADS, LIGHT ? 8 : chain::waves_per_simd<1>()) void front_kernel(
    const int32_t *__restrict__ len, const TableDesc *__restrict__ tables, const int32_t *__restrict__ indices,
    long long nnz, int n, int tiles, int chain_blocks, int per, unsigned B, unsigned magic, int T, float one,
    int32_t *__restrict__ offsets, ErrRecord *err, const PoolOut out, const ChainArgs<1> a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    int b = blockIdx.x;
    if (b < tiles) {
        if constexpr (LIGHT) {
            ScanShared &sh = *reinterpret_cast<ScanShared *>(smem);
            if (threadIdx.x < SCAN_THREADS) scan_offsets_tile<true>(len, n, nnz, TileLink{}, offsets, err, b, sh);
        } else {
            __shared__ ScanShared sh;
            if (threadIdx.x < SCAN_THREADS) scan_offsets_tile(len, n, nnz, TileLink{}, offsets, err, b, sh);
        }
        return;
    }
    b -= tiles;
    if (b < chain_blocks) {
        chain::touch_args<80 + sizeof(out) + sizeof(a)>();
        const int share = chain::touch_share(chain_blocks);
        if constexpr (LIGHT)
            chain::light_chain_block<true>(a, smem, b, 0, (b >> 3) % share, share);
        else
            chain::mlp_chain_block<true, 1, 1>(a, smem, b, 0, (b >> 3) % share, share);
        return;
    }
    static_assert((LIGHT ? LIGHT_BAGS : LONG_BAGS) <= (LIGHT ? 7 : 6) * 4 * chain::CH_THREADS, "one trip");
    pool_from_lengths<chain::CH_WAVES, LPR, HALF, STREAM, U>(len, tables, indices, nnz, n, b - chain_blocks, per,
                                                             BagTable{B, magic}, T, one, err, out);
}

// A block has the WK waves of the layer's tile.  TM = 0: no layer.
template <int LPR, bool HALF, bool STREAM, int TM, int TN, int WK>
__global__ __launch_bounds__(64 * WK, TM < 2 ? 6 : TN < 4 ? 4 : WK == 8 ? 4 : 2) void front_fc_kernel(
    const int32_t *__restrict__ len, const TableDesc *__restrict__ tables, const int32_t *__restrict__ indices,
    long long nnz, int n, int tiles, int fc_blocks, int per, unsigned B, unsigned magic, int T, float one,
    int32_t *__restrict__ offsets, ErrRecord *err, const PoolOut out, const Rider a)
{
    int b = blockIdx.x;
    if (b < tiles) {
        __shared__ ScanShared sh;
        if (threadIdx.x < SCAN_THREADS) scan_offsets_tile(len, n, nnz, TileLink{}, offsets, err, b, sh);
        return;
    }
    b -= tiles;
    if constexpr (TM > 0) {
        extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
        if (b < fc_blocks) {
            split::split_block<TM, TN, 1, WK, split::IN_F32, split::OUT_EITHER>(a.p, a.g, smem, b);
            return;
        }
        b -= fc_blocks;
    }
    pool_from_lengths<WK, LPR, HALF, STREAM>(len, tables, indices, nnz, n, b, per, BagTable{B, magic}, T, one,
                                                         err, out);
}

// Bags of one block of front_short_kernel: consecutive, each group of LPR lanes
// taking SHORT_BAGS of them a block's groups apart.
template <int LPR>
constexpr int short_groups() { return POOL_WAVES * (64 / LPR); }
template <int LPR>
constexpr int short_block_bags() { return short_groups<LPR>() * SHORT_BAGS; }

// FC: with a layer, in tiles of 16 x 32.
template <int LPR, bool HALF, bool FC>
__global__ __launch_bounds__(POOL_WAVES * 64) void front_short_kernel(
    const int32_t *__restrict__ len, const TableDesc *__restrict__ tables, const int32_t *__restrict__ indices,
    long long nnz, int n, int tiles, int extra, int per, unsigned B, unsigned magic, int T, float one, int vec_ok,
    int fc_blocks, int32_t *__restrict__ offsets, ErrRecord *err, const PoolOut out, const ConcatDense job,
    const typename std::conditional<FC, Rider, char>::type a)
{
    constexpr int THREADS = POOL_WAVES * 64, GROUPS = short_groups<LPR>(), BAGS = short_block_bags<LPR>();
    static_assert(THREADS == SCAN_THREADS && BAGS <= THREADS, "a thread per bag of the block");
    static_assert(POOL_WAVES == FRONT_SHORT_WAVES, "the layer's sums in the order of its own launch");
    int b = blockIdx.x;
    if (b < tiles) {
        __shared__ ScanShared sh;
        scan_offsets_tile(len, n, nnz, TileLink{}, offsets, err, b, sh);
        return;
    }
    b -= tiles;
    if (b < extra) {
        concat_dense_block<THREADS>(job, b, extra);
        return;
    }
    b -= extra;
    if constexpr (FC) {
        extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
        if (b < fc_blocks) {
            split::split_block<1, 2, 1, POOL_WAVES, split::IN_F32, split::OUT_EITHER>(a.p, a.g, smem, b);
            return;
        }
        b -= fc_blocks;
    }
    const BagTable div{B, magic};
    const int first = ((b & 7) * per + (b >> 3)) * BAGS;
    if (first >= n) return;
    __shared__ long long s_w[POOL_WAVES], s_scan[POOL_WAVES];
    __shared__ int s_off[BAGS + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int k = first + tid;
    const long long mine = tid < BAGS && k < n ? max(len[k], 0) : 0;
    block_offsets<THREADS>(mine, part_of_sum<THREADS>(len, first), nnz, BAGS, s_w, s_scan, s_off);
    __syncthreads();
    const int group = wave * (64 / LPR) + lane / LPR;
    bool live[SHORT_BAGS];
    int bag[SHORT_BAGS], pos[SHORT_BAGS], end[SHORT_BAGS];
#pragma unroll
    for (int g = 0; g < SHORT_BAGS; ++g) {
        const int at = group + g * GROUPS;
        live[g] = first + at < n;
        bag[g] = live[g] ? first + at : n - 1;
        pos[g] = s_off[at];
        end[g] = live[g] ? s_off[at + 1] : pos[g];
    }
    pool_short_bags<LPR, HALF, true>(tables, indices, out, vec_ok, div, T, live, bag, pos, end, one, err);
}

template <int LPR, bool HALF>
hipError_t launch_long(const FrontProblem &f, const ChainProblem &a, hipStream_t s)
{
    const int n = f.T * f.B, tiles = (n + SCAN_TILE - 1) / SCAN_TILE, chain_blocks = (a.M + 31) / 32;
    const int pool_blocks = ((n + chain::CH_WAVES - 1) / chain::CH_WAVES + 7) / 8 * 8;
    const BagTable div = BagTable::of_batch(f.B);
    static_assert(LONG_BAGS <= SUM_LOADS * 4 * chain::CH_THREADS && LIGHT_BAGS <= MANY_LOADS * 4 * chain::CH_THREADS, "one trip");
    auto k = !front_takes_light(n, f.nnz, LPR * 16, a.Kpad[0], a.num_cus)
                 ? (f.stream_rows ? front_kernel<LPR, HALF, true, false> : front_kernel<LPR, HALF, false, false>)
             : n <= MANY_BAGS
                 ? (f.stream_rows ? front_kernel<LPR, HALF, true, true> : front_kernel<LPR, HALF, false, true>)
                 : (f.stream_rows ? front_kernel<LPR, HALF, true, true, MANY_LOADS> : front_kernel<LPR, HALF, false, true, MANY_LOADS>);
    hipLaunchKernelGGL(k, dim3(tiles + chain_blocks + pool_blocks), dim3(chain::CH_THREADS),
                       std::max(chain::chain_lds_bytes<1>(a.ld_lds), sizeof(ScanShared)), s, f.lengths, f.tables, f.indices, f.nnz, n, tiles, chain_blocks,
                       pool_blocks / 8, div.B, div.magic, f.T, 1.0f, f.offsets, f.err, f.out, one_stack(a));
    return hipGetLastError();
}

template <int LPR, bool HALF, int TM, int TN, int WAVES>
hipError_t launch_fc_beside(const FrontProblem &f, hipStream_t s)
{
    const int n = f.T * f.B, tiles = (n + SCAN_TILE - 1) / SCAN_TILE;
    const int pool_blocks = ((n + WAVES - 1) / WAVES + 7) / 8 * 8;
    const BagTable div = BagTable::of_batch(f.B);
    Rider a{};
    size_t lds = 0;
    if constexpr (TM > 0) {
        a = split::rider_of(*f.layer, TM, TN, f.out.z, f.out.ldz, f.z_cols);
        lds = split::split_lds_bytes<TM, TN, 1, WAVES>();
    }
    const int fc_blocks = 8 * a.p.per_xcd;
    auto k = f.stream_rows ? front_fc_kernel<LPR, HALF, true, TM, TN, WAVES> : front_fc_kernel<LPR, HALF, false, TM, TN, WAVES>;
    hipLaunchKernelGGL(k, dim3(tiles + fc_blocks + pool_blocks), dim3(WAVES * 64), lds, s, f.lengths, f.tables, f.indices,
                       f.nnz, n, tiles, fc_blocks, pool_blocks / 8, div.B, div.magic, f.T, 1.0f, f.offsets, f.err, f.out, a);
    return hipGetLastError();
}

template <int LPR, bool HALF>
hipError_t launch_fc_front(const FrontProblem &f, hipStream_t s)
{
    if (!f.layer) return launch_fc_beside<LPR, HALF, 0, 0, 8>(f, s);
    const FcTile t = fc_split_tile(*f.layer);
    switch (t.tm * 100 + t.tn * 10 + t.wk) {
    case 118: return launch_fc_beside<LPR, HALF, 1, 1, 8>(f, s);
    case 128: return launch_fc_beside<LPR, HALF, 1, 2, 8>(f, s);
    case 224: return launch_fc_beside<LPR, HALF, 2, 2, 4>(f, s);
    case 228: return launch_fc_beside<LPR, HALF, 2, 2, 8>(f, s);
    case 248: return launch_fc_beside<LPR, HALF, 2, 4, 8>(f, s);
    case 244: return launch_fc_beside<LPR, HALF, 2, 4, 4>(f, s);
    }
    return hipErrorInvalidValue;
}

template <int LPR, bool HALF>
hipError_t launch_short(const FrontProblem &f, hipStream_t s)
{
    constexpr int NACC = HALF ? 8 : 4;
    const int n = f.T * f.B, tiles = (n + SCAN_TILE - 1) / SCAN_TILE;
    const int vec_ok = f.out.col0 % NACC == 0 && reinterpret_cast<uintptr_t>(f.out.z) % 16 == 0;
    const int extra = concat_dense_blocks(f.dense, POOL_WAVES);
    constexpr int BAGS = short_block_bags<LPR>();
    const BagTable div = BagTable::of_batch(f.B);
    const int pool_blocks = ((n + BAGS - 1) / BAGS + 7) / 8 * 8;
    if (f.layer) {
        const Rider a = split::rider_of(*f.layer, 1, 2, f.out.z, f.out.ldz, f.z_cols);
        const int fc_blocks = 8 * a.p.per_xcd;
        hipLaunchKernelGGL((front_short_kernel<LPR, HALF, true>), dim3(tiles + extra + fc_blocks + pool_blocks),
                           dim3(POOL_WAVES * 64), (split::split_lds_bytes<1, 2, 1, POOL_WAVES>()), s, f.lengths, f.tables,
                           f.indices, f.nnz, n, tiles, extra, pool_blocks / 8, div.B, div.magic, f.T, 1.0f, vec_ok, fc_blocks,
                           f.offsets, f.err, f.out, f.dense, a);
    } else {
        hipLaunchKernelGGL((front_short_kernel<LPR, HALF, false>), dim3(tiles + extra + pool_blocks), dim3(POOL_WAVES * 64), 0,
                           s, f.lengths, f.tables, f.indices, f.nnz, n, tiles, extra, pool_blocks / 8, div.B, div.magic, f.T,
                           1.0f, vec_ok, 0, f.offsets, f.err, f.out, f.dense, (char)0);
    }
    return hipGetLastError();
}

template <int LPR, bool HALF, int TM, int TN, int WAVES>
hipError_t prepare_fc_beside()
{
    constexpr size_t lds = split::split_lds_bytes<TM, TN, 1, WAVES>();
    const hipError_t e = grant_lds(front_fc_kernel<LPR, HALF, false, TM, TN, WAVES>, lds);
    return e == hipSuccess ? grant_lds(front_fc_kernel<LPR, HALF, true, TM, TN, WAVES>, lds) : e;
}

template <int LPR, bool HALF>
hipError_t prepare_long()
{
    constexpr size_t most = chain::chain_lds_bytes<1>(CHAIN_MAX_WIDTH + chain::CH_LDS_PAD);
    hipError_t e = grant_lds(front_kernel<LPR, HALF, false, false>, most);
    if (e == hipSuccess) e = grant_lds(front_kernel<LPR, HALF, true, false>, most);
    if (e == hipSuccess) e = grant_lds(front_kernel<LPR, HALF, false, true>, most);
    if (e == hipSuccess) e = grant_lds(front_kernel<LPR, HALF, true, true>, most);
    if (e == hipSuccess) e = grant_lds(front_kernel<LPR, HALF, false, true, MANY_LOADS>, most);
    if (e == hipSuccess) e = grant_lds(front_kernel<LPR, HALF, true, true, MANY_LOADS>, most);
    if (e == hipSuccess) e = prepare_fc_beside<LPR, HALF, 2, 2, 8>();
    if (e == hipSuccess) e = prepare_fc_beside<LPR, HALF, 2, 4, 8>();
    return e;
}

}  // namespace

// The light form of Bottom-FC, beside twice the pooling waves, beyond LONG_BAGS and up to there where
// pooling is the longer part: by the bytes of rows a compute unit gathers (us per forward, other form / light; 320 KB
// 19.4 / 18.3, 450 21.9 / 20.1; 256 23.4 / 23.9, 64 12.6 / 13.4).  Stacks of wider inputs have two blocks a compute unit by
// their LDS in either form and gain no wave (28 tables of 80 fp32 rows x 256 samples in front of x-64-64, 560 KB: 256 inputs
// 23.9 / 22.4, 500 24.0 / 24.1, 576 24.0 / 24.6, 1000 24.2 / 26.4).
bool front_takes_light(long long n, long long nnz, int rowbytes, int input, int num_cus)
{
    return n > LONG_BAGS || (input <= LIGHT_INPUT && nnz * rowbytes > (long long)num_cus * (288 * 1024));
}

bool front_applies(int T, int B, int D, int dtype, long long nnz, long long max_rows, bool concat, int ride_input)
{
    const long long n = (long long)T * B;
    const int rowbytes = D * (dtype == REC_F16 ? 2 : 4);
    const int light = T < 4 ? LIGHT_BAGS_FEW : LIGHT_BAGS;
    const int most = concat ? SHORT_FORM_BAGS : ride_input > 0 && ride_input <= LIGHT_INPUT ? light : LONG_BAGS;
    if (n > most || (rowbytes != 64 && rowbytes != 128 && rowbytes != 256)) return false;
    const bool sh = pool_short_applies(rowbytes, nnz, n);
    return concat ? sh : !sh && pool_narrow(max_rows, rowbytes);
}

hipError_t front_prepare()
{
    hipError_t e = prepare_long<4, true>();
    if (e == hipSuccess) e = prepare_long<8, true>();
    if (e == hipSuccess) e = prepare_long<16, true>();
    if (e == hipSuccess) e = prepare_long<4, false>();
    if (e == hipSuccess) e = prepare_long<8, false>();
    if (e == hipSuccess) e = prepare_long<16, false>();
    return e;
}

// Beside short bags a layer rides along in tiles of 16 x 32, where these are few; else
// in tiles of up to 32 rows.  Those of 48 and 80 would leave pooling one block a compute unit by their
// LDS, which every block of a launch gets, and those of 64 two: the layer beside the scan alone is the
// shorter forward (us, beside pooling / beside the scan; 1024 columns and 4 tables x 1790 samples, 600 inputs 38.1
// / 34.5, 1536 43.1 / 39.9, 2560 49.2 / 48.1; 2560, x 1600 45.8 / 48.2, the one that lost).
bool front_layer_rides(const FcProblem &a, bool concat)
{
    if (!fc_split_rides(a)) return false;
    if (concat) return (long long)((a.M + 15) / 16) * (a.Npad / 32) <= 512;
    const FcTile t = fc_split_tile(a);
    return t.tm <= 2;
}

bool front_takes(const ChainProblem &rider) { return chain::narrow_run(rider); }

hipError_t launch_front(const FrontProblem &f, const ChainProblem *rider, hipStream_t s)
{
    if (f.T <= 0 || f.B <= 0) return hipSuccess;
    const bool half = f.dtype == REC_F16;
    const int lpr = f.D * (half ? 2 : 4) / 16;
    if (rider) {
        if (!rider->a_f32 || rider->groups != 1 || !front_takes(*rider) || f.out.z) return hipErrorInvalidValue;
        ChainProblem a;
        const hipError_t e = chain_finalize(*rider, a);
        if (e != hipSuccess) return e;
        switch (lpr) {
        case 4: return half ? launch_long<4, true>(f, a, s) : launch_long<4, false>(f, a, s);
        case 8: return half ? launch_long<8, true>(f, a, s) : launch_long<8, false>(f, a, s);
        case 16: return half ? launch_long<16, true>(f, a, s) : launch_long<16, false>(f, a, s);
        default: return hipErrorInvalidValue;
        }
    }
    if (f.layer && !fc_split_rides(*f.layer)) return launch_fc_big_beside_pool(f, s);
    if (f.layer && (!front_layer_rides(*f.layer, f.out.z != nullptr) || (f.out.z && f.out.ldz % 4 != 0)))
        return hipErrorInvalidValue;
#define REC_FRONT_BY_ROW(LAUNCH)                                          \
    switch (lpr) {                                                        \
    case 4: return half ? LAUNCH<4, true>(f, s) : LAUNCH<4, false>(f, s);   \
    case 8: return half ? LAUNCH<8, true>(f, s) : LAUNCH<8, false>(f, s);   \
    case 16: return half ? LAUNCH<16, true>(f, s) : LAUNCH<16, false>(f, s); \
    default: return hipErrorInvalidValue;                                 \
    }
    if (!f.out.z) REC_FRONT_BY_ROW(launch_fc_front)
    if (!f.dense.x0) return hipErrorInvalidValue;
    if (f.T * f.B > SHORT_FORM_BAGS) return launch_lookups(f, s);
    REC_FRONT_BY_ROW(launch_short)
#undef REC_FRONT_BY_ROW
}

}  // namespace rec
