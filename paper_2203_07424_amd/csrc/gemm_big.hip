// S2 / S4 for wide layers on large batches (Table I: the 2560-wide Bottom-FC of
// DLRM-RMC3, the N towers of 1024-512-256 of MT-WnD): the same
// C = act(A W^T + b)  as fc_kernel, with block tiles of 256 x 256, 256 x 128 or
// 128 x 128 and 8 waves per block.
//
// A BM x BN tile moves (BM + BN) * 2 bytes per k for 2 * BM * BN flops, so large
// tiles ask least of the caches; the L2 can feed a compute unit about 49 bytes
// per clock (measured with a read-only probe on an L2-resident footprint) and a
// 256 x 256 tile needs 32 at full MFMA rate.  The tile pairs are double
// buffered in LDS (one barrier per k-tile; 256 x 256 x 64: 2 x 72 KB of the
// 160 KB), so one block owns a compute unit, two waves per SIMD.
//
// Per k-tile: tile kt is multiplied out of one LDS buffer while the registers
// holding tile kt+1 (fetched one iteration earlier) go to the other buffer and
// are refilled with tile kt+2, a quarter of that staging work per 16-wide step
// of matrix instructions.  Measured and not kept: 4 waves with 128 x 128 wave
// tiles (accumulators in AGPRs), 16 waves, and global loads written straight
// into LDS (swizzled rows, no staging registers) - each within 5 % of this.
#include <algorithm>

#include "pool_body.h"
#include "scan_body.h"

namespace rec {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int BK = 64;          // k extent of one staged tile
constexpr int LDS_LD = BK + 8;  // 144-byte row stride: 16-byte reads of 16 consecutive rows hit 16 different bank groups

template <int BM, int BN>
constexpr size_t big_lds_bytes() { return 2 * (size_t)(BM + BN) * LDS_LD * sizeof(__bf16); }

// 16 bytes of one activation row as fetched: 8 k in bf16, or 4 of raw fp32 (the model's
// dense input) that are narrowed only when they are written to LDS.  Neighbouring lanes fetch
// neighbouring 16 bytes: as 8 k a lane, 16 bytes of every 32 in one load, 4096 samples of 2560 -> 1024 beside the
// scan took 35.6 us and not 33.5 (from cold memory 50.1 and 47.3).
template <bool A_F32>
struct AReg;
template <>
struct AReg<false> {
    static constexpr int K = 8;
    bf16x8 v;
    __device__ inline void fetch(const char *p) { v = *reinterpret_cast<const bf16x8 *>(p); }
    __device__ inline bf16x8 narrow(bool) const { return v; }
};
template <>
struct AReg<true> {
    static constexpr int K = 4;
    f32x4 v;
    __device__ inline void fetch(const char *p) { v = *reinterpret_cast<const f32x4 *>(p); }
    __device__ inline bf16x4 narrow(bool valid) const
    {
        bf16x4 o;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = (__bf16)(valid ? v[i] : 0.0f);
        return o;
    }
};

struct BigLayer {
    const void *A, *W0;
    int lda, M, K, Kpad, grid_m, grid_n, tiles_per_group, per_xcd;
    long long a_stride;
    int relu;
    void *C;
    int ldc;
    long long c_stride;
};

// Block `block` of the launch; big_lds_bytes() of `smem`.
// A_F32: A is fp32 [M][lda] with only k < K valid (K a multiple of 8); chunks at
// k >= K are fetched from the row's last valid chunk and zeroed.
template <int BM, int BN, int WAVES_M, int WAVES_N, bool A_F32, bool OUT_F32, class Groups>
__device__ inline void big_block(const BigLayer &p, const Groups &groups, __bf16 *smem, int block)
{
    const void *__restrict__ A0 = p.A, *__restrict__ W0 = p.W0;
    const int lda = p.lda, M = p.M, K = p.K, Kpad = p.Kpad, grid_m = p.grid_m, grid_n = p.grid_n;
    const int tiles_per_group = p.tiles_per_group, per_xcd = p.per_xcd, relu = p.relu, ldc = p.ldc;
    const long long a_stride = p.a_stride, c_stride = p.c_stride;
    void *__restrict__ C0 = p.C;
    constexpr int THREADS = 64 * WAVES_M * WAVES_N;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;  // per-wave tile
    constexpr int TM = WM / 32, TN = WN / 32;            // 32 x 32 MFMA tiles per wave
    constexpr int ROWS_PER_PASS = THREADS / 8;           // 8 threads fetch the 64 k of one row
    constexpr int AK = AReg<A_F32>::K, A_THREADS = BK / AK;  // k of a load, threads that fetch a row of A
    constexpr int A_ROWS = THREADS / A_THREADS;
    constexpr int A_LOADS = BM / A_ROWS, W_LOADS = BN / ROWS_PER_PASS;
    constexpr int BUF = (BM + BN) * LDS_LD;              // elements of one tile pair
    static_assert(WM % 32 == 0 && WN % 32 == 0, "wave tile must be whole MFMA tiles");
    static_assert(BM % A_ROWS == 0 && BN % ROWS_PER_PASS == 0, "staging passes must tile the block");

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave % WAVES_M, wn = wave / WAVES_M;
    // XCD x (blocks are dealt round-robin) takes the x-th eighth of the tile
    // list; the list runs over strips of 4 row-tiles, column-tiles next, so the
    // tiles resident on one XCD form a compact patch that shares its slabs of A
    // and W in that XCD's L2.
    int v = block;
    if (per_xcd > 0) v = (block & 7) * per_xcd + (block >> 3);
    // Of a single stack the compiler is to know the index: a table of one looked up with a number
    // from the launch's arguments would be a copy in scratch memory.
    const int grp = sizeof(groups.W) == sizeof(void *) ? 0 : v / tiles_per_group;
    v -= grp * tiles_per_group;
    int bm, bn;
    if ((grid_m & 3) == 0) {
        const int strip = v / (4 * grid_n), w = v - strip * 4 * grid_n;
        bn = w >> 2;
        bm = strip * 4 + (w & 3);
    } else {
        bm = v / grid_n;
        bn = v - bm * grid_n;
    }
    const int m0 = bm * BM, n0 = bn * BN;
    constexpr int A_ELT = A_F32 ? 4 : 2;
    const char *__restrict__ A = static_cast<const char *>(A0) + grp * a_stride * A_ELT;
    const __bf16 *__restrict__ W = static_cast<const __bf16 *>(grp == 0 ? W0 : groups.W[grp]);
    const float *__restrict__ bias = groups.bias[grp];

    const int ld_row = tid >> 3, ld_chunk = tid & 7;
    const int a_row = tid / A_THREADS, a_k = tid % A_THREADS * AK;
    const char *a_src[A_LOADS];  // this thread's chunk of k-tile 0 in each of its rows
    const __bf16 *w_src[W_LOADS];
#pragma unroll
    for (int i = 0; i < A_LOADS; ++i) {
        int row = m0 + a_row + A_ROWS * i;
        row = row < M ? row : M - 1;  // rows past M are computed and dropped
        a_src[i] = A + (long long)row * lda * A_ELT;
    }
#pragma unroll
    for (int i = 0; i < W_LOADS; ++i)
        w_src[i] = W + (long long)(n0 + ld_row + ROWS_PER_PASS * i) * Kpad + ld_chunk * 8;

    f32x16 acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    AReg<A_F32> ra[A_LOADS];
    bf16x8 rw[W_LOADS];
    const int nk = Kpad / BK;

    // The staging work of a k-tile (BK / 16 = 4 steps of MFMAs) is cut into 4 parts,
    // one per step, so that LDS writes, global loads and LDS reads are issued in
    // the shadow of the matrix instructions instead of in a burst of their own.
    constexpr int KSTEPS = BK / 16;
    constexpr int A_PART = (A_LOADS + KSTEPS - 1) / KSTEPS, W_PART = (W_LOADS + KSTEPS - 1) / KSTEPS;
#define REC_BIG_FETCH_PART(kt, part)                                                       \
    do {                                                                                   \
        int k_ = (kt) * BK + a_k;                                                          \
        if (A_F32) k_ = k_ < K ? k_ : K - AK;                                              \
        _Pragma("unroll") for (int i = (part) * A_PART; i < ((part) + 1) * A_PART && i < A_LOADS; ++i) \
            ra[i].fetch(a_src[i] + (long long)k_ * A_ELT);                                 \
        _Pragma("unroll") for (int i = (part) * W_PART; i < ((part) + 1) * W_PART && i < W_LOADS; ++i) \
            rw[i] = *reinterpret_cast<const bf16x8 *>(w_src[i] + (kt) * BK);               \
    } while (0)
#define REC_BIG_STASH_PART(kt, buf, part)                                                  \
    do {                                                                                   \
        __bf16 *sa_ = smem + (buf) * BUF, *sw_ = sa_ + BM * LDS_LD;                        \
        const bool valid_ = !A_F32 || (kt) * BK + a_k < K; /* the chunk held in ra lies below K */ \
        _Pragma("unroll") for (int i = (part) * A_PART; i < ((part) + 1) * A_PART && i < A_LOADS; ++i) \
            *reinterpret_cast<decltype(ra[i].narrow(true)) *>(&sa_[(a_row + A_ROWS * i) * LDS_LD + a_k]) = ra[i].narrow(valid_); \
        _Pragma("unroll") for (int i = (part) * W_PART; i < ((part) + 1) * W_PART && i < W_LOADS; ++i) \
            *reinterpret_cast<bf16x8 *>(&sw_[(ld_row + ROWS_PER_PASS * i) * LDS_LD + ld_chunk * 8]) = rw[i]; \
    } while (0)
    // One k-tile: multiply tile kt out of buffer kt & 1; meanwhile (STASH) put the
    // registers holding tile kt+1 into the other buffer, whose last readers passed
    // the previous barrier, and (FETCH) refill them with tile kt+2.
#define REC_BIG_ITERATION(kt, STASH, FETCH)                                                \
    do {                                                                                   \
        const int cur_ = (kt) & 1;                                                         \
        const __bf16 *sA = smem + cur_ * BUF, *sW = sA + BM * LDS_LD;                      \
        _Pragma("unroll") for (int kk = 0; kk < KSTEPS; ++kk) {                            \
            const int kofs = kk * 16 + (lane >> 5) * 8;                                    \
            bf16x8 fw[TN], fa[TM];                                                         \
            _Pragma("unroll") for (int i = 0; i < TN; ++i)                                 \
                fw[i] = *reinterpret_cast<const bf16x8 *>(&sW[(wn * WN + i * 32 + (lane & 31)) * LDS_LD + kofs]); \
            _Pragma("unroll") for (int j = 0; j < TM; ++j)                                 \
                fa[j] = *reinterpret_cast<const bf16x8 *>(&sA[(wm * WM + j * 32 + (lane & 31)) * LDS_LD + kofs]); \
            if (STASH) REC_BIG_STASH_PART((kt) + 1, cur_ ^ 1, kk);                                   \
            if (FETCH) REC_BIG_FETCH_PART((kt) + 2, kk);                                   \
            __builtin_amdgcn_sched_barrier(0); /* else the compiler sinks all fetches to the end of the k-tile */ \
            _Pragma("unroll") for (int i = 0; i < TN; ++i)                                 \
                _Pragma("unroll") for (int j = 0; j < TM; ++j)                             \
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[i], fa[j], acc[i][j], 0, 0, 0); \
        }                                                                                  \
        __syncthreads();                                                                   \
    } while (0)

#pragma unroll
    for (int part = 0; part < KSTEPS; ++part) REC_BIG_FETCH_PART(0, part);
#pragma unroll
    for (int part = 0; part < KSTEPS; ++part) REC_BIG_STASH_PART(0, 0, part);
    if (nk > 1) {
#pragma unroll
        for (int part = 0; part < KSTEPS; ++part) REC_BIG_FETCH_PART(1, part);
    }
    __syncthreads();

    int kt = 0;
    for (; kt + 2 < nk; ++kt) REC_BIG_ITERATION(kt, true, true);
    if (kt + 1 < nk) {
        REC_BIG_ITERATION(kt, true, false);
        ++kt;
    }
    REC_BIG_ITERATION(kt, false, false);
#undef REC_BIG_ITERATION
#undef REC_BIG_FETCH_PART
#undef REC_BIG_STASH_PART

    // acc[i][j][r]: feature n = 8 * (r / 4) + 4 * (lane / 32) + r % 4, sample m = lane % 32.
    // A lane therefore holds 4 consecutive features of 32 different rows: stored
    // as they are, every store instruction would touch 32 lines with 16 bytes
    // each.  bf16 output goes through LDS instead (the operand tiles are done
    // with after the loop's last barrier): each wave lays its WM x WN tile out
    // row-major in a region of its own and writes it back as whole 128-byte rows.
    void *C = static_cast<char *>(C0) + grp * c_stride * (OUT_F32 ? 4 : 2);
    constexpr int EP_LD = WN + 8;  // padded row pitch of the staged tile (elements)
    static_assert(OUT_F32 || (size_t)WAVES_M * WAVES_N * WM * EP_LD <= 2 * (size_t)BUF, "staged C tiles must fit the LDS");
    __bf16 *stage = smem + (size_t)wave * WM * EP_LD;
#pragma unroll
    for (int i = 0; i < TN; ++i) {
#pragma unroll
        for (int j = 0; j < TM; ++j) {
            const int m = m0 + wm * WM + j * 32 + (lane & 31);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int nl = i * 32 + 8 * q + 4 * (lane >> 5);  // column inside the wave tile
                const int n = n0 + wn * WN + nl;
                const f32x4 bv = *reinterpret_cast<const f32x4 *>(bias + n);
                f32x4 o;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float x = acc[i][j][4 * q + r] + bv[r];
                    o[r] = (relu && x < 0.0f) ? 0.0f : x;
                }
                if (OUT_F32) {
                    if (m < M) *reinterpret_cast<f32x4 *>(static_cast<float *>(C) + (long long)m * ldc + n) = o;
                } else {
                    bf16x4 h;
#pragma unroll
                    for (int r = 0; r < 4; ++r) h[r] = (__bf16)o[r];
                    *reinterpret_cast<bf16x4 *>(&stage[(j * 32 + (lane & 31)) * EP_LD + nl]) = h;
                }
            }
        }
    }
    if (!OUT_F32) {
        constexpr int LANES_PER_ROW = WN / 8;            // 16 bytes per lane
        constexpr int ROWS_PER_STORE = 64 / LANES_PER_ROW;
        const int sr = lane / LANES_PER_ROW, sc = (lane % LANES_PER_ROW) * 8;
        __bf16 *Cb = static_cast<__bf16 *>(C) + n0 + wn * WN + sc;
#pragma unroll
        for (int r0 = 0; r0 < WM; r0 += ROWS_PER_STORE) {
            const int row = r0 + sr;
            const bf16x8 v = *reinterpret_cast<const bf16x8 *>(&stage[row * EP_LD + sc]);
            const int m = m0 + wm * WM + row;
            if (m < M) *reinterpret_cast<bf16x8 *>(Cb + (long long)m * ldc) = v;
        }
    }
}

template <int BM, int BN, int WAVES_M, int WAVES_N, bool A_F32, bool OUT_F32>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void fc_big_kernel(
    const void *__restrict__ A0, const void *__restrict__ W0, int lda, int M, int K, int Kpad, int grid_m, int grid_n,
    int tiles_per_group, int per_xcd, long long a_stride, int relu, void *__restrict__ C0, int ldc, long long c_stride,
    const FcGroups groups)
{
    extern __shared__ __attribute__((aligned(16))) __bf16 smem[];
    big_block<BM, BN, WAVES_M, WAVES_N, A_F32, OUT_F32>(
        BigLayer{A0, W0, lda, M, K, Kpad, grid_m, grid_n, tiles_per_group, per_xcd, a_stride, relu, C0, ldc, c_stride}, groups,
        smem, blockIdx.x);
}

// Bags of a pooling block beside a wide layer: one block a compute unit, whole rounds of four
// bags for each of its waves; a thread for each bag, and its sums in LDS.
constexpr int BESIDE_WIDE_BAGS = 256, BESIDE_WIDE_COLUMNS = 15360;
inline long long beside_wide_bags(long long n, int num_cus) { return ((n + num_cus - 1) / num_cus + 31) / 32 * 32; }
inline bool beside_wide_fits(long long n, int D, int num_cus)
{
    const long long bags = beside_wide_bags(n, num_cus);
    return bags <= BESIDE_WIDE_BAGS && bags * D <= BESIDE_WIDE_COLUMNS;
}

// One stack's layer of fp32 rows behind the blocks of a scan, which are done before the
// layer is a quarter through: two blocks of 128 x 128 tiles fit a compute unit (115
// registers, 72 KB of LDS, the scan's inside it), so no tile waits for them: 4096 samples,
// 2560-1024 beside 10 tables 76.4 -> 71.2 us per forward, 2400 beside 8 74.2 -> 66.7.  What bounds it is the chain
// of trips and barriers of one block in lock-step: 24 bytes of operands a clock and compute unit at 388 cycles a
// line, the matrix pipe busy 25 % of the launch.
template <bool OUT_F32>
__global__ __launch_bounds__(512, 4) void fc_big_behind_scan_kernel(
    const void *__restrict__ A0, const void *__restrict__ W0, int lda, int M, int K, int Kpad, int grid_m, int grid_n,
    int tiles_per_group, int per_xcd, int relu, void *__restrict__ C0, int ldc, const float *__restrict__ bias, const ScanBlocks b)
{
    extern __shared__ __attribute__((aligned(16))) __bf16 smem[];
    static_assert(sizeof(scan::ScanShared) <= big_lds_bytes<128, 128>(), "the scan's LDS is part of the tiles'");
    if ((int)blockIdx.x < b.tiles) {
        if (threadIdx.x < SCAN_THREADS)
            scan::scan_offsets_tile(b.lengths, b.n, b.nnz, scan::TileLink{b.words, b.tiles, b.polls}, b.offsets, b.err,
                                    blockIdx.x, *reinterpret_cast<scan::ScanShared *>(smem));
        return;
    }
    struct {
        const void *W[1];
        const float *bias[1];
    } groups{{W0}, {bias}};
    big_block<128, 128, 2, 4, true, OUT_F32>(
        BigLayer{A0, W0, lda, M, K, Kpad, grid_m, grid_n, tiles_per_group, per_xcd, 0, relu, C0, ldc, 0}, groups, smem,
        blockIdx.x - b.tiles);
}

// The same with scan and pooling in further blocks of the launch, for which the layer leaves
// half of a compute unit's registers and LDS, and most of the time of its memory pipes: the layer takes 35 to 38 us
// beside them, 33.5 with the scan alone.  What bounds a pooling block, eight waves on its compute unit: the
// earlier lengths, which it adds up itself (6 us for 80 KB, 10 for 160), then a trip for each of its waves' rounds of
// four bags (3 us with hot rows, 5.8 with cold ones).  us per forward, scan with layer and then pooling / one launch: 10
// tables of 20 fp32 rows of 128 bytes, uniform ids x 4096 samples behind 2560 -> 1024 71.0 / 60.7.
struct PoolBlocks {
    long long nnz;
    int n, per, bags;  // per: blocks of an XCD
    pool::BagTable div;
    int T;
    float one;
    int32_t *offsets;
    ErrRecord *err;
    PoolOut out;
};
struct PoolShared {
    unsigned keys[8 * pool::QUAD_IDS];
    long long sum[8], scan[8];
    int next[4];
    int off[BESIDE_WIDE_BAGS + 4];
    float sums[BESIDE_WIDE_COLUMNS];
};

template <int LPR, bool HALF, bool STREAM>
__global__ __launch_bounds__(512, 4) void fc_big_beside_pool_kernel(
    const void *__restrict__ A0, const void *__restrict__ W0, int lda, int M, int K, int Kpad, int grid_m, int grid_n,
    int tiles, int per_xcd, int relu, void *__restrict__ C0, int ldc, const float *__restrict__ bias,
    const int32_t *__restrict__ lengths, const int32_t *__restrict__ indices, const TableDesc *__restrict__ tables, const PoolBlocks p)
{
    extern __shared__ __attribute__((aligned(16))) __bf16 smem[];
    static_assert(sizeof(PoolShared) <= big_lds_bytes<128, 128>(), "pooling's LDS is part of the tiles'");
    static_assert(BESIDE_WIDE_BAGS <= 64 * pool::QUAD, "a lane to four bags");
    if ((int)blockIdx.x < tiles) {
        struct {
            const void *W[1];
            const float *bias[1];
        } groups{{W0}, {bias}};
        big_block<128, 128, 2, 4, true, false>(
            BigLayer{A0, W0, lda, M, K, Kpad, grid_m, grid_n, tiles, per_xcd, 0, relu, C0, ldc, 0}, groups, smem, blockIdx.x);
        return;
    }
    const int b = blockIdx.x - tiles, first = ((b & 7) * p.per + (b >> 3)) * p.bags;
    if (first >= p.n) return;
    PoolShared &sh = *reinterpret_cast<PoolShared *>(smem);
    if (threadIdx.x < 2) sh.next[threadIdx.x] = threadIdx.x == 0 ? 8 : 0;  // read behind the barriers below
    scan::offsets_of_block<512, 8>(lengths, p.n, p.nnz, first, p.bags, p.offsets, p.err, sh.sum, sh.scan, sh.off);
    pool::pool_quads<8, LPR, HALF, STREAM>(tables, indices, p.out, p.div, p.T, p.n, first, p.bags, sh.off, sh.keys, sh.sums, sh.next, p.one,
                                           p.err);
}

template <int LPR, bool HALF, bool STREAM>
hipError_t launch_beside_pool(const FrontProblem &f, const FcProblem &a, hipStream_t s)
{
    const int n = f.T * f.B, bags = (int)beside_wide_bags(n, f.num_cus);
    const int blocks = ((n + bags - 1) / bags + 7) / 8 * 8;
    const int grid_m = (a.M + 127) / 128, grid_n = a.Npad / 128, tiles = grid_m * grid_n;
    const PoolBlocks p{f.nnz, n, blocks / 8, bags, pool::BagTable::of_batch(f.B), f.T, 1.0f,
                       f.offsets, f.err, f.out};
    hipLaunchKernelGGL((fc_big_beside_pool_kernel<LPR, HALF, STREAM>), dim3(tiles + blocks), dim3(512),
                       (big_lds_bytes<128, 128>()), s, a.A, a.g.W[0], a.lda, a.M, a.K, a.Kpad, grid_m, grid_n, tiles,
                       tiles % 8 == 0 ? tiles / 8 : 0, a.relu ? 1 : 0, a.C, a.ldc, a.g.bias[0], f.lengths, f.indices, f.tables, p);
    return hipGetLastError();
}

template <int LPR>
hipError_t launch_beside_pool(const FrontProblem &f, const FcProblem &a, hipStream_t s)
{
    if (f.dtype == REC_F16)
        return f.stream_rows ? launch_beside_pool<LPR, true, true>(f, a, s) : launch_beside_pool<LPR, true, false>(f, a, s);
    return f.stream_rows ? launch_beside_pool<LPR, false, true>(f, a, s) : launch_beside_pool<LPR, false, false>(f, a, s);
}

template <int LPR>
hipError_t prepare_beside_pool()
{
    constexpr size_t lds = big_lds_bytes<128, 128>();
    hipError_t e = grant_lds(fc_big_beside_pool_kernel<LPR, true, true>, lds);
    if (e == hipSuccess) e = grant_lds(fc_big_beside_pool_kernel<LPR, true, false>, lds);
    if (e == hipSuccess) e = grant_lds(fc_big_beside_pool_kernel<LPR, false, true>, lds);
    if (e == hipSuccess) e = grant_lds(fc_big_beside_pool_kernel<LPR, false, false>, lds);
    return e;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, bool A_F32, bool OUT_F32>
hipError_t launch_big_as(const FcProblem &a, hipStream_t s)
{
    const int grid_m = (a.M + BM - 1) / BM, grid_n = a.Npad / BN;
    const int tiles = grid_m * grid_n;
    const dim3 grid(tiles * a.groups), block(64 * WAVES_M * WAVES_N);
    constexpr size_t lds = big_lds_bytes<BM, BN>();
    auto k = fc_big_kernel<BM, BN, WAVES_M, WAVES_N, A_F32, OUT_F32>;
    hipLaunchKernelGGL(k, grid, block, lds, s, a.A, a.g.W[0], a.lda, a.M, a.K, a.Kpad, grid_m, grid_n, tiles,
                       (int)(grid.x % 8 == 0 ? grid.x / 8 : 0), a.a_stride, a.relu ? 1 : 0, a.C, a.ldc, a.c_stride, a.g);
    return hipGetLastError();
}

template <int BM, int BN, int WAVES_M, int WAVES_N>
hipError_t launch_big(const FcProblem &a, hipStream_t s)
{
    if constexpr (BM == 128) {
        if (a.a_f32) {
            if (a.out_f32) return launch_big_as<BM, BN, WAVES_M, WAVES_N, true, true>(a, s);
            return launch_big_as<BM, BN, WAVES_M, WAVES_N, true, false>(a, s);
        }
    }
    if (a.a_f32) return hipErrorInvalidValue;  // big_tile_choice() has bf16 rows only in these tiles
    if (a.out_f32) return launch_big_as<BM, BN, WAVES_M, WAVES_N, false, true>(a, s);
    return launch_big_as<BM, BN, WAVES_M, WAVES_N, false, false>(a, s);
}

template <int BM, int BN, int WAVES_M, int WAVES_N>
hipError_t prepare_tiles()
{
    constexpr size_t lds = big_lds_bytes<BM, BN>();
    hipError_t e = grant_lds(fc_big_kernel<BM, BN, WAVES_M, WAVES_N, false, false>, lds);
    if (e == hipSuccess) e = grant_lds(fc_big_kernel<BM, BN, WAVES_M, WAVES_N, false, true>, lds);
    if constexpr (BM == 128) {
        if (e == hipSuccess) e = grant_lds(fc_big_kernel<BM, BN, WAVES_M, WAVES_N, true, false>, lds);
        if (e == hipSuccess) e = grant_lds(fc_big_kernel<BM, BN, WAVES_M, WAVES_N, true, true>, lds);
    }
    return e;
}

// Which block tile, if any: 256 x 256, 256 x 128 (bf16 input) or 128 x 128, the
// largest whose tiles still cover three quarters of the compute units (the last: half, against many small ones).
// One stack of bf16 rows beside a pooling launch that is there for long keeps to 1024 rows and three
// quarters: below, launch_fc() has a form of four waves for it that finds room beside pooling's (pipelined
// forwards, us per batch, that form / half a round of these: 40 tables of 80 ids, 4500 samples 281.1 / 283.5; 20
// ids 122.3 / 120.4; 884 -> 1024, 2100 samples, 40 ids 103.0 / 106.8, 80 157.3 / 160.9, 8 57.8 / 53.1).  Several
// stacks and fp32 rows win with these beside any pooling (four of 1728 -> 1024, 600 samples, 1 id 71.8 / 58.9, 80
// 91.4 / 78.1; 2560 fp32 -> 1024, 2100 samples, 20 ids 82.3 / 74.3, 80 103.1 / 92.6).
int big_tile_choice(const FcProblem &a, int num_cus)
{
    const bool keeps = a.corun && !a.a_f32 && a.groups == 1;
    if (a.dot_out || a.M < (keeps ? 1024 : 512) || a.Kpad % BK != 0 || a.groups < 1 || a.groups > MAX_GROUPS) return 0;
    if (a.a_f32 && (a.K % 8 != 0 || a.lda % 4 != 0 || a.a_stride % 4 != 0 ||
                    reinterpret_cast<uintptr_t>(a.A) % 16 != 0))
        return 0;
    const long long need = (long long)num_cus * 3 / 4;
    const long long m256 = (a.M + 255) / 256, m128 = (a.M + 127) / 128;
    if (!a.a_f32 && a.Npad % 256 == 0 && a.groups * m256 * (a.Npad / 256) >= need) return 1;
    if (!a.a_f32 && a.Npad % 128 == 0 && a.groups * m256 * (a.Npad / 128) >= need) return 2;
    const long long tiles = a.groups * m128 * (a.Npad / 128);
    if (a.Npad % 128 == 0 && tiles >= need) return 3;
    // One round of these, at least half full, against three and more of 64 x 64 tiles
    // (csrc/gemm_split.hip).  us per forward, those / these: 2560 fp32 -> 1024, 2060 samples 66.8 / 61.4
    // (136 tiles), 2400 69.7 / 62.5, 2900 70.6 / 64.2; four towers of 1728 -> 1024, 520 samples 42.5 /
    // 42.1 (160), 600 47.7 / 44.0, 800 51.6 / 46.2; three, 900 51.7 / 44.7; with two rounds of 64 x 64
    // (400 samples, 448 of them, 14 us a launch) half a round of these is no shorter.
    if (!keeps && a.Npad % 128 == 0 && 2 * tiles > num_cus && a.groups * ((a.M + 63) / 64) * (a.Npad / 64) > 2 * num_cus) return 3;
    return 0;
}

}  // namespace

bool fc_big_applies(const FcProblem &a, int num_cus) { return big_tile_choice(a, num_cus) != 0; }

FcTile fc_big_tile(const FcProblem &a, int num_cus)
{
    switch (big_tile_choice(a, num_cus)) {
    case 1: return FcTile{16, 16, 1};
    case 2: return FcTile{16, 8, 1};
    case 3: return FcTile{8, 8, 1};
    }
    return FcTile{0, 0, 0};
}

bool fc_big_rides(const FcProblem &a, int num_cus)
{
    return a.a_f32 && a.groups == 1 && !a.corun && num_cus > 0 && big_tile_choice(a, num_cus) == 3;
}

// Where a pooling block, with a quarter of the waves of a launch of its own, is done about when the layer is: by
// its bags, which the layer's depth allows (10 a k-tile), and by its rows (6400 a compute unit).  us per forward, two
// launches / one, Zipf ids; 2560 -> 1024, 10 tables of 20 rows of 128 bytes x 6000 samples 89.8 / 79.5, of 40 of 256 x 4096
// 76.4 / 75.9, 14 of 28 of 64 bytes x 4096 67.2 / 64.2; 1000 -> 1024, 10 of 20 of 128 x 4096 47.6 / 44.4, 4 of 55 x 6000 57.2 /
// 55.7.  Beyond: 2560, 14 of 40 of 256 x 4096 (8960 rows) 93.3 / 96.4, 14 of 50 of 64 x 2500 (6836) 61.8 / 63.4, 30 of 8 x 4096
// (480 bags) 84.2 / 87.8; 1000, 14 of 20 of 64 bytes x 4096 (224 bags) 50.8 / 53.8, 14 of 10 x 6000 64.8 / 72.5.
// For lengths near each other; of geometric ones four bags wait for their longest, which shows where the bags are long and
// their rows hot (Zipf of 1.2): 10 of 20 x 2560 behind 1000 43.5 / 44.2, of 40 46.5 / 51.3, of 40 behind 2560 60.9 / 61.1.
bool fc_big_beside_pool_applies(const FcProblem &a, int T, int B, int D, int dtype, long long nnz, long long max_rows)
{
    const long long n = (long long)T * B;
    const int rowbytes = D * (dtype == REC_F16 ? 2 : 4);
    if (a.out_f32 || !fc_big_rides(a, a.num_cus) || (rowbytes != 64 && rowbytes != 128 && rowbytes != 256)) return false;
    if (!beside_wide_fits(n, D, a.num_cus) || pool_short_applies(rowbytes, nnz, n) || !pool_narrow(max_rows, rowbytes)) return false;
    return n <= (long long)a.num_cus * std::min(240, 10 * (a.Kpad / BK)) && nnz <= 6400ll * a.num_cus && nnz <= 56 * n;
}

hipError_t launch_fc_big_beside_pool(const FrontProblem &f, hipStream_t s)
{
    const FcProblem &a = *f.layer;
    if (f.out.z || f.num_cus <= 0 || a.out_f32 || !fc_big_rides(a, f.num_cus) || !beside_wide_fits((long long)f.T * f.B, f.D, f.num_cus))
        return hipErrorInvalidValue;
    switch (f.D * (f.dtype == REC_F16 ? 2 : 4) / 16) {
    case 4: return launch_beside_pool<4>(f, a, s);
    case 8: return launch_beside_pool<8>(f, a, s);
    case 16: return launch_beside_pool<16>(f, a, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_fc_big_behind_scan(const FcProblem &a, const ScanBlocks &scan, hipStream_t s)
{
    const int grid_m = (a.M + 127) / 128, grid_n = a.Npad / 128, tiles = grid_m * grid_n;
    auto k = a.out_f32 ? fc_big_behind_scan_kernel<true> : fc_big_behind_scan_kernel<false>;
    hipLaunchKernelGGL(k, dim3(scan.tiles + tiles), dim3(512), (big_lds_bytes<128, 128>()), s, a.A, a.g.W[0], a.lda, a.M, a.K,
                       a.Kpad, grid_m, grid_n, tiles, tiles % 8 == 0 ? tiles / 8 : 0, a.relu ? 1 : 0, a.C, a.ldc, a.g.bias[0], scan);
    return hipGetLastError();
}

hipError_t fc_big_prepare()
{
    hipError_t e = grant_lds(fc_big_behind_scan_kernel<true>, big_lds_bytes<128, 128>());
    if (e == hipSuccess) e = grant_lds(fc_big_behind_scan_kernel<false>, big_lds_bytes<128, 128>());
    if (e == hipSuccess) e = prepare_beside_pool<4>();
    if (e == hipSuccess) e = prepare_beside_pool<8>();
    if (e == hipSuccess) e = prepare_beside_pool<16>();
    if (e == hipSuccess) e = prepare_tiles<256, 256, 2, 4>();
    if (e == hipSuccess) e = prepare_tiles<256, 128, 4, 2>();
    if (e == hipSuccess) e = prepare_tiles<128, 128, 2, 4>();
    return e;
}

hipError_t launch_fc_big(const FcProblem &a, int num_cus, hipStream_t s)
{
    switch (big_tile_choice(a, num_cus)) {
    case 1: return launch_big<256, 256, 2, 4>(a, s);
    case 2: return launch_big<256, 128, 4, 2>(a, s);
    case 3: return launch_big<128, 128, 2, 4>(a, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace rec
