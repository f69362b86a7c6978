// S1: embedding-bag pooling (SparseLengthsSum; "Gather-Reduce", Sec. VI-B).
//
// pooled[b][t][:] = sum of rows E_t[id][:] over the ids of bag (t, b).
//
// One 64-lane wavefront per bag.  A row is D * sizeof(element) bytes; a lane
// moves 16 bytes (one 128-bit load), so LPR = rowbytes / 16 lanes cover a row
// and one wave-wide load fetches RPW = 64 / LPR different rows of the bag.
// The wave reads 64 ids with one coalesced load, hands them out by cross-lane
// permute, keeps several row loads in flight, accumulates in fp32 and folds the
// RPW partial sums in a fixed order, so results do not vary from run to run.
//
// The work is random-gather traffic, but a wave64 vector instruction holds its
// SIMD for four cycles, and a version that spent some 33 vector instructions
// per wave-wide load (address arithmetic, validity selects, widen + select +
// add per element) was bound by instruction issue even with every row in the
// L1.  Per wave-wide load the loop below spends one permute, one add, the load
// and one fused multiply-add per element: rows come through a buffer descriptor
// whose range check returns zero for the offsets that stand for "no row", the
// permute's slot is an immediate, and loads a partial group does not need are
// skipped by wave-uniform branches.
//
// Bags of a few ids (one lookup per table and no pooling, Table I row MT-WnD)
// would leave most of such a wave idle: pool_short_kernel gives each group of
// LPR lanes a bag of its own, RPW bags per wave.  (Giving bags of 20-50 ids, the
// DLRM-RMC3 range of Table I, 4 * LPR lanes each was measured too: slower than
// one wave per bag.)
//
// STREAM: the rows are loaded with the non-temporal hint (they are not kept in
// the caches ahead of other lines).  For id streams without reuse (uniform ids)
// that is 2.5 % faster; for skewed ids, whose hot rows the caches serve, it is
// 20 % slower, so it is an option the caller sets from what it knows of its ids.
//
// In the concatenation model the sums go, narrowed to bf16, straight into the
// Predict-FC input row of their sample (concatenation and conversion fused,
// Sec. IV-A) instead of the fp32 pooled buffer.
#include "pool_body.h"

namespace rec {

namespace {

using namespace pool;

// Arguments: a wave starts with the leading 14 words of them in registers, as far as they
// are scalars; the rest, and the launch's own sizes (gridDim), are a trip to cold memory.
// So what stands between a wave and its first loads comes first, structs last.

template <int LPR, bool HALF, bool CONCAT, bool STREAM, bool NARROW>
__global__ __launch_bounds__(POOL_WAVES * 64) void pool_kernel(
    const TableDesc *__restrict__ tables, const int32_t *__restrict__ indices,
    const int32_t *__restrict__ offsets, int per, int nbags, unsigned B, unsigned magic, int T, float one,
    int vec_ok, ErrRecord *err, const PoolOut out, const TileWords left)
{
    // Blocks are handed to the 8 XCDs round-robin; give XCD x the x-th eighth
    // of the (table-major) bag list so that each L2 sees few tables at a time.
    // The grid is 8 per blocks; surplus blocks fall past nbags.
    const BagTable div{B, magic};
    const int vblk = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    int bag = vblk * POOL_WAVES + (threadIdx.x >> 6);
    if (bag >= nbags) return;
    bag = __builtin_amdgcn_readfirstlane(bag);
    const int t = div.of(bag);
    pool_bag<LPR, HALF, CONCAT, STREAM, NARROW>(tables, indices, out, vec_ok, T, bag - t * (int)div.B, t,
                                                offsets[bag],
                                                offsets[bag + 1], one, err);
    if (bag == 0) clear_tile_words(left);  // last: its arguments are not waited for in front of the first id
}

// Group g of the launch takes bags g, g + groups, ...
template <int LPR, bool HALF, bool CONCAT>
__global__ __launch_bounds__(POOL_WAVES * 64) void pool_short_kernel(
    const TableDesc *__restrict__ tables, const int32_t *__restrict__ indices,
    const int32_t *__restrict__ offsets, int per, int nbags, unsigned B, unsigned magic, int T, float one,
    int groups, int vec_ok, ErrRecord *err, const PoolOut out, const TileWords left)
{
    constexpr int RPW = 64 / LPR;
    const BagTable div{B, magic};
    const int vblk = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    const long long group = ((long long)vblk * POOL_WAVES + (threadIdx.x >> 6)) * RPW + (threadIdx.x & 63) / LPR;
    bool live[SHORT_BAGS];
    int bag[SHORT_BAGS], pos[SHORT_BAGS], end[SHORT_BAGS];
#pragma unroll
    for (int g = 0; g < SHORT_BAGS; ++g) {
        const long long slot = group + (long long)g * groups;
        live[g] = slot < nbags;
        bag[g] = live[g] ? (int)slot : nbags - 1;
        pos[g] = offsets[bag[g]];
        end[g] = live[g] ? offsets[bag[g] + 1] : pos[g];
    }
    pool_short_bags<LPR, HALF, CONCAT>(tables, indices, out, vec_ok, div, T, live, bag, pos, end, one, err);
    if (blockIdx.x == 0 && threadIdx.x < 64) clear_tile_words(left);
}

template <int LPR, bool HALF, bool CONCAT>
hipError_t launch_shape(bool short_bags, bool stream_rows, bool narrow, const TableDesc *tables, int T, int B, const int32_t *indices,
                        const int32_t *offsets, const PoolOut &out, const TileWords &left, ErrRecord *err, hipStream_t s)
{
    constexpr int NACC = HALF ? 8 : 4;
    const int nbags = T * B;
    const int vec_ok = CONCAT && out.col0 % NACC == 0 && reinterpret_cast<uintptr_t>(out.z) % 16 == 0;
    const dim3 block(POOL_WAVES * 64);
    const BagTable div = BagTable::of_batch(B);
    if (short_bags) {
        const int groups_per_block = POOL_WAVES * (64 / LPR);
        const int per_block = groups_per_block * SHORT_BAGS;
        const dim3 grid(((nbags + per_block - 1) / per_block + 7) / 8 * 8);
        const int groups = (int)grid.x * groups_per_block;
        hipLaunchKernelGGL((pool_short_kernel<LPR, HALF, CONCAT>), grid, block, 0, s, tables, indices,
                           offsets, (int)grid.x / 8, nbags, div.B, div.magic, T, 1.0f, groups, vec_ok, err, out, left);
    } else {
        const dim3 grid(((nbags + POOL_WAVES - 1) / POOL_WAVES + 7) / 8 * 8);
#define REC_POOL_LAUNCH(STREAM, NARROW)                                                                  \
    hipLaunchKernelGGL((pool_kernel<LPR, HALF, CONCAT, STREAM, NARROW>), grid, block, 0, s, tables, indices, \
                       offsets, (int)grid.x / 8, nbags, div.B, div.magic, T, 1.0f, vec_ok, err, out, left)
        if (stream_rows) {
            if (narrow) REC_POOL_LAUNCH(true, true); else REC_POOL_LAUNCH(true, false);
        } else {
            if (narrow) REC_POOL_LAUNCH(false, true); else REC_POOL_LAUNCH(false, false);
        }
#undef REC_POOL_LAUNCH
    }
    return hipGetLastError();
}

template <int LPR>
hipError_t launch_lpr(bool half, bool short_bags, bool stream_rows, bool narrow, const TableDesc *tables, int T, int B,
                      const int32_t *indices, const int32_t *offsets, const PoolOut &out, const TileWords &left,
                      ErrRecord *err, hipStream_t s)
{
    if (out.z) {
        if (half) return launch_shape<LPR, true, true>(short_bags, stream_rows, narrow, tables, T, B, indices, offsets, out, left, err, s);
        return launch_shape<LPR, false, true>(short_bags, stream_rows, narrow, tables, T, B, indices, offsets, out, left, err, s);
    }
    if (half) return launch_shape<LPR, true, false>(short_bags, stream_rows, narrow, tables, T, B, indices, offsets, out, left, err, s);
    return launch_shape<LPR, false, false>(short_bags, stream_rows, narrow, tables, T, B, indices, offsets, out, left, err, s);
}

}  // namespace

bool pool_short_applies(int rowbytes, long long nnz, long long bags)
{
    return rowbytes < 1024 && nnz <= SHORT_MEAN * bags;
}

// 32-bit byte offsets reach every row, and leave room above the table for the
// offsets that stand for "no row".
bool pool_narrow(long long max_rows, int rowbytes) { return max_rows * rowbytes <= 0xFFFF0000ll; }

hipError_t launch_pool(const TableDesc *tables, int dtype, int T, int D, int B,
                       const int32_t *indices, const int32_t *offsets, PoolOut out, long long nnz,
                       bool stream_rows, long long max_rows, const TileWords &left, ErrRecord *err, hipStream_t s)
{
    if (T <= 0 || B <= 0) return hipSuccess;
    const bool half = dtype == REC_F16;
    const int rowbytes = D * (half ? 2 : 4);
    const bool narrow = pool_narrow(max_rows, rowbytes);
    const bool sh = pool_short_applies(rowbytes, nnz, (long long)T * B);
    switch (rowbytes / 16) {
    case 1: return launch_lpr<1>(half, sh, stream_rows, narrow, tables, T, B, indices, offsets, out, left, err, s);
    case 2: return launch_lpr<2>(half, sh, stream_rows, narrow, tables, T, B, indices, offsets, out, left, err, s);
    case 4: return launch_lpr<4>(half, sh, stream_rows, narrow, tables, T, B, indices, offsets, out, left, err, s);
    case 8: return launch_lpr<8>(half, sh, stream_rows, narrow, tables, T, B, indices, offsets, out, left, err, s);
    case 16: return launch_lpr<16>(half, sh, stream_rows, narrow, tables, T, B, indices, offsets, out, left, err, s);
    case 32: return launch_lpr<32>(half, sh, stream_rows, narrow, tables, T, B, indices, offsets, out, left, err, s);
    case 64: return launch_lpr<64>(half, sh, stream_rows, narrow, tables, T, B, indices, offsets, out, left, err, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace rec
