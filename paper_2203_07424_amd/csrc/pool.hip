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

// Two neighbouring bags of a table by one wave, one after the other: the ids of both in one
// trip, and no store before the last row.  (Behind a store the next bag's loads wait until it
// has reached memory: loads and stores count in one order.)  With a wave a bag the trips
// to a bag's offsets and ids are about a quarter of its life.  60 tables x 16384 samples on changing inputs
// 645 -> 604 us per forward (in another run, 650 -> 610, four bags a wave 605, eight 615).  For launches of many rounds of waves, where the longer
// life of the last ones does not show: 40 x 4096, 20 rounds, 160.5 -> 161.3.
// Waves share nothing, so a block is one of them: its slot is taken again when it ends and
// not when the last of four does (632 -> 618).  Waves that live for one bag, and for short ones above
// all, come faster in fours (12 x 1737 of 9 ids, a wave a bag, 21.7 -> 23.2 in ones).  Beside launches that want wave
// slots these blocks are larger, or the others find none between them: eight waves, and four in a launch so long that the
// others are the smaller part of it.  Eight pipelined batches, us with a wave a bag / two bags in blocks of one wave, four, eight:
// 40 x 4096 of 80 ids 1273 / 1422, 1419, 1275, of 20 727 / -, 789, 706; 60 x 4096 1809 / -, 1960, 1805; 40 x 8000 2321 / -,
// 2268, 2205; 40 x 16384 of 20 2466 / -, 2192, 2390; 60 x 16384 6248 / -, 6079, 6379.
constexpr int TWO_IDS = 256;  // of the two bags, or they are taken as two waves would

template <int LPR, bool HALF, bool STREAM>
__global__ __launch_bounds__(512) void pool_two_kernel(
    const TableDesc *__restrict__ tables, const int32_t *__restrict__ indices,
    const int32_t *__restrict__ offsets, int per, int npairs, unsigned pairs, unsigned magic, int T, float one,
    int B, int log_waves, ErrRecord *err, const PoolOut out, const TileWords left)
{
    typedef RowSource<LPR * 16, true, STREAM> Rows;
    constexpr int RPW = 64 / LPR, CHUNKS = TWO_IDS / 64, D = LPR * 16 / (HALF ? 2 : 4);
    extern __shared__ unsigned two_keys[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const BagTable div{pairs, magic};
    const int vblk = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    int pair = (vblk << log_waves) + wave;
    if (pair >= npairs) return;
    pair = __builtin_amdgcn_readfirstlane(pair);
    const int t = div.of(pair), b = 2 * (pair - t * (int)pairs), bag = t * B + b;
    const bool both = b + 1 < B;
    int start[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) start[i] = offsets[bag + (i < 2 || both ? i : 1)];
    const int total = start[2] - start[0];
    if (total > TWO_IDS) {
        for (int i = 0; i < (both ? 2 : 1); ++i)
            pool_bag<LPR, HALF, false, STREAM, true>(tables, indices, out, 0, T, b + i, t, offsets[bag + i],
                                                     offsets[bag + i + 1], one, err);
    } else {
        const long long rows = tables[t].rows;
        int id[CHUNKS];
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
            id[c] = -1;
            if (c * 64 + lane < total) id[c] = indices[start[0] + c * 64 + lane];
        }
        // What a lane hands out goes through LDS, where a bag may start anywhere.
        unsigned *keys = two_keys + wave * TWO_IDS;
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
            if (c * 64 >= total) break;
            // Ids outside the table contribute zero and leave a record.
            if (c * 64 + lane < total && (unsigned long long)(long long)id[c] >= (unsigned long long)rows) {
                atomicMin(&err->first_bad_idx, (unsigned long long)(start[0] + c * 64 + lane));
                atomicOr(&err->flags, ERR_INDEX_RANGE);
                id[c] = -1;
            }
            keys[c * 64 + lane] = Rows::key(id[c]);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const int sub = row_of_lane<LPR>(lane);
        const Rows src(tables[t].base, rows, lane % LPR);
        Acc<HALF> acc[2];
        int col = 0;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
#pragma unroll
            for (int e = 0; e < Acc<HALF>::N; ++e) acc[i].v[e] = 0.0f;
            const int n = start[i + 1] - start[i], full = n / RPW;  // wave-wide loads all of whose rows are there
            const unsigned *mine = keys + (start[i] - start[0]) + sub;
            int j = 0;
            for (; j + POOL_UNROLL <= full; j += POOL_UNROLL) {
                u32x4 raw[POOL_UNROLL];
#pragma unroll
                for (int u = 0; u < POOL_UNROLL; ++u) raw[u] = src.fetch(mine[(j + u) * RPW]);
#pragma unroll
                for (int u = 0; u < POOL_UNROLL; ++u) accumulate<HALF>(acc[i], raw[u], one);
            }
            if (j * RPW < n) {
                u32x4 raw[POOL_UNROLL];
#pragma unroll
                for (int u = 0; u < POOL_UNROLL; ++u)
                    if ((j + u) * RPW < n) {
                        const int at = (j + u) * RPW;
                        raw[u] = src.fetch(at + sub < n ? mine[at] : Rows::key(-1));
                    }
#pragma unroll
                for (int u = 0; u < POOL_UNROLL; ++u)
                    if ((j + u) * RPW < n) accumulate<HALF>(acc[i], raw[u], one);
            }
            col = fold_sums<LPR, HALF>(acc[i], lane, lane % LPR);
        }
        if (LPR > 8 || (lane & 15) < LPR) {
            store_sums<folded_columns<LPR, HALF>(), false>(acc[0].v, out, 0, b, t, T, D, col);
            if (both) store_sums<folded_columns<LPR, HALF>(), false>(acc[1].v, out, 0, b + 1, t, T, D, col);
        }
    }
    if (pair == 0) clear_tile_words(left);
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

// What a launch gets besides its template parameters.
struct PoolProblem {
    const TableDesc *tables;
    int T, B;
    const int32_t *indices, *offsets;
    PoolOut out;
    TileWords left;
    ErrRecord *err;
    bool short_bags, two_bags, stream_rows, narrow, corun;
    int num_cus;
};

template <int LPR, bool HALF, bool CONCAT>
hipError_t launch_shape(const PoolProblem &p, hipStream_t s)
{
    constexpr int NACC = HALF ? 8 : 4;
    const int nbags = p.T * p.B;
    const int vec_ok = CONCAT && p.out.col0 % NACC == 0 && reinterpret_cast<uintptr_t>(p.out.z) % 16 == 0;
    const auto blocks_of = [](int n, int per_block) { return dim3(((n + per_block - 1) / per_block + 7) / 8 * 8); };
    const dim3 block(POOL_WAVES * 64);
    const BagTable div = BagTable::of_batch(p.B);
    if (p.short_bags) {
        const int groups_per_block = POOL_WAVES * (64 / LPR);
        const dim3 grid = blocks_of(nbags, groups_per_block * SHORT_BAGS);
        const int groups = (int)grid.x * groups_per_block;
        hipLaunchKernelGGL((pool_short_kernel<LPR, HALF, CONCAT>), grid, block, 0, s, p.tables, p.indices, p.offsets,
                           (int)grid.x / 8, nbags, div.B, div.magic, p.T, 1.0f, groups, vec_ok, p.err, p.out, p.left);
        return hipGetLastError();
    }
    if constexpr (!CONCAT && LPR >= 4 && LPR <= 16) {
        if (p.two_bags) {
            const BagTable by_pair = BagTable::of_batch((p.B + 1) / 2);
            const int npairs = p.T * (int)by_pair.B, log_waves = !p.corun ? 0 : nbags < 64 * 32 * p.num_cus ? 3 : 2, waves = 1 << log_waves;
            const dim3 grid = blocks_of(npairs, waves);
            auto k = p.stream_rows ? pool_two_kernel<LPR, HALF, true> : pool_two_kernel<LPR, HALF, false>;
            hipLaunchKernelGGL(k, grid, dim3(waves * 64), waves * TWO_IDS * sizeof(unsigned), s, p.tables, p.indices, p.offsets,
                               (int)grid.x / 8, npairs, by_pair.B, by_pair.magic, p.T, 1.0f, p.B, log_waves, p.err, p.out, p.left);
            return hipGetLastError();
        }
    }
    const dim3 grid = blocks_of(nbags, POOL_WAVES);
    auto k = p.stream_rows ? (p.narrow ? pool_kernel<LPR, HALF, CONCAT, true, true> : pool_kernel<LPR, HALF, CONCAT, true, false>)
                           : (p.narrow ? pool_kernel<LPR, HALF, CONCAT, false, true> : pool_kernel<LPR, HALF, CONCAT, false, false>);
    hipLaunchKernelGGL(k, grid, block, 0, s, p.tables, p.indices, p.offsets, (int)grid.x / 8, nbags, div.B, div.magic, p.T, 1.0f,
                       vec_ok, p.err, p.out, p.left);
    return hipGetLastError();
}

template <int LPR>
hipError_t launch_lpr(bool half, const PoolProblem &p, hipStream_t s)
{
    if (p.out.z) return half ? launch_shape<LPR, true, true>(p, s) : launch_shape<LPR, false, true>(p, s);
    return half ? launch_shape<LPR, true, false>(p, s) : launch_shape<LPR, false, false>(p, s);
}

}  // namespace

bool pool_short_applies(int rowbytes, long long nnz, long long bags)
{
    return rowbytes < 1024 && nnz <= SHORT_MEAN * bags;
}

// Rows of 64 to 256 bytes, bags whose ids fit, and more rounds of waves the longer a wave lives.  us per forward, a
// wave a bag / two bags a wave, Zipf and uniform ids; 10 ids of 128 bytes, 42 000 bags 31.1 / 29.8 and 33.8 / 32.0, 500 000 of
// 64 bytes 173 / 142 and 195 / 166; 30 of 128, 36 000 bags 26.6 / 26.0 and 38.7 / 39.6, 66 000 37.0 / 34.5 and
// 65.2 / 64.1; 20 of 256, 66 000 45.5 / 43.3 and 84.7 / 85.0; 80 of 128, 200 000 167.5 / 165.0 and 337 / 336 (but
// 2 M rows a table, 164 000 bags, 160.5 / 161.3); 40 of 256, 150 000 135.5 / 136.4, 500 000 379.3 / 379.1; 110 of
// 64, 260 000 226.1 / 227.9 and 465.8 / 467.1.
bool pool_two_applies(int rowbytes, long long nnz, long long bags, bool narrow, int num_cus)
{
    if (!narrow || rowbytes < 64 || rowbytes > 256 || nnz > 88 * bags) return false;
    const long long round = 32ll * num_cus, bytes = nnz * rowbytes;
    return bags >= (bytes <= 2048 * bags ? 5 : bytes <= 4096 * bags ? 8 : 24) * round;
}

// 32-bit byte offsets reach every row, and leave room above the table for the
// offsets that stand for "no row".
bool pool_narrow(long long max_rows, int rowbytes) { return max_rows * rowbytes <= 0xFFFF0000ll; }

hipError_t launch_pool(const TableDesc *tables, int dtype, int T, int D, int B,
                       const int32_t *indices, const int32_t *offsets, PoolOut out, long long nnz,
                       bool stream_rows, long long max_rows, int num_cus, bool corun, const TileWords &left, ErrRecord *err,
                       hipStream_t s)
{
    if (T <= 0 || B <= 0) return hipSuccess;
    const bool half = dtype == REC_F16;
    const int rowbytes = D * (half ? 2 : 4);
    const long long bags = (long long)T * B;
    const bool narrow = pool_narrow(max_rows, rowbytes), short_bags = pool_short_applies(rowbytes, nnz, bags);
    const PoolProblem p{tables, T, B, indices, offsets, out, left, err, short_bags,
                        pool_two_applies(rowbytes, nnz, bags, narrow, num_cus), stream_rows, narrow, corun, num_cus};
    switch (rowbytes / 16) {
    case 1: return launch_lpr<1>(half, p, s);
    case 2: return launch_lpr<2>(half, p, s);
    case 4: return launch_lpr<4>(half, p, s);
    case 8: return launch_lpr<8>(half, p, s);
    case 16: return launch_lpr<16>(half, p, s);
    case 32: return launch_lpr<32>(half, p, s);
    case 64: return launch_lpr<64>(half, p, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace rec
