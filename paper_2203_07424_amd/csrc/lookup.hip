// S0 and S1 of a concatenation model without Bottom-FC in one launch, for more lookups than
// front_short_kernel (csrc/front.hip) is for: about one id a bag, few blocks of many bags, so that
// each can read all earlier lengths; the offsets and their checks come from them too.  Behind its
// blocks those that narrow the dense part.  What bounds it: the last block's half a megabyte
// of lengths, then a trip for ids and one for rows: 26 tables x 4096 11.8 us against 7.4 + 7.6 in two launches, from
// cold memory 15.1 against 9.0 + 10.2 (in four trips for the lengths instead of one 16.9).  us per forward, two launches /
// one, with towers of 96-72: 26 fp16 tables of 64 x 500 16.9 / 14.9, x 1923 23.8 / 20.1, x 4096 30.0 / 26.6, x 5000
// (130 000 bags) 32.5 / 31.4; 13 fp32 of 64 x 3846 22.6 / 18.4; in more blocks than compute units (256 bags a block
// there) x 5076 27.0 / 27.5, x 8192 30.3 / 32.1.
// Only the mean of the bags' lengths is known in advance; us per forward, two launches / one, 26 of 64 with 1 % of bags of
// 20 ids x 600 22.1 / 19.9, x 4096 37.9 / 30.3, one bag of 2000 x 600 515 / 195, one table of 6 ids x 600 16.9 / 16.8.
#include <algorithm>

#include "pool_body.h"
#include "scan_body.h"

namespace rec {

namespace {

using namespace scan;
using namespace pool;

// A thread for each bag of a block at most, LOOKUP_BAGS bags for each group of lanes that loads a row.
constexpr int LOOKUP_THREADS = 1024, LOOKUP_BAGS = 4;
constexpr int MOST_LOOKUPS = 64 * SCAN_TILE;

// Bags of one block: consecutive, each group of LPR lanes taking
// LOOKUP_BAGS of them a block's groups apart.
template <int LPR>
constexpr int lookup_block_bags() { return LOOKUP_THREADS / LPR * LOOKUP_BAGS; }

template <int LPR, bool HALF>
__global__ __launch_bounds__(LOOKUP_THREADS) void front_lookup_kernel(
    const int32_t *__restrict__ len, const TableDesc *__restrict__ tables, const int32_t *__restrict__ indices,
    long long nnz, int n, int blocks, int extra, int per, unsigned B, unsigned magic, int T, float one, int vec_ok,
    int32_t *__restrict__ offsets, ErrRecord *err, const PoolOut out, const ConcatDense job)
{
    constexpr int THREADS = LOOKUP_THREADS, WAVES = THREADS / 64, GROUPS = THREADS / LPR, BAGS = lookup_block_bags<LPR>();
    static_assert(BAGS <= THREADS, "a thread per bag of the block");
    int b = blockIdx.x;
    if (b >= blocks) {
        concat_dense_block<THREADS>(job, b - blocks, extra);
        return;
    }
    const BagTable div{B, magic};
    const int first = ((b & 7) * per + (b >> 3)) * BAGS;
    if (first >= n) return;
    __shared__ long long s_w[WAVES], s_scan[WAVES];
    __shared__ int s_off[BAGS + 1];
    offsets_of_block<THREADS, 26>(len, n, nnz, first, BAGS, offsets, err, s_w, s_scan, s_off);
    const int group = threadIdx.x / LPR;
    bool live[LOOKUP_BAGS];
    int bag[LOOKUP_BAGS], pos[LOOKUP_BAGS], end[LOOKUP_BAGS];
#pragma unroll
    for (int g = 0; g < LOOKUP_BAGS; ++g) {
        const int at = group + g * GROUPS;
        live[g] = first + at < n;
        bag[g] = live[g] ? first + at : n - 1;
        pos[g] = s_off[at];
        end[g] = live[g] ? s_off[at + 1] : pos[g];
    }
    pool_short_bags<LPR, HALF, true, LOOKUP_BAGS, 1, true>(tables, indices, out, vec_ok, div, T, live, bag, pos, end, one, err);
}

template <int LPR, bool HALF>
hipError_t launch_lookup(const FrontProblem &f, hipStream_t s)
{
    constexpr int NACC = HALF ? 8 : 4, BAGS = lookup_block_bags<LPR>();
    const int n = f.T * f.B;
    const int vec_ok = f.out.col0 % NACC == 0 && reinterpret_cast<uintptr_t>(f.out.z) % 16 == 0;
    const BagTable div = BagTable::of_batch(f.B);
    const int blocks = ((n + BAGS - 1) / BAGS + 7) / 8 * 8;
    const int extra = lookup_dense_blocks(f.dense, f.num_cus - blocks);
    hipLaunchKernelGGL((front_lookup_kernel<LPR, HALF>), dim3(blocks + extra), dim3(LOOKUP_THREADS), 0, s, f.lengths, f.tables,
                       f.indices, f.nnz, n, blocks, extra, blocks / 8, div.B, div.magic, f.T, 1.0f, vec_ok, f.offsets, f.err,
                       f.out, f.dense);
    return hipGetLastError();
}

}  // namespace

// A block for each compute unit that the others leave, as long as a wave is done with its units when these are; else
// so many that they come behind them, on all compute units (one more than there are compute units is a round: 13 tables x
// 7000 samples with 300 features, a block a unit that is left / nine more 25.3 / 29.6 us per forward; 26 x 2400, eight left, 12
// units a wave / four 29.4 / 24.4, 1000 features 32.2 / 26.1).
int lookup_dense_blocks(const ConcatDense &job, int left)
{
    constexpr int WAVES = LOOKUP_THREADS / 64;
    if (concat_dense_blocks(job, WAVES, 12) <= left) return std::min(concat_dense_blocks(job, WAVES, 2), left);
    return concat_dense_blocks(job, WAVES, 4);
}

bool front_lookup_applies(int T, int B, int D, int dtype, long long nnz, int num_cus)
{
    const long long n = (long long)T * B;
    const int rowbytes = D * (dtype == REC_F16 ? 2 : 4);
    if (rowbytes != 64 && rowbytes != 128 && rowbytes != 256) return false;
    const long long one_round = (long long)num_cus * (LOOKUP_THREADS * 16 / rowbytes * LOOKUP_BAGS);
    return n > SHORT_FORM_BAGS && n <= std::min<long long>(MOST_LOOKUPS, one_round) && nnz <= n + n / 4;
}

hipError_t launch_lookups(const FrontProblem &f, hipStream_t s)
{
    if (!f.out.z || !f.dense.x0 || f.layer) return hipErrorInvalidValue;
    const bool half = f.dtype == REC_F16;
    switch (f.D * (half ? 2 : 4) / 16) {
    case 4: return half ? launch_lookup<4, true>(f, s) : launch_lookup<4, false>(f, s);
    case 8: return half ? launch_lookup<8, true>(f, s) : launch_lookup<8, false>(f, s);
    case 16: return half ? launch_lookup<16, true>(f, s) : launch_lookup<16, false>(f, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace rec
