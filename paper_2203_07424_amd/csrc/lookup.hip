// S0 and S1 of a concatenation model without Bottom-FC in one launch, for more lookups than
// front_short_kernel (csrc/front.hip) is for: about one id a bag, few blocks of many bags, so that
// each can read all earlier lengths; the offsets and their checks come from them too.  Behind its
// blocks those that narrow the dense part.  What bounds it: the last block's half a megabyte
// of lengths, then a trip for ids and one for rows: 26 tables x 4096 11.8 us against 7.4 + 7.6 in two launches, from
// cold memory 15.1 against 9.0 + 10.2 (in four trips for the lengths instead of one 16.9).  us per forward, two launches /
// one, with towers of 96-72: 26 fp16 tables of 64 x 500 16.9 / 14.9, x 1923 23.8 / 20.1, x 4096 30.0 / 26.6, x 5000
// (130 000 bags) 32.5 / 31.4; 13 fp32 of 64 x 3846 22.6 / 18.4; in more blocks than compute units (256 bags a block
// there) x 5076 27.0 / 27.5, x 8192 30.3 / 32.1.
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

// As part_of_sum(), over up to 2048 lengths a thread, n not zero: loads past n read zeros (a buffer's range
// check), and of each length there is an addition and an "or", in 32 bits; a thread that has seen a bit from the
// 20th on (a sign among them) adds its lengths up again in 64.  426 KB by a block of 1024 threads: 104 lengths
// a thread, some 5 vector instructions each in part_of_sum() (a launch of 13.2 us, 11.8 with this).
template <int THREADS, int U>
__device__ inline long long part_of_long_sum(const int32_t *__restrict__ len, int n)
{
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t *>(len), 0, n * 4, 0x00020000);
    unsigned sum = 0, seen = 0;
    for (int k0 = 4 * (int)threadIdx.x; k0 < n; k0 += 4 * THREADS * U) {
        u32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = __builtin_amdgcn_raw_buffer_load_b128(src, (k0 + u * 4 * THREADS) * 4, 0, 0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            sum += v[u][0] + v[u][1];
            sum += v[u][2] + v[u][3];
            seen |= v[u][0] | v[u][1];
            seen |= v[u][2] | v[u][3];
        }
    }
    if (seen >> 20 == 0) return sum;
    long long exact = 0;
    for (int k0 = 4 * (int)threadIdx.x; k0 < n; k0 += 4 * THREADS)
        for (int e = 0; e < 4; ++e) exact += max(len[k0 + e], 0);
    return exact;
}

// Sum over max(len, 0) of lengths [0, n) by all threads of the block, in one trip where these are up to
// 104 a thread; s_w: a word per wave.
template <int THREADS>
__device__ inline long long sum_before(const int32_t *__restrict__ len, int n, long long *s_w)
{
    const long long sum = wave_sum(n <= 4 * 8 * THREADS ? part_of_long_sum<THREADS, 8>(len, n) : part_of_long_sum<THREADS, 26>(len, n));
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = sum;
    __syncthreads();
    long long all = 0;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) all += s_w[w];
    return all;
}

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
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int k = first + tid;
    int own = tid < BAGS && k < n ? len[k] : 0;
    if (own < 0) {  // counts as 0
        atomicMin(&err->first_bad_len, (unsigned long long)k);
        atomicOr(&err->flags, ERR_NEG_LENGTH);
        own = 0;
    }
    long long incl = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const long long up = __shfl_up(incl, o, 64);
        if (lane >= o) incl += up;
    }
    if (lane == 63) s_scan[wave] = incl;
    long long run = sum_before<THREADS>(len, first, s_w);  // its barrier makes s_scan visible too
    for (int w = 0; w < wave; ++w) run += s_scan[w];
    run += incl;
    if (tid < BAGS) {
        s_off[tid] = (int)min(run - own, nnz);
        if (k < n) offsets[k] = (int)min(run - own, nnz);
        if (tid == BAGS - 1) s_off[BAGS] = (int)min(run, nnz);
        if (k == n - 1) {
            offsets[n] = (int)min(run, nnz);
            if (run != nnz) atomicOr(&err->flags, ERR_TOTAL_MISMATCH);
        }
    }
    __syncthreads();
    const int group = tid / LPR;
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
    pool_short_bags<LPR, HALF, true, LOOKUP_BAGS, 1>(tables, indices, out, vec_ok, div, T, live, bag, pos, end, one, err);
}

template <int LPR, bool HALF>
hipError_t launch_lookup(const FrontProblem &f, hipStream_t s)
{
    constexpr int NACC = HALF ? 8 : 4, BAGS = lookup_block_bags<LPR>();
    const int n = f.T * f.B;
    const int vec_ok = f.out.col0 % NACC == 0 && reinterpret_cast<uintptr_t>(f.out.z) % 16 == 0;
    const BagTable div = BagTable::of_batch(f.B);
    const int blocks = ((n + BAGS - 1) / BAGS + 7) / 8 * 8;
    // as many as the compute units that the others leave, a block each
    const int extra = concat_dense_blocks(f.dense, LOOKUP_THREADS / 64, std::max(16, f.num_cus - blocks));
    hipLaunchKernelGGL((front_lookup_kernel<LPR, HALF>), dim3(blocks + extra), dim3(LOOKUP_THREADS), 0, s, f.lengths, f.tables,
                       f.indices, f.nnz, n, blocks, extra, blocks / 8, div.B, div.magic, f.T, 1.0f, vec_ok, f.offsets, f.err,
                       f.out, f.dense);
    return hipGetLastError();
}

}  // namespace

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
