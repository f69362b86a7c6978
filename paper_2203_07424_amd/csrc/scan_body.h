// Bodies of the scan's kernels (csrc/scan.hip has the description) as device
// functions, for the launches that do more than the scan.
#ifndef REC_SCAN_BODY_H
#define REC_SCAN_BODY_H
#include <algorithm>

#include "rec_internal.h"

namespace rec {
namespace scan {

__device__ inline long long wave_sum(long long v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    return v;  // valid in lane 0
}

// Sum over the block, returned to every thread.
__device__ inline long long block_sum(long long v, long long *s_w)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    v = wave_sum(v);
    __syncthreads();
    if (lane == 0) s_w[wave] = v;
    __syncthreads();
    long long r = 0;
#pragma unroll
    for (int w = 0; w < SCAN_THREADS / 64; ++w) r += s_w[w];
    return r;
}

// This thread's part of the sum over max(len, 0) of lengths [0, n), n a multiple of 4
// and a few thousand; threads [0, THREADS) of the block.  Up to U 16-byte loads a
// thread in flight: with four single ones 7800 lengths were eight trips in a row
// (26 tables x 300 samples 37.9 -> 33.5 us per forward).
constexpr int SUM_LOADS = 6;
template <int THREADS, int U = SUM_LOADS>
__device__ inline long long part_of_sum(const int32_t *__restrict__ len, int n)
{
    typedef int i32x4 __attribute__((ext_vector_type(4)));
    const bool wide = (reinterpret_cast<uintptr_t>(len) & 15) == 0;
    long long sum = 0;
    for (int k0 = 4 * (int)threadIdx.x; k0 < n; k0 += 4 * THREADS * U) {
        i32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t *p = len + min(k0 + u * 4 * THREADS, n - 4);
            if (wide)
                v[u] = *reinterpret_cast<const i32x4 *>(p);
            else
                v[u] = i32x4{p[0], p[1], p[2], p[3]};
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) sum += k0 + u * 4 * THREADS < n && v[u][e] > 0 ? v[u][e] : 0;
    }
    return sum;
}

// Dense part of the Predict-FC input rows of a concatenation model, narrowed, and the zero
// padding behind each row.  Dealt to waves in units of DENSE_ACCESSES wave-wide accesses, an access 64 columns of a
// row or, of a part of half the columns and fewer, of several rows.  By rows alone a wave walked all columns of
// its own: us per forward by rows / in units, 26 tables, 2560 features x 300 samples 41.1 / 14.3, x 4096 90.1 / 42.3, 1000 x
// 1000 31.1 / 16.5; 4 tables, 7 x 30 000 55.9 / 32.2; 64 features as long as before.
constexpr int DENSE_ACCESSES = 4;
struct DenseUnits {
    int log_cols, log_pad;  // lanes to a row of the part and of its padding
    int groups;             // of 64 columns
    int copies, all;        // units that copy; with those that pad
};
__host__ __device__ inline int lanes_log(int columns) { return columns <= 1 ? 0 : columns > 32 ? 6 : 32 - __builtin_clz(columns - 1); }
__host__ __device__ inline DenseUnits dense_units(int rows, int columns, int pad)
{
    const auto row_groups = [rows](int log) { return (int)((rows + (256u >> log) - 1) >> (8 - log)); };
    DenseUnits d;
    d.log_cols = lanes_log(columns);
    d.log_pad = lanes_log(pad);
    d.groups = (columns + 63) / 64;
    d.copies = row_groups(d.log_cols) * d.groups;
    d.all = d.copies + (pad > 0 ? row_groups(d.log_pad) : 0);
    return d;
}

// Block `b` of `nb` blocks of THREADS threads.
template <int THREADS>
__device__ inline void concat_dense_block(const ConcatDense &job, int b, int nb)
{
    static_assert(DENSE_ACCESSES == 4, "rows of a unit");
    constexpr int WAVES = THREADS / 64, U = DENSE_ACCESSES;
    __bf16 *z = static_cast<__bf16 *>(job.z_bf16);
    const int lane = threadIdx.x & 63, pad = job.ldz - job.width;
    const unsigned B = job.B;
    const DenseUnits d = dense_units(job.B, job.w0, pad);
    for (int i = b * WAVES + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); i < d.all; i += nb * WAVES) {
        const bool copy = i < d.copies;
        const int log = copy ? d.log_cols : d.log_pad;
        const int group = !copy ? i - d.copies : d.groups == 1 ? i : i / d.groups;
        const int col = (lane & ((1 << log) - 1)) + (copy ? (i - group * d.groups) * 64 : 0);
        const unsigned r0 = ((unsigned)group << (8 - log)) + (lane >> log), step = 64u >> log;
        if (copy) {
            float v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = job.x0[(long long)min(r0 + u * step, B - 1) * job.ldx0 + min(col, job.w0 - 1)];
            // All of them in flight: else a load moves into the branch around its store, behind the stores before it.
            asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));
            if (col < job.w0)
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (r0 + u * step < B) z[(long long)(r0 + u * step) * job.ldz + col] = (__bf16)v[u];
        } else if (col < pad) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (r0 + u * step < B) z[(long long)(r0 + u * step) * job.ldz + job.width + col] = (__bf16)0.0f;
        }
    }
}

// Blocks of `waves` waves for it, so that a wave has `units` of them at most.
inline int concat_dense_blocks(const ConcatDense &job, int waves, int units)
{
    if (!job.x0) return 0;
    const int of_block = waves * units;
    return (dense_units(job.B, job.w0, job.ldz - job.width).all + of_block - 1) / of_block;
}
// In a launch of many small blocks: two a wave, up to 256 blocks.
inline int concat_dense_blocks(const ConcatDense &job, int waves) { return std::min(concat_dense_blocks(job, waves, 2), 256); }

// How the blocks of a scan that is one launch learn what lies before their tile:
// each publishes the sum of its own (value * 2 + 1, so that the word says by itself
// that it is there), except the last, whose sum nobody reads, and adds up those of
// earlier tiles.  A word only ever goes from zero to its value within the launch;
// the launch behind it on the stream clears it.  So there is no order between
// accesses to different words to keep, and nothing that a call leaves behind
// outlives its own pooling launch, whatever else ran beside it.
// A block waits for words of blocks with smaller numbers only, which never wait
// for it; past `polls` polls it adds up the lengths of that tile itself.
struct TileLink {
    unsigned long long *words = nullptr;  // one per tile, zero before the launch
    int tiles = 0, polls = 0;
};

__device__ inline long long linked_sum(const TileLink &l, int tile, const int32_t *__restrict__ len)
{
    long long sum = 0;
    for (int j = threadIdx.x; j < tile; j += SCAN_THREADS) {
        unsigned long long w = 0;
        for (int p = 0; p < l.polls && !(w & 1); ++p)
            w = __hip_atomic_load(l.words + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (w & 1) {
            sum += (long long)(w >> 1);
        } else {  // tiles before `tile` are full
            for (int k = 0; k < SCAN_TILE; ++k) sum += max(len[(long long)j * SCAN_TILE + k], 0);
        }
    }
    return sum;
}

// As part_of_sum(), over up to 2048 lengths a thread, n a multiple of 4 or zero: loads past n read zeros (a buffer's range
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

// Offsets of a block's bags, a thread for each of the first `bags`, into s_off[0 ... bags], by all threads of the
// block.  own: the thread's length, not negative; before: its part of the sum of all earlier lengths.  Returned
// where the thread's bag ends.  s_w, s_scan: a word per wave each.
template <int THREADS>
__device__ inline long long block_offsets(long long own, long long before, long long nnz, int bags, long long *s_w, long long *s_scan,
                                          int *s_off)
{
    constexpr int WAVES = THREADS / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    long long incl = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const long long up = __shfl_up(incl, o, 64);
        if (lane >= o) incl += up;
    }
    if (lane == 63) s_scan[wave] = incl;
    before = wave_sum(before);
    if (lane == 0) s_w[wave] = before;
    __syncthreads();
    long long run = incl;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) run += s_w[w];
    for (int w = 0; w < wave; ++w) run += s_scan[w];
    if (tid < bags) {
        s_off[tid] = (int)min(run - own, nnz);
        if (tid == bags - 1) s_off[bags] = (int)min(run, nnz);
    }
    return run;
}

// Offsets of bags [first, first + bags) into s_off[0 ... bags] and `offsets`, and the checks of
// their lengths, by all threads of a block, which add up all earlier lengths: `first` a multiple
// of 4 and at most 2048 a thread, a thread for each bag.  U: loads of a thread in flight where the
// earlier lengths are many.
template <int THREADS, int U>
__device__ inline void offsets_of_block(const int32_t *__restrict__ len, int n, long long nnz, int first, int bags,
                                        int32_t *__restrict__ offsets, ErrRecord *err, long long *s_w, long long *s_scan,
                                        int *s_off)
{
    const int tid = threadIdx.x, k = first + tid;
    int own = tid < bags && k < n ? len[k] : 0;
    if (own < 0) {  // counts as 0
        atomicMin(&err->first_bad_len, (unsigned long long)k);
        atomicOr(&err->flags, ERR_NEG_LENGTH);
        own = 0;
    }
    const long long before = U == 8 || first <= 4 * 8 * THREADS ? part_of_long_sum<THREADS, 8>(len, first) : part_of_long_sum<THREADS, U>(len, first);
    const long long run = block_offsets<THREADS>(own, before, nnz, bags, s_w, s_scan, s_off);
    if (tid < bags && k < n) {
        offsets[k] = (int)min(run - own, nnz);
        if (k == n - 1) {
            offsets[n] = (int)min(run, nnz);
            if (run != nnz) atomicOr(&err->flags, ERR_TOTAL_MISMATCH);
        }
    }
    __syncthreads();
}

// LDS of a scan block.
struct ScanShared {
    // One extra word per 32 keeps the 8-per-thread strided reads off one bank.
    int tile[SCAN_TILE + SCAN_TILE / 32];
    long long w[SCAN_THREADS / 64], wave_excl[SCAN_THREADS / 64];
};

// Offsets of tile `tile`; the threads with threadIdx.x < SCAN_THREADS call it,
// all of them.  The sum of earlier tiles comes by `link`, or (no words: a few
// tiles) from their lengths.  LEAN: in few registers, about 0.2 us longer where nothing else lasts as long (one
// sample of 8 tables 11.1 -> 11.3 us per forward).
template <bool LEAN = false>
__device__ inline void scan_offsets_tile(const int32_t *__restrict__ len, int n, long long nnz, const TileLink &link,
                                         int32_t *__restrict__ offsets, ErrRecord *err, int tile, ScanShared &sh)
{
    int *s_tile = sh.tile;
    long long *s_w = sh.w, *s_wave_excl = sh.wave_excl;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const long long base = (long long)tile * SCAN_TILE;

    // Coalesced load of this tile; negative lengths count as 0.
    long long own = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        const int p = i * SCAN_THREADS + tid;
        const long long k = base + p;
        int v = 0;
        if (k < n) v = len[k];
        if (v < 0) {
            atomicMin(&err->first_bad_len, (unsigned long long)k);
            atomicOr(&err->flags, ERR_NEG_LENGTH);
        }
        v = max(v, 0);
        s_tile[p + (p >> 5)] = v;
        own += v;
    }
    long long before = 0;
    if (link.words) {
        own = block_sum(own, s_w);
        if (tid == 0 && tile + 1 < link.tiles)
            __hip_atomic_store(link.words + tile, (unsigned long long)own * 2 + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        before = linked_sum(link, tile, len);
    } else {
        before = part_of_sum<SCAN_THREADS>(len, (int)base);
    }
    before = block_sum(before, s_w);
    __syncthreads();

    // Each thread owns SCAN_ITEMS consecutive entries.
    int mine[SCAN_ITEMS];
    long long tsum = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        const int p = tid * SCAN_ITEMS + i;
        mine[i] = s_tile[p + (p >> 5)];
        tsum += mine[i];
    }
    // Inclusive scan of the thread sums inside the wave, then across waves.
    long long incl = tsum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const long long up = __shfl_up(incl, o, 64);
        if (lane >= o) incl += up;
    }
    if (lane == 63) s_w[wave] = incl;
    __syncthreads();
    if (tid == 0) {
        long long run = 0;
#pragma unroll
        for (int w = 0; w < SCAN_THREADS / 64; ++w) {
            s_wave_excl[w] = run;
            run += s_w[w];
        }
    }
    __syncthreads();
    long long run = before + s_wave_excl[wave] + (incl - tsum);
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        const int p = tid * SCAN_ITEMS + i;
        // Clamping to nnz keeps every bag inside the ids the caller passed.
        s_tile[p + (p >> 5)] = (int)(run < nnz ? run : nnz);
        run += mine[i];
    }
    // `run` of the thread owning the last valid entry is the grand total.
    const long long last = (long long)n - 1 - base;
    if (last >= 0 && last < SCAN_TILE && tid == (int)(last / SCAN_ITEMS)) {
        long long total = before + s_wave_excl[wave] + (incl - tsum);
        for (int i = 0; i <= (int)(last % SCAN_ITEMS); ++i) total += mine[i];
        offsets[n] = (int)(total < nnz ? total : nnz);
        if (total != nnz) atomicOr(&err->flags, ERR_TOTAL_MISMATCH);
    }
    __syncthreads();
    int at = tid;
    if (LEAN) asm volatile("" : "+v"(at));  // else the addresses of the first loop are kept in registers until here
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        const int p = i * SCAN_THREADS + at;
        const long long k = base + p;
        if (k < n) offsets[k] = s_tile[p + (p >> 5)];
    }
}

}  // namespace scan
}  // namespace rec
#endif
