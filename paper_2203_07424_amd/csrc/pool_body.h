// Bodies of the pooling kernels (csrc/pool.hip has the description) as device
// functions: the waves that call them belong to those kernels, which read bag
// offsets, or to the launch that computes the offsets too (csrc/front.hip).
#ifndef REC_POOL_BODY_H
#define REC_POOL_BODY_H
#include <hip/hip_fp16.h>

#include <type_traits>

#include "rec_internal.h"

namespace rec {
namespace pool {

// Both were swept on the RMC2-style workload (2..8 loads, 2..8 waves); these are the best.
constexpr int POOL_WAVES = 4;   // bags per block
constexpr int POOL_UNROLL = 4;  // row loads in flight per lane and step

constexpr int SHORT_UNROLL = 4;  // row loads in flight per lane in the short-bag kernel
constexpr int SHORT_BAGS = 2;    // bags a group of lanes works on at a time
constexpr int SHORT_MEAN = 4;    // mean ids per bag up to which bags share a wave

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// bag -> table, bag / B, without a division on the way to a wave's first load (some 30
// dependent instructions, v_rcp_f32 among them; a wave lives for one bag, and 60
// tables x 16384 take about 1 % less per forward without it).  magic = floor((2^32 - 1) / B) is short of 2^32 / B by at most
// 1, so for bag < 2^31 the high product is short by less than 1/2 and its floor by
// at most one.
struct BagTable {
    unsigned B, magic;
    static BagTable of_batch(int batch) { return {(unsigned)batch, 0xFFFFFFFFu / (unsigned)batch}; }
    __device__ inline int of(int bag) const
    {
        const unsigned t = __umulhi((unsigned)bag, magic);
        return (int)((unsigned)bag - t * B >= B ? t + 1 : t);
    }
};

template <bool HALF>
struct Acc {
    static constexpr int N = HALF ? 8 : 4;
    float v[N];
};

// One more row into the sums.  `one` is 1.0f held in a register: the product
// form lets each fp16 element be widened, and added, by a single mixed-precision
// fused multiply-add (bit-identical to widening and adding, the product being exact).
template <bool HALF>
__device__ inline void accumulate(Acc<HALF> &a, const u32x4 raw, float one)
{
    if (HALF) {
        const f16x8 h = __builtin_bit_cast(f16x8, raw);
#pragma unroll
        for (int i = 0; i < 8; ++i) a.v[i] = __builtin_fmaf((float)h[i], one, a.v[i]);
    } else {
        const f32x4 f = __builtin_bit_cast(f32x4, raw);
#pragma unroll
        for (int i = 0; i < 4; ++i) a.v[i] += f[i];
    }
}

// Rows of one table, 16 bytes per lane.  NARROW (table smaller than 4 GiB): a
// buffer descriptor over the table and 32-bit byte offsets; an offset past the
// table reads as zero, which is how ids marked invalid (key 0xFFFFFFFF..) add
// nothing.  Otherwise 64-bit addresses, invalid keys masked by hand.
template <int ROWBYTES, bool NARROW, bool STREAM>
struct RowSource {
    __amdgpu_buffer_rsrc_t rsrc;
    const __attribute__((address_space(1))) char *lane_base;
    unsigned lane_off;

    __device__ inline RowSource(const void *base, long long rows, int chunk)
    {
        lane_off = chunk * 16;
        if (NARROW)
            rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0,
                                                     (int)(unsigned)(rows * ROWBYTES), 0x00020000);
        else
            lane_base = (const __attribute__((address_space(1))) char *)base + chunk * 16;
    }
    // What a lane hands out for id (id < 0: invalid).
    __device__ static inline unsigned key(int id) { return NARROW ? (unsigned)id * ROWBYTES : (unsigned)id; }
    __device__ inline u32x4 fetch(unsigned k) const
    {
        if (NARROW) return __builtin_amdgcn_raw_buffer_load_b128(rsrc, k + lane_off, 0, STREAM ? 2 : 0);
        const bool ok = (int)k >= 0;
        typedef const __attribute__((address_space(1))) u32x4 *row_ptr;
        const row_ptr src = (row_ptr)(lane_base + (unsigned long long)(ok ? k : 0u) * ROWBYTES);
        u32x4 v = STREAM ? __builtin_nontemporal_load(src) : *src;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = ok ? v[i] : 0u;
        return v;
    }
};

// N sums a lane holds (columns col ... of bag (t, b)) to where they belong.
template <int N, bool CONCAT>
__device__ inline void store_sums(const float *v, const PoolOut &out, int vec_ok, int b, int t, int T,
                                  int D, int col)
{
    typedef __bf16 bvec __attribute__((ext_vector_type(N)));
    if (CONCAT) {
        __bf16 *o = static_cast<__bf16 *>(out.z) + (long long)b * out.ldz + out.col0 + t * D + col;
        if (vec_ok) {
            bvec h;
#pragma unroll
            for (int i = 0; i < N; ++i) h[i] = (__bf16)v[i];
            *reinterpret_cast<bvec *>(o) = h;
        } else {
#pragma unroll
            for (int i = 0; i < N; ++i) o[i] = (__bf16)v[i];
        }
    } else {
        constexpr int W = N < 4 ? N : 4;  // at most 16 bytes a store
        typedef float wvec __attribute__((ext_vector_type(W)));
        float *o = out.pooled + ((long long)b * T + t) * D + col;
#pragma unroll
        for (int i = 0; i < N; i += W) {
            wvec w;
#pragma unroll
            for (int k = 0; k < W; ++k) w[k] = v[i + k];
            *reinterpret_cast<wvec *>(o + i) = w;
        }
    }
}

// a <- a + (a of lane ^ M) in lanes that keep a, b + (b of lane ^ M) in the others
// (lanes with bit M set), M = 32 or 16: one register swap and one add.
template <int M>
__device__ inline float fold_pair(float a, float b)
{
    const unsigned ua = __builtin_bit_cast(unsigned, a), ub = __builtin_bit_cast(unsigned, b);
    const auto r = M == 32 ? __builtin_amdgcn_permlane32_swap(ua, ub, false, false)
                           : __builtin_amdgcn_permlane16_swap(ua, ub, false, false);
    return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}

// v + v of the lane R further on in its row of 16 lanes.
template <int R>
__device__ inline float add_ror(float v)
{
    const int x = __builtin_bit_cast(int, v);
    return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(x, x, 0x120 + R, 0xf, 0xf, false));
}

// Columns a lane ends up with when the partial sums of a wave are folded.
template <int LPR, bool HALF>
constexpr int folded_columns()
{
    constexpr int N = HALF ? 8 : 4, N1 = LPR <= 32 ? N / 2 : N;
    return LPR <= 16 ? N1 / 2 : N1;
}

// Folds the RPW partial sums, lanes l and l ^ m holding the same columns; the lane's columns
// are then acc.v[0 ...] from the one returned on.  While
// m is 32 or 16 a lane passes half of its columns to l ^ m and keeps the sum of
// the other half; within a row of 16 lanes the rest are rotate-and-add.  None of
// it goes through the LDS: folding with __shfl_xor, 24 of the 34 permutes a
// bag of 80 fp16 rows of 64 needed, queued on it.  In terms of the rows of a
// load the order is r with r ^ 1, then r ^ 2, r ^ 4, ...: fp32 sums depend on it.
template <int LPR, bool HALF>
__device__ inline int fold_sums(Acc<HALF> &acc, int lane, int chunk)
{
    float *v = acc.v;
    int col = chunk * Acc<HALF>::N;
    constexpr int N1 = LPR <= 32 ? Acc<HALF>::N / 2 : Acc<HALF>::N, N2 = folded_columns<LPR, HALF>();
    if constexpr (LPR <= 32) {
#pragma unroll
        for (int i = 0; i < N1; ++i) v[i] = fold_pair<32>(v[i], v[i + N1]);
        col += (lane >> 5) * N1;
    }
    if constexpr (LPR <= 16) {
#pragma unroll
        for (int i = 0; i < N2; ++i) v[i] = fold_pair<16>(v[i], v[i + N2]);
        col += (lane >> 4 & 1) * N2;
    }
#pragma unroll
    for (int i = 0; i < N2; ++i) {
        if (LPR <= 8) v[i] = add_ror<8>(v[i]);
        if (LPR <= 4) v[i] = add_ror<4>(v[i]);
        if (LPR <= 2) v[i] = add_ror<2>(v[i]);
        if (LPR <= 1) v[i] = add_ror<1>(v[i]);
    }
    return col;
}

// Which of the 64 / LPR rows of a wave-wide load a lane fetches a part of: lane / LPR with its
// bits in reverse, so that neighbouring rows sit 32 lanes apart, the next pair 16, and so on.
template <int LPR>
__device__ inline int row_of_lane(int lane)
{
    return (int)(__builtin_bitreverse32((unsigned)lane) >> 26) & (64 / LPR - 1);
}

// The sum of bag (t, b), ids [start, end), by one wave.
template <int LPR, bool HALF, bool CONCAT, bool STREAM, bool NARROW>
__device__ inline void pool_bag(const TableDesc *__restrict__ tables, const int32_t *__restrict__ indices,
                                const PoolOut &out, int vec_ok, int T, int b, int t, int start, int end, float one,
                                ErrRecord *err)
{
    constexpr int RPW = 64 / LPR;
    constexpr int ROWBYTES = LPR * 16;
    constexpr int NACC = HALF ? 8 : 4;
    constexpr int D = ROWBYTES / (HALF ? 2 : 4);
    typedef RowSource<ROWBYTES, NARROW, STREAM> Rows;
    const int lane = threadIdx.x & 63;
    const long long rows = tables[t].rows;

    const int sub = row_of_lane<LPR>(lane);
    const int chunk = lane % LPR;
    const Rows src(tables[t].base, rows, chunk);

    Acc<HALF> acc;
#pragma unroll
    for (int i = 0; i < NACC; ++i) acc.v[i] = 0.0f;

    int ids = -1;
    if (start + lane < end) ids = indices[start + lane];
    for (int k0 = start; k0 < end; k0 += 64) {
        const int n = min(64, end - k0);
        int cur = ids;  // -1 in the lanes past the end of the bag
        // Ids outside the table contribute zero and leave a record.
        if (lane < n && (unsigned long long)(long long)cur >= (unsigned long long)rows) {
            atomicMin(&err->first_bad_idx, (unsigned long long)(k0 + lane));
            atomicOr(&err->flags, ERR_INDEX_RANGE);
            cur = -1;
        }
        const unsigned key = Rows::key(cur);
        // Next 64 ids, requested before the row loads of this step.
        ids = -1;
        if (k0 + 64 + lane < end) ids = indices[k0 + 64 + lane];

        const int steps = (n + RPW - 1) / RPW;  // wave-wide loads this chunk needs
        // slot4: byte address of this lane's slot in the cross-lane permute (the
        // hardware takes it modulo the wave).
        int j = 0;
        for (; j + POOL_UNROLL <= steps; j += POOL_UNROLL) {
            const int slot4 = (j * RPW + sub) * 4;
            u32x4 raw[POOL_UNROLL];
#pragma unroll
            for (int u = 0; u < POOL_UNROLL; ++u)
                raw[u] = src.fetch(__builtin_amdgcn_ds_bpermute(slot4 + u * RPW * 4, key));
#pragma unroll
            for (int u = 0; u < POOL_UNROLL; ++u) accumulate<HALF>(acc, raw[u], one);
        }
        if (j < steps) {  // the last, partial group: loads it does not need are not issued
            const int slot4 = (j * RPW + sub) * 4;
            u32x4 raw[POOL_UNROLL - 1];
#pragma unroll
            for (int u = 0; u < POOL_UNROLL - 1; ++u)
                if (j + u < steps) raw[u] = src.fetch(__builtin_amdgcn_ds_bpermute(slot4 + u * RPW * 4, key));
#pragma unroll
            for (int u = 0; u < POOL_UNROLL - 1; ++u)
                if (j + u < steps) accumulate<HALF>(acc, raw[u], one);
        }
    }

    const int col = fold_sums<LPR, HALF>(acc, lane, chunk);
    constexpr int N = folded_columns<LPR, HALF>();
    if (LPR > 8 || (lane & 15) < LPR) store_sums<N, CONCAT>(acc.v, out, vec_ok, b, t, T, D, col);
}

// Bags [first, first + bags) of the n of a launch by a block of WAVES waves, offsets in s_off[0 ... bags]: four
// neighbouring bags a wave at a time, their rows requested together, and the ids of its next four
// in front of these, all sums stored at the end (behind a store the next rows wait until it has reached memory);
// for waves that have few others on their compute unit.  Sums in pool_bag()'s order.
// keys: QUAD_IDS words a wave; sums: D a bag; next: WAVES and 0.  Waves take fours as they are done with others, and at
// the end (in the loop, their loads cost the others waits) the bags of fours of two tables or of more ids one by one.  With
// every eighth four a wave's own, beside 1536 -> 1024 on 4096 samples of 10 tables, us per forward: all lengths 29 but 2 % of 300
// 80.3 -> 66.6 (72.0 in two launches), geometric of mean 35 75.2 -> 68.0 (70.8); 20 ids beside 2560 -> 1024 59.4 as before.
constexpr int QUAD = 4, QUAD_IDS = 256;

template <int WAVES, int LPR, bool HALF, bool STREAM>
__device__ inline void pool_quads(const TableDesc *__restrict__ tables, const int32_t *__restrict__ indices,
                                  const PoolOut &out, const BagTable &div, int T, int n, int first, int bags, const int *s_off,
                                  unsigned *keys, float *sums, int *next, float one, ErrRecord *err)
{
    typedef RowSource<LPR * 16, true, STREAM> Rows;
    constexpr int RPW = 64 / LPR, CHUNKS = QUAD_IDS / 64, D = LPR * 16 / (HALF ? 2 : 4), U = 3;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int sub = row_of_lane<LPR>(lane);
    const auto read_offsets = [&](int q, int (&offs)[QUAD + 1]) {
        const int v = s_off[q + min(lane, QUAD)];
#pragma unroll
        for (int i = 0; i <= QUAD; ++i) offs[i] = __builtin_amdgcn_readlane(v, i);
    };
    int id[CHUNKS];
    const auto request = [&](int q) {  // the ids of four bags
        int offs[QUAD + 1];
        read_offsets(q, offs);
        const int from = offs[0], count = offs[QUAD] - from;
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
            id[c] = -1;
            if (c * 64 + lane < count) id[c] = indices[from + c * 64 + lane];
        }
    };
    const auto joint = [&](int ids, int bag, int live, int t) { return ids <= QUAD_IDS && bag + live <= (t + 1) * (int)div.B; };
    keys += wave * QUAD_IDS;
    const int mine = min(bags, n - first);  // n - first > 0
    const auto ticket = [&](int *count) {
        int v = 0;
        if (lane == 0) v = __hip_atomic_fetch_add(count, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        return __builtin_amdgcn_readfirstlane(v);
    };
    unsigned long long own = 0;  // fours whose sums this wave has in LDS
    if (wave * QUAD < mine) request(wave * QUAD);
    for (int q = wave * QUAD, after; q < mine; q = after) {
        after = ticket(next) * QUAD;
        const int live = min(QUAD, mine - q), bag = first + q;
        int offs[QUAD + 1];
        read_offsets(q, offs);
        const int t = div.of(bag), from = offs[0], total = offs[QUAD] - from;
        const bool together = joint(total, bag, live, t);
        const long long rows = tables[t].rows;
        if (together) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int c = 0; c < CHUNKS; ++c) {
                // Ids outside the table contribute zero and leave a record.
                if (c * 64 + lane < total && (unsigned long long)(long long)id[c] >= (unsigned long long)rows) {
                    atomicMin(&err->first_bad_idx, (unsigned long long)(from + c * 64 + lane));
                    atomicOr(&err->flags, ERR_INDEX_RANGE);
                    id[c] = -1;
                }
                keys[c * 64 + lane] = Rows::key(id[c]);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        if (after < mine) request(after);
        if (!together) continue;
        own |= 1ull << q / QUAD;
        const Rows src(tables[t].base, rows, lane % LPR);
        Acc<HALF> acc[QUAD];
        int at0[QUAD], len[QUAD], most = 0;  // of bags past the last one no ids
#pragma unroll
        for (int i = 0; i < QUAD; ++i) {
#pragma unroll
            for (int e = 0; e < Acc<HALF>::N; ++e) acc[i].v[e] = 0.0f;
            at0[i] = offs[i] - from;
            len[i] = offs[i + 1] - offs[i];
            most = max(most, len[i]);
        }
        // Without branches around the loads: with them the compiler waits for the next ids in front of the rows.
        for (int j = 0; j < most; j += U * RPW) {
            unsigned key[QUAD][U];
#pragma unroll
            for (int i = 0; i < QUAD; ++i)
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int k = j + u * RPW + sub;
                    const unsigned v = keys[k < len[i] ? at0[i] + k : 0];
                    key[i][u] = k < len[i] ? v : Rows::key(-1);
                }
            u32x4 raw[QUAD][U];
#pragma unroll
            for (int i = 0; i < QUAD; ++i)
#pragma unroll
                for (int u = 0; u < U; ++u) raw[i][u] = src.fetch(key[i][u]);
#pragma unroll
            for (int i = 0; i < QUAD; ++i)
#pragma unroll
                for (int u = 0; u < U; ++u) accumulate<HALF>(acc[i], raw[i][u], one);
        }
#pragma unroll
        for (int i = 0; i < QUAD; ++i) {
            const int col = fold_sums<LPR, HALF>(acc[i], lane, lane % LPR);
            if (LPR > 8 || (lane & 15) < LPR)
#pragma unroll
                for (int e = 0; e < folded_columns<LPR, HALF>(); ++e) sums[(q + i) * D + col + e] = acc[i].v[e];
        }
    }
    // The bags of all other fours of the block, dealt to its waves: a lane looks at a four (their number fits a wave).
    const int at = min(lane * QUAD, mine - 1) / QUAD * QUAD;
    unsigned long long left = __builtin_amdgcn_ballot_w64(
        lane * QUAD < mine && !joint(s_off[at + QUAD] - s_off[at], first + at, min(QUAD, mine - at), div.of(first + at)));
    for (int turn = 0, my = left != 0 ? ticket(next + 1) : 0; left != 0; left &= left - 1) {
        const int q = __builtin_ctzll(left) * QUAD;
        for (int i = 0; i < min(QUAD, mine - q); ++i, ++turn) {
            if (turn != my) continue;
            const int bag = first + q + i, t = div.of(bag);
            pool_bag<LPR, HALF, false, STREAM, true>(tables, indices, out, 0, T, bag - t * (int)div.B, t,
                                                     __builtin_amdgcn_readfirstlane(s_off[q + i]),
                                                     __builtin_amdgcn_readfirstlane(s_off[q + i + 1]), one, err);
            my = ticket(next + 1);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    for (; own != 0; own &= own - 1) {
        const int q = __builtin_ctzll(own) * QUAD, live = min(QUAD, mine - q), t = div.of(first + q), b = first + q - t * (int)div.B;
        for (int k = lane; k < live * (D / 4); k += 64)
            *reinterpret_cast<f32x4 *>(out.pooled + ((long long)(b + k / (D / 4)) * T + t) * D + k % (D / 4) * 4) =
                *reinterpret_cast<const f32x4 *>(&sums[q * D + k * 4]);
    }
}

// BAGS bags per group of LPR lanes, their load chains (ids -> rows, PER_BAG at a time) running
// side by side.  bag[g] with ids [pos[g], end[g]); groups without a bag work on a
// copy of another (live[g] false) and store nothing.
// MOSTLY_ONE: bags that are longer than most come one after the other, four ids at a time: a trip of all
// bags for the sake of one is mostly vector instructions on nothing.
// A trip has no branch around a load: with branches there, and the faults in front of the rows, each id was waited for by
// itself (16 000 samples of 26 tables, two ids of a bag at a time, 48.9 -> 46.3 us per forward, of 0 to 3 ids 54.8 -> 50.0).
template <int LPR, bool HALF, bool CONCAT, int BAGS = SHORT_BAGS, int PER_BAG = SHORT_UNROLL / SHORT_BAGS, bool MOSTLY_ONE = false>
__device__ inline void pool_short_bags(const TableDesc *__restrict__ tables, const int32_t *__restrict__ indices,
                                       const PoolOut &out, int vec_ok, const BagTable &div, int T, const bool (&live)[BAGS],
                                       const int (&bag)[BAGS], int (&pos)[BAGS],
                                       const int (&end)[BAGS], float one, ErrRecord *err)
{
    typedef const __attribute__((address_space(1))) char *table_ptr;
    typedef const __attribute__((address_space(1))) u32x4 *row_ptr;
    constexpr int ROWBYTES = LPR * 16;
    constexpr int NACC = HALF ? 8 : 4;
    constexpr int D = ROWBYTES / (HALF ? 2 : 4);
    const int chunk = (threadIdx.x & 63) % LPR;
    int t[BAGS], b[BAGS];
    table_ptr lane_base[BAGS];
    long long rows[BAGS];
    Acc<HALF> acc[BAGS];
#pragma unroll
    for (int g = 0; g < BAGS; ++g) {
        t[g] = div.of(bag[g]);
        b[g] = bag[g] - t[g] * (int)div.B;
        lane_base[g] = (table_ptr)tables[t[g]].base + chunk * 16;
        rows[g] = tables[t[g]].rows;
#pragma unroll
        for (int i = 0; i < NACC; ++i) acc[g].v[i] = 0.0f;
    }

    bool more = false;
#pragma unroll
    for (int g = 0; g < BAGS; ++g) more |= pos[g] < end[g];
    // `ids` ids of each of bags [from, from + n).  A lane in a trip has a bag with ids left, so there are ids to read.
    const auto trip = [&](auto from, auto n, auto ids) {
        constexpr int G = from, N = n, IDS = ids;
        int id[N][IDS];
        bool ok[N][IDS], bad = false;
        u32x4 raw[N][IDS];
#pragma unroll
        for (int g = 0; g < N; ++g)
#pragma unroll
            for (int u = 0; u < IDS; ++u)  // positions past the bag re-read its last id (of an empty bag, some id)
                id[g][u] = indices[max(min(pos[G + g] + u, end[G + g] - 1), 0)];
#pragma unroll
        for (int g = 0; g < N; ++g)
#pragma unroll
            for (int u = 0; u < IDS; ++u) {
                const bool in = pos[G + g] + u < end[G + g];
                ok[g][u] = in && (unsigned long long)(long long)id[g][u] < (unsigned long long)rows[G + g];
                bad |= in && !ok[g][u];
                const long long row = ok[g][u] ? id[g][u] : 0;
                raw[g][u] = *(row_ptr)(lane_base[G + g] + row * ROWBYTES);
            }
        if (bad && chunk == 0) {
#pragma unroll
            for (int g = 0; g < N; ++g)
#pragma unroll
                for (int u = 0; u < IDS; ++u)
                    if (pos[G + g] + u < end[G + g] && !ok[g][u]) {
                        atomicMin(&err->first_bad_idx, (unsigned long long)(pos[G + g] + u));
                        atomicOr(&err->flags, ERR_INDEX_RANGE);
                    }
        }
        more = false;
#pragma unroll
        for (int g = 0; g < N; ++g) {
#pragma unroll
            for (int u = 0; u < IDS; ++u) {
#pragma unroll
                for (int i = 0; i < 4; ++i) raw[g][u][i] = ok[g][u] ? raw[g][u][i] : 0u;
                accumulate<HALF>(acc[G + g], raw[g][u], one);
            }
            pos[G + g] = min(pos[G + g] + IDS, end[G + g]);
            more |= pos[G + g] < end[G + g];
        }
    };
    constexpr std::integral_constant<int, 0> from_first{};
    constexpr std::integral_constant<int, BAGS> all{};
    constexpr std::integral_constant<int, PER_BAG> some{};
    if constexpr (MOSTLY_ONE) {
        static_assert(BAGS == 4 && PER_BAG == 1, "bag by bag");
        constexpr std::integral_constant<int, 1> single{};
        constexpr std::integral_constant<int, 4> four{};
        if (more) trip(from_first, all, single);
        if (more) trip(from_first, all, single);
        for (;;) {
            int most = 0;  // ids left of the lane's longest bag
#pragma unroll
            for (int g = 0; g < BAGS; ++g) most = max(most, end[g] - pos[g]);
            if (most == 0 || __builtin_amdgcn_ballot_w64(most > 2) != 0) break;
            trip(from_first, all, single);
        }
        while (pos[0] < end[0]) trip(std::integral_constant<int, 0>{}, single, four);
        while (pos[1] < end[1]) trip(std::integral_constant<int, 1>{}, single, four);
        while (pos[2] < end[2]) trip(std::integral_constant<int, 2>{}, single, four);
        while (pos[3] < end[3]) trip(std::integral_constant<int, 3>{}, single, four);
    } else {
        while (more) trip(from_first, all, some);
    }
#pragma unroll
    for (int g = 0; g < BAGS; ++g)
        if (live[g]) store_sums<NACC, CONCAT>(acc[g].v, out, vec_ok, b[g], t[g], T, D, chunk * NACC);
}

}  // namespace pool
}  // namespace rec
#endif
