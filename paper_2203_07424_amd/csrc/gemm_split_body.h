// Body of the FC kernels that deal the k of a tile to the waves of a block
// (csrc/gemm_split.hip has the description), as a device function: the block that calls
// it is that kernel's own or one beside the sparse side's blocks (csrc/front.hip).
#ifndef REC_GEMM_SPLIT_BODY_H
#define REC_GEMM_SPLIT_BODY_H
#include "rec_internal.h"

namespace rec {
namespace split {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int UNIT = 64;         // k a wave takes at a time
constexpr int SP_LD = UNIT + 8;  // row pitch of staged activations (elements): conflict-free 16-byte reads

// Input rows: bf16; fp32 in aligned vectors of four; fp32 otherwise.
enum { IN_BF16 = 0, IN_F32 = 1, IN_F32_ANY = 2 };
// OUT is a CHAIN_OUT_* value, or this: bf16 or (SplitLayer::out_f32) fp32, and with
// SplitLayer::z bf16 rows there as well.
constexpr int OUT_EITHER = 3;

// What the stacks of a launch have of their own.
struct SplitStack {
    const void *W;  // fragment order
    const float *bias, *dot_w, *dot_bias;
};
template <int G>
struct SplitGroups {
    SplitStack s[G];
};

// A wave's 16 TM rows of one unit on their way from memory to LDS, 16 bytes a lane and load.
template <int TM, int IN>
struct RowUnit {
    static constexpr int LANES = IN == IN_BF16 ? 8 : 16;  // a row's 64 k
    static constexpr int LOADS = TM * 16 * LANES / 64;
    static constexpr int PER = IN == IN_BF16 ? 8 : 4;     // elements of a load
    u32x4 q[LOADS];

    // row: byte offset of each load's row
    __device__ inline void fetch(const char *A, const unsigned (&row)[LOADS], int unit, int K)
    {
        const int k = unit * UNIT + (int)(threadIdx.x % LANES) * PER;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            if (IN == IN_BF16) {
                q[i] = *reinterpret_cast<const u32x4 *>(A + (row[i] + (unsigned)k * 2u));
            } else if (IN == IN_F32) {  // K is a multiple of 4: all four lie below K or none
                q[i] = *reinterpret_cast<const u32x4 *>(A + (row[i] + (unsigned)min(k, K - 4) * 4u));
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    q[i][e] = *reinterpret_cast<const unsigned *>(A + (row[i] + (unsigned)min(k + e, K - 1) * 4u));
            }
        }
    }
    __device__ inline void stash(__bf16 *dst, int unit, int K) const
    {
        const int lane = threadIdx.x & 63, c = lane % LANES, r = lane / LANES;
        const int k = unit * UNIT + c * PER;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            __bf16 *d = dst + (r + i * (64 / LANES)) * SP_LD + c * PER;
            if (IN == IN_BF16) {
                *reinterpret_cast<u32x4 *>(d) = q[i];
            } else {
                const f32x4 f = __builtin_bit_cast(f32x4, q[i]);
                bf16x4 h;
#pragma unroll
                for (int e = 0; e < 4; ++e) h[e] = (__bf16)(k + e < K ? f[e] : 0.0f);
                *reinterpret_cast<bf16x4 *>(d) = h;
            }
        }
    }
};

// Partial tiles that are in LDS at a time: where all of them are more than 64 KB those of the
// upper half of the waves are added to the lower half's first.
template <int TM, int TN, int WN, int WK>
constexpr int partial_tiles() { return WK >= 8 && WN * WK * TM * TN > 64 ? WK / 2 : WK; }

template <int TM, int TN, int WN, int WK>
constexpr size_t split_lds_bytes()
{
    constexpr size_t stage = (size_t)WN * WK * TM * 16 * SP_LD * 2, sums = (size_t)WN * partial_tiles<TM, TN, WN, WK>() * TM * TN * 1024;
    return stage > sums ? stage : sums;
}

// One layer of `n_groups` stacks as the blocks of a launch see it: grid_m x grid_n tiles a
// stack, 8 per_xcd blocks.
struct SplitLayer {
    const void *A, *W0;  // W0: the first stack's weights, fragment order
    int lda, M, K, Kpad, grid_m, grid_n, m_fast, per_xcd, n_groups, relu;
    long long a_stride;
    void *C;
    int ldc;
    long long c_stride;
    float *dot_out;
    int dot_ld;
    int out_f32;  // OUT_EITHER
    void *z;      // OUT_EITHER: columns [0, zcols) of C narrowed to bf16, row stride ldz (a multiple of 4), or null
    int ldz, zcols;
};

// Block `block` of the launch: 16 TM rows x 16 TN WN columns; WN waves side by side, WK
// deep; 64 WN WK threads, split_lds_bytes() of `smem`.  CHAIN_OUT_DOT needs all columns of
// the layer in the block.
template <int TM, int TN, int WN, int WK, int IN, int OUT, class Groups>
__device__ inline void split_block(const SplitLayer &p, const Groups &groups, unsigned char *smem, int block)
{
    constexpr int THREADS = 64 * WN * WK, BM = 16 * TM, BN = 16 * TN * WN;
    constexpr int QUADS = WN * TM * TN * 64;  // groups of four sums of the block tile, as the lanes of a wave hold them
    constexpr int MINE = (QUADS + THREADS - 1) / THREADS;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % WN, wk = wave / WN;
    // Blocks are dealt to the 8 XCDs round-robin: XCD x takes the x-th eighth of the
    // tile list, rows or columns fastest, whichever operand is then read by few L2s.
    const int per_group = p.grid_m * p.grid_n;
    int v = (block & 7) * p.per_xcd + (block >> 3);
    const int g = v / per_group;
    if (g >= p.n_groups) return;  // the launch has 8 per_xcd blocks
    v -= g * per_group;
    const int bm = p.m_fast ? v % p.grid_m : v / p.grid_n, bn = p.m_fast ? v / p.grid_m : v - bm * p.grid_n;
    const int m0 = bm * BM, n0 = bn * BN;
    constexpr int ELT = IN == IN_BF16 ? 2 : 4;
    typedef RowUnit<TM, IN> Rows;
    const char *A = static_cast<const char *>(p.A) + ((long long)g * p.a_stride + (long long)m0 * p.lda) * ELT;
    unsigned row[Rows::LOADS];
#pragma unroll
    for (int i = 0; i < Rows::LOADS; ++i)  // rows past M are computed and dropped
        row[i] = (unsigned)min(lane / Rows::LANES + i * (64 / Rows::LANES), p.M - 1 - m0) * (unsigned)p.lda * ELT;
    // Fragment (nc, ks) of 32 columns x 16 k is the KiB at (nc * Kpad / 16 + ks) * 1024:
    // 16 bytes for the lower 8 k of each column, then for the upper 8.
    const char *W = static_cast<const char *>(g == 0 ? p.W0 : groups.s[g].W);
    unsigned wofs[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        const int c16 = (n0 >> 4) + wn * TN + t;
        wofs[t] = (unsigned)(c16 >> 1) * (unsigned)(p.Kpad / 16) * 1024u + (lane >> 5) * 1024u + (lane >> 4 & 1) * 512u +
                  (c16 & 1) * 256u + (lane & 15) * 16u;
    }
    // Quad i: lane i % 64 of tile (wn, row tile, column tile) = i / 64, the last fastest.
    const auto quad_n = [&](int i) { return n0 + i / (64 * TM * TN) * 16 * TN + i / 64 % TN * 16 + 4 * (lane >> 4); };
    const float *bias = groups.s[g].bias, *dot_w = groups.s[g].dot_w;
    f32x4 bv[MINE], dw[MINE];
#pragma unroll
    for (int j = 0; j < MINE; ++j) {
        const int i = tid + j * THREADS;
        if (i < QUADS) {
            bv[j] = *reinterpret_cast<const f32x4 *>(bias + quad_n(i));
            if (OUT == CHAIN_OUT_DOT) dw[j] = *reinterpret_cast<const f32x4 *>(dot_w + quad_n(i));
        }
    }

    // acc[j][t][r]: row 16 j + lane % 16, column 16 t + 4 (lane / 16) + r of the wave's tile.
    f32x4 acc[TM][TN];
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
        for (int t = 0; t < TN; ++t) acc[j][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    __bf16 *own = reinterpret_cast<__bf16 *>(smem) + wave * (BM * SP_LD);
    for (int u = wk; u < p.Kpad / UNIT; u += WK) {
        Rows a;
        a.fetch(A, row, u, p.K);
        u32x4 w[TN][2];
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int s = 0; s < 2; ++s)
                w[t][s] = *reinterpret_cast<const u32x4 *>(W + (wofs[t] + (unsigned)u * 4096u + s * 2048u));
        __builtin_amdgcn_sched_barrier(0);  // all of the unit's loads in flight together
        a.stash(own, u, p.K);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            bf16x8 f[TM];
#pragma unroll
            for (int j = 0; j < TM; ++j)
                f[j] = *reinterpret_cast<const bf16x8 *>(own + (16 * j + (lane & 15)) * SP_LD + 32 * s + 8 * (lane >> 4));
#pragma unroll
            for (int j = 0; j < TM; ++j)
#pragma unroll
                for (int t = 0; t < TN; ++t)
                    acc[j][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[t][s]), f[j],
                                                                        acc[j][t], 0, 0, 0);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }

    __syncthreads();  // the staged rows are done with
    constexpr int PARTS = partial_tiles<TM, TN, WN, WK>();
    f32x4 *sums = reinterpret_cast<f32x4 *>(smem);  // [PARTS][QUADS]
    f32x4 *mine = sums + (wk % PARTS) * QUADS + wn * TM * TN * 64 + lane;
    if (PARTS < WK) {
        if (wk >= PARTS) {
#pragma unroll
            for (int i = 0; i < TM * TN; ++i) mine[i * 64] = acc[i / TN][i % TN];
        }
        __syncthreads();
        if (wk < PARTS) {
#pragma unroll
            for (int i = 0; i < TM * TN; ++i) acc[i / TN][i % TN] += mine[i * 64];
        }
    }
    if (wk < PARTS) {
#pragma unroll
        for (int i = 0; i < TM * TN; ++i) mine[i * 64] = acc[i / TN][i % TN];
    }
    __syncthreads();
    float part[MINE];
#pragma unroll
    for (int j = 0; j < MINE; ++j) {
        const int i = tid + j * THREADS;
        if (i >= QUADS) break;
        f32x4 x = sums[i];
#pragma unroll
        for (int k = 1; k < PARTS; ++k) x += sums[k * QUADS + i];
        const int m = m0 + i / 64 / TN % TM * 16 + (lane & 15), n = quad_n(i);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            x[e] += bv[j][e];
            x[e] = p.relu && x[e] < 0.0f ? 0.0f : x[e];
        }
        if (OUT == CHAIN_OUT_DOT) {
            part[j] = x[0] * dw[j][0] + x[1] * dw[j][1] + x[2] * dw[j][2] + x[3] * dw[j][3];
        } else if (m < p.M) {
            const long long at = (long long)m * p.ldc + (long long)g * p.c_stride + n;
            bf16x4 h;
#pragma unroll
            for (int e = 0; e < 4; ++e) h[e] = (__bf16)x[e];
            if (OUT == CHAIN_OUT_F32 || (OUT == OUT_EITHER && p.out_f32))
                *reinterpret_cast<f32x4 *>(static_cast<float *>(p.C) + at) = x;
            else
                *reinterpret_cast<bf16x4 *>(static_cast<__bf16 *>(p.C) + at) = h;
            if (OUT == OUT_EITHER && p.z) {
                __bf16 *z = static_cast<__bf16 *>(p.z) + (long long)m * p.ldz + n;
                if (n + 4 <= p.zcols) {
                    *reinterpret_cast<bf16x4 *>(z) = h;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (n + e < p.zcols) z[e] = h[e];
                }
            }
        }
    }
    if (OUT == CHAIN_OUT_DOT) {
        __syncthreads();
        float *parts = reinterpret_cast<float *>(smem);  // [QUADS]
#pragma unroll
        for (int j = 0; j < MINE; ++j)
            if (tid + j * THREADS < QUADS) parts[tid + j * THREADS] = part[j];
        __syncthreads();
        if (tid < BM && m0 + tid < p.M) {
            float x = 0.0f;
#pragma unroll
            for (int t = 0; t < WN * TN; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    x += parts[((t / TN * TM + tid / 16) * TN + t % TN) * 64 + q * 16 + tid % 16];
            p.dot_out[(long long)(m0 + tid) * p.dot_ld + g] = x + groups.s[g].dot_bias[0];
        }
    }
}

// Layer `a` in tiles of 16 tm x 16 tn wn.
inline SplitLayer layer_in_tiles(const FcProblem &a, int tm, int tn, int wn)
{
    SplitLayer p{};
    p.A = a.A; p.W0 = a.frag[0]; p.lda = a.lda; p.M = a.M; p.K = a.K; p.Kpad = a.Kpad;
    p.grid_m = (a.M + 16 * tm - 1) / (16 * tm);
    p.grid_n = a.Npad / (16 * tn * wn);
    p.m_fast = (long long)a.M * (a.a_f32 ? 2 : 1) < a.Npad;
    p.per_xcd = (p.grid_m * p.grid_n * a.groups + 7) / 8;
    p.n_groups = a.groups; p.relu = a.relu ? 1 : 0;
    p.a_stride = a.a_stride; p.C = a.C; p.ldc = a.ldc; p.c_stride = a.c_stride;
    p.dot_out = a.dot_out; p.dot_ld = a.dot_ld; p.out_f32 = a.out_f32 ? 1 : 0;
    return p;
}
// fp32 input rows that can be read in aligned vectors of four.
inline bool rows_in_vectors(const FcProblem &a)
{
    return a.K % 4 == 0 && a.lda % 4 == 0 && a.a_stride % 4 == 0 && reinterpret_cast<uintptr_t>(a.A) % 16 == 0;
}

// What a launch with other work gets of a layer that rides along (OUT_EITHER).
struct Rider {
    SplitLayer p;
    SplitGroups<1> g;
};
inline Rider rider_of(const FcProblem &a, int tm, int tn, void *z, int ldz, int zcols)
{
    Rider r{};
    r.p = layer_in_tiles(a, tm, tn, 1);
    r.p.z = z; r.p.ldz = ldz; r.p.zcols = zcols;
    r.g.s[0] = SplitStack{a.frag[0], a.g.bias[0], nullptr, nullptr};
    return r;
}
}  // namespace split
}  // namespace rec
#endif
