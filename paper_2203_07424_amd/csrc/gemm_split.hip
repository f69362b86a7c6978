// S2 / S4: one fully connected layer, or the last hidden one with the one-output
// layer behind it, where a launch is short: the k of a block tile are dealt to the
// block's waves, and no wave waits for another before the sums are put together.
//
//   C[m][n] = act( sum_k A[m][k] * W[n][k] + bias[n] )
//
// What bounds it: at up to a few hundred samples the trip to memory (weights that
// other launches have pushed out of the L2s) and the launch itself; the kernels
// that bring operands through LDS a k-tile at a time for the whole block
// (csrc/gemm.hip) pay two barriers and most of a trip to L2 per 64 k.  Here wave w takes
// the units of 64 k w, w + WK, ...: weights straight into operand registers from the
// fragment order of csrc/mlp_chain.hip, contiguous KiBs; activation rows as whole 128-byte
// lines into a corner of LDS that only this wave uses (read as fragments from memory
// each lane of a load would touch another line).  The partial tiles are added up through LDS
// in the order of the waves, once.  us per launch, k-tile by k-tile / here:
// 16 samples, 1728 -> 1024 four towers 12.2 / 4.4; 300 samples 17.3 / 12.6, 1024 -> 512 8.5 / 6.6,
// 512 -> 256 -> 1 10.5 / 6.2; 256 samples, 884 -> 512 8.5 / 3.5, 512 -> 128 -> 1 6.0 / 4.2;
// one sample of 2560 fp32 -> 1024 16.8 / 4.6.
//
// More waves or more units in flight a wave change nothing or lose: two or more blocks
// on a compute unit cover one another's trips.
#include "rec_internal.h"

namespace rec {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int UNIT = 64;         // k a wave takes at a time
constexpr int SP_LD = UNIT + 8;  // row pitch of staged activations (elements): conflict-free 16-byte reads

// Input rows: bf16; fp32 in aligned vectors of four; fp32 otherwise.
enum { IN_BF16 = 0, IN_F32 = 1, IN_F32_ANY = 2 };

// What the stacks of a launch have of their own.
struct SplitStack {
    const void *W;  // fragment order
    const float *bias, *dot_w, *dot_bias;
};
// Of the arguments the leading scalars, up to 14 words, are in registers when a wave
// starts; the rest is a trip to cold memory that loads need not wait for.
struct SplitGroups {
    SplitStack s[MAX_GROUPS];
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

template <int TM, int TN, int WN, int WK>
constexpr size_t split_lds_bytes()
{
    constexpr size_t stage = (size_t)WN * WK * TM * 16 * SP_LD * 2, sums = (size_t)WN * WK * TM * TN * 1024;
    return stage > sums ? stage : sums;
}

// 16 TM rows x 16 TN WN columns a block; WN waves side by side, WK deep.  OUT is a
// CHAIN_OUT_* value; CHAIN_OUT_DOT needs all columns of the layer in the block.
template <int TM, int TN, int WN, int WK, int IN, int OUT>
__global__ __launch_bounds__(64 * WN * WK, TM * TN >= 16 || (IN != IN_BF16 && TM * TN >= 8) ? 2 : 4) void fc_split_kernel(
    const void *__restrict__ A0, const void *__restrict__ W0, int lda, int M, int K, int Kpad, int grid_m, int grid_n,
    int m_fast, int per_xcd, int n_groups, int relu, long long a_stride, void *__restrict__ C0, int ldc,
    long long c_stride, float *__restrict__ dot_out, int dot_ld, const SplitGroups groups)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int THREADS = 64 * WN * WK, BM = 16 * TM, BN = 16 * TN * WN;
    constexpr int QUADS = WN * TM * TN * 64;  // groups of four sums of the block tile, as the lanes of a wave hold them
    constexpr int MINE = (QUADS + THREADS - 1) / THREADS;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % WN, wk = wave / WN;
    // Blocks are dealt to the 8 XCDs round-robin: XCD x takes the x-th eighth of the
    // tile list, rows or columns fastest, whichever operand is then read by few L2s.
    const int per_group = grid_m * grid_n;
    int v = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    const int g = v / per_group;
    if (g >= n_groups) return;  // the grid is 8 per_xcd blocks
    v -= g * per_group;
    const int bm = m_fast ? v % grid_m : v / grid_n, bn = m_fast ? v / grid_m : v - bm * grid_n;
    const int m0 = bm * BM, n0 = bn * BN;
    constexpr int ELT = IN == IN_BF16 ? 2 : 4;
    typedef RowUnit<TM, IN> Rows;
    const char *A = static_cast<const char *>(A0) + ((long long)g * a_stride + (long long)m0 * lda) * ELT;
    unsigned row[Rows::LOADS];
#pragma unroll
    for (int i = 0; i < Rows::LOADS; ++i)  // rows past M are computed and dropped
        row[i] = (unsigned)min(lane / Rows::LANES + i * (64 / Rows::LANES), M - 1 - m0) * (unsigned)lda * ELT;
    // Fragment (nc, ks) of 32 columns x 16 k is the KiB at (nc * Kpad / 16 + ks) * 1024:
    // 16 bytes for the lower 8 k of each column, then for the upper 8.
    const char *W = static_cast<const char *>(g == 0 ? W0 : groups.s[g].W);
    unsigned wofs[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        const int c16 = (n0 >> 4) + wn * TN + t;
        wofs[t] = (unsigned)(c16 >> 1) * (unsigned)(Kpad / 16) * 1024u + (lane >> 5) * 1024u + (lane >> 4 & 1) * 512u +
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
    for (int u = wk; u < Kpad / UNIT; u += WK) {
        Rows a;
        a.fetch(A, row, u, K);
        u32x4 w[TN][2];
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int s = 0; s < 2; ++s)
                w[t][s] = *reinterpret_cast<const u32x4 *>(W + (wofs[t] + (unsigned)u * 4096u + s * 2048u));
        __builtin_amdgcn_sched_barrier(0);  // all of the unit's loads in flight together
        a.stash(own, u, K);
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
    f32x4 *sums = reinterpret_cast<f32x4 *>(smem);  // [WK][QUADS]
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
        for (int t = 0; t < TN; ++t) sums[wk * QUADS + ((wn * TM + j) * TN + t) * 64 + lane] = acc[j][t];
    __syncthreads();
    float part[MINE];
#pragma unroll
    for (int j = 0; j < MINE; ++j) {
        const int i = tid + j * THREADS;
        if (i >= QUADS) break;
        f32x4 x = sums[i];
#pragma unroll
        for (int k = 1; k < WK; ++k) x += sums[k * QUADS + i];
        const int m = m0 + i / 64 / TN % TM * 16 + (lane & 15), n = quad_n(i);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            x[e] += bv[j][e];
            x[e] = relu && x[e] < 0.0f ? 0.0f : x[e];
        }
        if (OUT == CHAIN_OUT_DOT) {
            part[j] = x[0] * dw[j][0] + x[1] * dw[j][1] + x[2] * dw[j][2] + x[3] * dw[j][3];
        } else if (m < M) {
            const long long at = (long long)m * ldc + (long long)g * c_stride + n;
            if (OUT == CHAIN_OUT_F32) {
                *reinterpret_cast<f32x4 *>(static_cast<float *>(C0) + at) = x;
            } else {
                bf16x4 h;
#pragma unroll
                for (int e = 0; e < 4; ++e) h[e] = (__bf16)x[e];
                *reinterpret_cast<bf16x4 *>(static_cast<__bf16 *>(C0) + at) = h;
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
        if (tid < BM && m0 + tid < M) {
            float x = 0.0f;
#pragma unroll
            for (int t = 0; t < WN * TN; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    x += parts[((t / TN * TM + tid / 16) * TN + t % TN) * 64 + q * 16 + tid % 16];
            dot_out[(long long)(m0 + tid) * dot_ld + g] = x + groups.s[g].dot_bias[0];
        }
    }
}

template <int TM, int TN, int WN, int WK, int IN, int OUT>
hipError_t launch_as(const FcProblem &a, hipStream_t s)
{
    const int grid_m = (a.M + 16 * TM - 1) / (16 * TM), grid_n = a.Npad / (16 * TN * WN);
    SplitGroups g{};
    for (int i = 0; i < a.groups; ++i) g.s[i] = SplitStack{a.frag[i], a.g.bias[i], a.g.dot_w[i], a.g.dot_bias[i]};
    const int m_fast = (long long)a.M * (IN == IN_BF16 ? 1 : 2) < a.Npad;
    const int per_xcd = (grid_m * grid_n * a.groups + 7) / 8;
    hipLaunchKernelGGL((fc_split_kernel<TM, TN, WN, WK, IN, OUT>), dim3(8 * per_xcd), dim3(64 * WN * WK),
                       (split_lds_bytes<TM, TN, WN, WK>()), s, a.A, a.frag[0], a.lda, a.M, a.K, a.Kpad, grid_m, grid_n,
                       m_fast, per_xcd, a.groups, a.relu ? 1 : 0, a.a_stride, a.C, a.ldc, a.c_stride, a.dot_out,
                       a.dot_ld, g);
    return hipGetLastError();
}

// The tile whose blocks bring the least through the busiest compute unit's L1: rounds
// of blocks times bytes of both operands per k.  Tiles of 64 x 64 count a fifth more
// (300 samples, four towers of 1728 -> 1024: 12.5 in 32 x 64, 13.6 in 64 x 64).
struct Tile {
    int tm, tn;
};
Tile pick_tile(const FcProblem &a, int cus)
{
    static const Tile tiles[] = {{1, 1}, {1, 2}, {2, 2}, {2, 4}, {4, 4}};
    Tile best{0, 0};
    long long least = 0;
    for (const Tile &t : tiles) {
        const long long blocks = (long long)((a.M + 16 * t.tm - 1) / (16 * t.tm)) * (a.Npad / (16 * t.tn)) * a.groups;
        long long cost = (blocks + cus - 1) / cus * (t.tm * (a.a_f32 ? 2 : 1) + t.tn) * 5;
        if (t.tm == 4) cost = cost * 6 / 5;
        if (best.tm == 0 || cost < least) {
            best = t;
            least = cost;
        }
    }
    return best;
}

template <int IN, int OUT>
hipError_t launch_tiles(const FcProblem &a, hipStream_t s)
{
    const Tile t = pick_tile(a, a.num_cus > 0 ? a.num_cus : 256);
    if (t.tm == 1) return t.tn == 1 ? launch_as<1, 1, 1, 8, IN, OUT>(a, s) : launch_as<1, 2, 1, 8, IN, OUT>(a, s);
    if (t.tm == 2) return t.tn == 2 ? launch_as<2, 2, 1, 4, IN, OUT>(a, s) : launch_as<2, 4, 1, 4, IN, OUT>(a, s);
    return launch_as<4, 4, 1, 4, IN, OUT>(a, s);
}

// With the one-output layer: a block has all columns, and as many rows as still give
// every compute unit a block.
template <int IN>
hipError_t launch_dot(const FcProblem &a, hipStream_t s)
{
    const long long cus = a.num_cus > 0 ? a.num_cus : 256, blocks16 = (a.M + 15) / 16 * (long long)a.groups;
    if (a.Npad == 64) return launch_as<1, 4, 1, 8, IN, CHAIN_OUT_DOT>(a, s);
    if (a.Npad == 128)
        return blocks16 < 3 * cus ? launch_as<1, 4, 2, 4, IN, CHAIN_OUT_DOT>(a, s) : launch_as<2, 4, 2, 4, IN, CHAIN_OUT_DOT>(a, s);
    if (blocks16 <= cus) return launch_as<1, 4, 4, 2, IN, CHAIN_OUT_DOT>(a, s);
    return blocks16 <= 2 * cus ? launch_as<2, 4, 4, 2, IN, CHAIN_OUT_DOT>(a, s) : launch_as<4, 4, 4, 2, IN, CHAIN_OUT_DOT>(a, s);
}

template <int IN>
hipError_t launch_in(const FcProblem &a, hipStream_t s)
{
    if (a.dot_out) return launch_dot<IN>(a, s);
    return a.out_f32 ? launch_tiles<IN, CHAIN_OUT_F32>(a, s) : launch_tiles<IN, CHAIN_OUT_BF16>(a, s);
}

template <int TM>
hipError_t prepare_dot()
{
    constexpr size_t lds = split_lds_bytes<TM, 4, 4, 2>();
    const void *kernels[] = {reinterpret_cast<const void *>(fc_split_kernel<TM, 4, 4, 2, IN_BF16, CHAIN_OUT_DOT>),
                             reinterpret_cast<const void *>(fc_split_kernel<TM, 4, 4, 2, IN_F32, CHAIN_OUT_DOT>),
                             reinterpret_cast<const void *>(fc_split_kernel<TM, 4, 4, 2, IN_F32_ANY, CHAIN_OUT_DOT>)};
    for (const void *k : kernels) {
        const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

hipError_t fc_split_prepare() { return prepare_dot<4>(); }

bool fc_split_applies(const FcProblem &a)
{
    for (int g = 0; g < a.groups; ++g)
        if (!a.frag[g]) return false;
    // 32-bit byte offsets inside a block's rows and a stack's weights
    return a.lda <= 1 << 22 && (long long)a.Npad * a.Kpad <= 1ll << 30;
}

hipError_t launch_fc_split(const FcProblem &a, hipStream_t s)
{
    if (!a.a_f32) return launch_in<IN_BF16>(a, s);
    const bool vec = a.K % 4 == 0 && a.lda % 4 == 0 && a.a_stride % 4 == 0 && reinterpret_cast<uintptr_t>(a.A) % 16 == 0;
    return vec ? launch_in<IN_F32>(a, s) : launch_in<IN_F32_ANY>(a, s);
}

}  // namespace rec
