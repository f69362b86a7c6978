// Body of the kernels that run a stack of fully connected layers on chip
// (csrc/mlp_chain.hip has the description), as device functions: the block that
// calls them may be one of that kernel's own, a spare block of the scan that the
// stack rides along with, or a block that has just put the stack's input
// together in LDS itself (csrc/tail.hip).
#ifndef REC_MLP_CHAIN_BODY_H
#define REC_MLP_CHAIN_BODY_H
#include "rec_internal.h"

namespace rec {
namespace chain {

constexpr int CH_WAVES = 8;
constexpr int CH_THREADS = CH_WAVES * 64;
static_assert(CHAIN_MAX_WIDTH <= 4 * 32 * CH_WAVES, "a wave takes at most four chunks of 32 output columns");
static_assert(CHAIN_NARROW_WIDTH <= 32 * CH_WAVES, "and one in the narrow form");
constexpr int CH_LDS_PAD = 8; // elements added to an LDS row: consecutive rows start 4 banks apart

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// Rows of activations a block holds: RT tiles of 32.
template <int RT>
constexpr int rows_of() { return 32 * RT; }

// Eight (bf16) or four (fp32) columns of an input row; zero from column K on.
template <bool A_F32>
struct InVec;
template <>
struct InVec<true> {
    static constexpr int W = 4;
    f32x4 v;
    __device__ inline void load(const float *p, int, int) { v = *reinterpret_cast<const f32x4 *>(p); }
    __device__ inline void zero() { v = f32x4{0.0f, 0.0f, 0.0f, 0.0f}; }
    __device__ inline void store(__bf16 *d) const
    {
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (__bf16)v[e];
        *reinterpret_cast<bf16x4 *>(d) = o;
    }
};
template <>
struct InVec<false> {
    static constexpr int W = 8;
    bf16x8 v;
    __device__ inline void load(const __bf16 *p, int k, int K)
    {
        v = *reinterpret_cast<const bf16x8 *>(p);
        if (k + 8 > K) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (k + e >= K) v[e] = (__bf16)0.0f;
        }
    }
    __device__ inline void zero()
    {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = (__bf16)0.0f;
    }
    __device__ inline void store(__bf16 *d) const { *reinterpret_cast<bf16x8 *>(d) = v; }
};

// Input rows -> LDS as bf16, zero for rows >= M and columns >= K.  Each of the
// `rows` (a power of two) has CH_THREADS / rows threads of its own; up to BATCH
// loads of a thread are in flight.
template <bool A_F32, int BATCH, class Run>
__device__ inline void stage_input(const Run &a, int g, int row0, int rows, __bf16 *dst, int ld)
{
    typedef typename std::conditional<A_F32, float, __bf16>::type elem;
    const int TPR = CH_THREADS / rows;
    const int Kpad = a.Kpad[0];
    const int r = threadIdx.x / TPR, c = threadIdx.x % TPR;
    const bool live = row0 + r < a.M;
    const elem *A = static_cast<const elem *>(a.A) + (long long)g * a.a_stride + (long long)(row0 + r) * a.lda;
    __bf16 *row = dst + r * ld;
    if (a.a_vec) {
        typedef InVec<A_F32> Vec;
        const int STEP = TPR * Vec::W;
        for (int k0 = c * Vec::W; k0 < Kpad; k0 += BATCH * STEP) {
            Vec v[BATCH];
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int k = k0 + u * STEP;
                v[u].zero();
                if (live && k < a.K) v[u].load(A + k, k, a.K);
            }
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int k = k0 + u * STEP;
                if (k < Kpad) v[u].store(row + k);
            }
        }
    } else {
        for (int k0 = c; k0 < Kpad; k0 += BATCH * TPR) {
            float v[BATCH];
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int k = k0 + u * TPR;
                v[u] = live && k < a.K ? (float)A[k] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < BATCH; ++u)
                if (k0 + u * TPR < Kpad) row[k0 + u * TPR] = (__bf16)v[u];
        }
    }
}

// k-steps (of 16) a weight fragment is requested before its use.
template <int CNT>
constexpr int fetch_ahead() { return CNT <= 2 ? 8 : 4; }

// The weights of CNT chunks of 32 output columns on their way to the products:
// fragments straight from global memory (L2) into operand registers, requested
// fetch_ahead() steps before their use in straight-line code (a branch around a
// request makes the compiler wait for all of them).
template <int CNT, int AHEAD = fetch_ahead<CNT>()>
struct WeightStream {
    static constexpr int PF = AHEAD;
    const char *w;   // chunk 0's first fragment (the same in all lanes), chunk c wstep bytes further on
    unsigned wstep, lane16;
    int KS;          // k-steps in all, a multiple of 4
    u32x4 q[PF][CNT];

    __device__ inline u32x4 at(int c, int k) const
    {
        return *reinterpret_cast<const u32x4 *>(w + (c * wstep + (unsigned)k * 1024u) + lane16);
    }
    WeightStream() = default;
    __device__ inline WeightStream(const char *w_, unsigned wstep_, int KS_) : w(w_), wstep(wstep_), KS(KS_)
    {
        lane16 = (threadIdx.x & 63) * 16;
#pragma unroll
        for (int p = 0; p < PF; ++p)
#pragma unroll
            for (int c = 0; c < CNT; ++c) q[p][c] = at(c, min(p, KS - 1));
    }
};

// acc[c][j] += W_c X_j^T over the KS k-steps of RT tiles of 32 samples; x is this
// lane's part of row tile 0.  The activation fragments are read from LDS a group
// of XG steps before their products, so that neither their latency nor the
// weights' is met at a product.
template <int CNT, int RT, int PF, int XG = CNT * RT >= 8 ? 1 : CNT * RT >= 4 ? 2 : 4>
__device__ inline void chunk_product(WeightStream<CNT, PF> &ws, const __bf16 *x, int xstep, int KS,
                                     f32x16 (&acc)[CNT][RT])
{
    const auto rows = [&](bf16x8 (&f)[XG][RT], int k) {
#pragma unroll
        for (int p = 0; p < XG; ++p)
#pragma unroll
            for (int j = 0; j < RT; ++j) f[p][j] = *reinterpret_cast<const bf16x8 *>(x + j * xstep + (k + p) * 16);
    };
    bf16x8 xf[XG][RT];
    rows(xf, 0);

    int ks = 0;
    for (; ks + PF < KS; ks += PF) {
#pragma unroll
        for (int g = 0; g < PF / XG; ++g) {
            bf16x8 xn[XG][RT];
            rows(xn, ks + XG * (g + 1));
#pragma unroll
            for (int p = 0; p < XG; ++p) {
                const int slot = XG * g + p;
#pragma unroll
                for (int c = 0; c < CNT; ++c)
#pragma unroll
                    for (int j = 0; j < RT; ++j)
                        acc[c][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ws.q[slot][c]),
                                                                            xf[p][j], acc[c][j], 0, 0, 0);
                const int k = min(ks + slot + PF, KS - 1);
#pragma unroll
                for (int c = 0; c < CNT; ++c) ws.q[slot][c] = ws.at(c, k);
                __builtin_amdgcn_sched_barrier(0);  // keep each request where it is written
            }
#pragma unroll
            for (int p = 0; p < XG; ++p)
#pragma unroll
                for (int j = 0; j < RT; ++j) xf[p][j] = xn[p][j];
        }
    }
    // The last up to PF steps, a multiple of 4: no weights are requested any more.
#pragma unroll
    for (int g = 0; g < PF / XG; ++g) {
        if (ks + XG * g < KS) {
            if (g > 0) rows(xf, ks + XG * g);
#pragma unroll
            for (int p = 0; p < XG; ++p)
#pragma unroll
                for (int c = 0; c < CNT; ++c)
#pragma unroll
                    for (int j = 0; j < RT; ++j)
                        acc[c][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ws.q[XG * g + p][c]),
                                                                            xf[p][j], acc[c][j], 0, 0, 0);
        }
    }
}

// All blocks walk the weights in the same order at the same time, so a line missing
// in the L2 is missing for every block that wants it, and one compute unit's
// misses in flight are few.  So the blocks that share an L2 each touch a slice of
// the weights up front, one load per 128-byte line, all in flight together.  The
// caller consumes the result (done()) once it has something else to wait for.
constexpr int TOUCH = 4;  // lines a thread touches at most
struct Touched {
    unsigned v[TOUCH];
    __device__ inline void done() const
    {
#pragma unroll
        for (int u = 0; u < TOUCH; ++u) asm volatile("" ::"v"(v[u]));
    }
};
// Slice `mine` of `share` of the run's weights.
template <class Run>
__device__ inline Touched touch_weights(const Run &a, int g, int mine, int share)
{
    int total = 0;
    for (int L = 0; L < a.n_layers; ++L) total += a.Kpad[L] * a.Npad[L] / 64;  // bf16: 64 elements per line
    const int per = (total + share - 1) / share, end = min(total, (mine + 1) * per);
    Touched t;
#pragma unroll
    for (int u = 0; u < TOUCH; ++u) t.v[u] = 0;
    int base = 0;
    for (int L = 0; L < a.n_layers; ++L) {
        const unsigned *w = static_cast<const unsigned *>(a.W[g][L]);
        const int lines = a.Kpad[L] * a.Npad[L] / 64;
#pragma unroll
        for (int u = 0; u < TOUCH; ++u) {
            const int f = mine * per + u * CH_THREADS + (int)threadIdx.x;
            if (f < end && f >= base && f < base + lines) t.v[u] = w[(size_t)(f - base) * 32];
        }
        base += lines;
    }
    return t;
}
// Blocks are dealt to the 8 XCDs round-robin.  Of a launch of n blocks, how many
// share an XCD's touching; beyond 32 a slice is down to a few lines a wave.
__device__ inline int touch_share(int n) { return min(32, max(1, n >> 3)); }

// A launch's arguments are cold memory to every compute unit, and the layers of a run
// read them line by line, each a trip in front of a layer: all lines of the kernel's
// BYTES of arguments at once, first (8 tables x 150 samples, launches of three and two
// layers: 16.0 -> 14.4 us).
template <int BYTES>
__device__ inline void touch_args()
{
    typedef const __attribute__((address_space(4))) unsigned *arg_ptr;
    const arg_ptr args = (arg_ptr)__builtin_amdgcn_kernarg_segment_ptr();
    unsigned v[(BYTES + 63) / 64];
#pragma unroll
    for (int i = 0; i < (BYTES + 63) / 64; ++i) v[i] = args[i * 16];
#pragma unroll
    for (int i = 0; i < (BYTES + 63) / 64; ++i) asm volatile("" ::"s"(v[i]));
}

// What the layers of a run share.
struct RunCtx {
    __bf16 *X;     // activations, bf16 [rows][ld]
    float *x0s;    // fp32 copy of the last activations for the caller (or null), [rows][x0_ld]
    int ld, x0_ld;
    int g, row0;
    int last_row;  // rows - 1: lanes past it work on copies and leave nothing behind
};

__device__ inline bf16x4 narrowed(const f32x4 &v)
{
    bf16x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (__bf16)v[e];
    return o;
}

// Columns n .. n + 3 of the run's last activations of row `row`, to where they go.
template <class Run>
__device__ inline void store_last(const Run &a, const RunCtx &t, int row, int n, const f32x4 &v)
{
    if ((row & 31) > t.last_row) return;
    if (t.x0s && n < t.x0_ld) *reinterpret_cast<f32x4 *>(t.x0s + row * t.x0_ld + n) = v;
    if (t.row0 + row >= a.M) return;
    const long long at = (long long)(t.row0 + row) * a.ldc + (long long)t.g * a.c_stride + n;
    if (a.out_mode == CHAIN_OUT_F32)
        *reinterpret_cast<f32x4 *>(static_cast<float *>(a.C) + at) = v;
    else
        *reinterpret_cast<bf16x4 *>(static_cast<__bf16 *>(a.C) + at) = narrowed(v);
}

// One layer for a wave that has CNT chunks (first, first + 8, ...) of row tiles
// tile .. tile + RT - 1: product, the block's barrier if the output goes back to
// X, epilogue.  Adds the wave's part of the one-output layer behind the run to
// dot_part.
template <int CNT, int RT, class Run>
__device__ inline void layer_pass(const Run &a, const RunCtx &t, int L, int first, int tile, float (&dot_part)[RT])
{
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));  // else every address below is kept in registers across all layers
    const int m = lane & 31, half = lane >> 5;  // sample of this lane in a row tile, and which 8 of a step's 16 k
    const int KS = a.Kpad[L] / 16;
    const bool last = L + 1 == a.n_layers, relu = a.relu[L] != 0;
    // acc[c][j][r] is output column n = 32 (first + 8 c) + 8 (r / 4) + 4 half + r % 4
    // of sample 32 (tile + j) + m.
    f32x16 acc[CNT][RT];
    f32x4 bv[CNT][4];
    const auto load_bias = [&]() {
        const float *bias = a.bias[t.g][L] + first * 32 + 4 * half;
#pragma unroll
        for (int c = 0; c < CNT; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i) bv[c][i] = *reinterpret_cast<const f32x4 *>(bias + c * CH_WAVES * 32 + 8 * i);
    };
    if (CNT <= 2) load_bias();  // early, where there are registers to keep it in
#pragma unroll
    for (int c = 0; c < CNT; ++c)
#pragma unroll
        for (int j = 0; j < RT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[c][j][r] = 0.0f;
    // fragment (nc, ks) is the KiB at W + (nc * KS + ks) * 1024
    WeightStream<CNT> ws(static_cast<const char *>(a.W[t.g][L]) + (size_t)first * KS * 1024,
                         (unsigned)(CH_WAVES * KS * 1024), KS);
    chunk_product<CNT, RT>(ws, t.X + (tile * 32 + (m & t.last_row)) * t.ld + half * 8, 32 * t.ld, KS, acc);
    if (CNT > 2) load_bias();
    __builtin_amdgcn_sched_barrier(0);  // nothing of the epilogue into the product's registers
    if (!last) __syncthreads();  // every wave has read the input: the output may replace it
#pragma unroll
    for (int c = 0; c < CNT; ++c) {
#pragma unroll
        for (int j = 0; j < RT; ++j) {
            const int row = (tile + j) * 32 + m;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int n = (first + c * CH_WAVES) * 32 + 8 * q + 4 * half;
                f32x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float s = acc[c][j][4 * q + e] + bv[c][q][e];
                    v[e] = relu && s < 0.0f ? 0.0f : s;
                }
                if (!last) {
                    if (m <= t.last_row) *reinterpret_cast<bf16x4 *>(t.X + row * t.ld + n) = narrowed(v);
                } else if (a.out_mode == CHAIN_OUT_DOT) {
                    const f32x4 wq = *reinterpret_cast<const f32x4 *>(a.dot_w[t.g] + n);
#pragma unroll
                    for (int e = 0; e < 4; ++e) dot_part[j] += v[e] * wq[e];
                } else {
                    store_last(a, t, row, n, v);
                }
            }
        }
    }
}

// The first weights of a layer, requested before its input is complete.
// Narrow runs only: a wave has one chunk of 32 columns or none.
template <int MAXC>
struct Ahead {
    template <class Run>
    __device__ inline void request(const Run &, int, int) {}
};
template <>
struct Ahead<1> {
    WeightStream<1> ws;
    f32x4 bias[4];
    template <class Run>
    __device__ inline void request(const Run &a, int g, int L)
    {
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), KS = a.Kpad[L] / 16;
        if (wave >= a.Npad[L] / 32) return;
        ws = WeightStream<1>(static_cast<const char *>(a.W[g][L]) + (size_t)wave * KS * 1024, 0, KS);
        const float *b = a.bias[g][L] + wave * 32 + 4 * ((threadIdx.x & 63) >> 5);
#pragma unroll
        for (int i = 0; i < 4; ++i) bias[i] = *reinterpret_cast<const f32x4 *>(b + 8 * i);
    }
};

// The layers of a narrow run.  A layer is a trip to L2 for its weights and little
// else, so the next one's are requested as soon as this one's products have let go of
// the registers, in front of the two barriers and the epilogue.
template <class Run>
__device__ inline void narrow_layers(const Run &a, const RunCtx &t, Ahead<1> &ahead, float &dot_part)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    for (int L = 0; L < a.n_layers; ++L) {
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));  // else every address below is kept in registers across all layers
        const int m = lane & 31, half = lane >> 5;
        const bool last = L + 1 == a.n_layers, has = wave < a.Npad[L] / 32, dot = last && a.out_mode == CHAIN_OUT_DOT;
        const int n0 = wave * 32 + 4 * half;
        f32x16 acc[1][1];
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][0][r] = 0.0f;
        f32x4 bv[4], dw[4];
        if (has) {
            if (dot) {
#pragma unroll
                for (int q = 0; q < 4; ++q) dw[q] = *reinterpret_cast<const f32x4 *>(a.dot_w[t.g] + n0 + 8 * q);
            }
            chunk_product<1, 1>(ahead.ws, t.X + (m & t.last_row) * t.ld + half * 8, 0, a.Kpad[L] / 16, acc);
#pragma unroll
            for (int q = 0; q < 4; ++q) bv[q] = ahead.bias[q];
        }
        __builtin_amdgcn_sched_barrier(0);
        if (!last) {
            ahead.request(a, t.g, L + 1);
            __syncthreads();  // every wave has read the input: the output may replace it
        }
        if (has) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int n = n0 + 8 * q;
                f32x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float s = acc[0][0][4 * q + e] + bv[q][e];
                    v[e] = a.relu[L] != 0 && s < 0.0f ? 0.0f : s;
                }
                if (dot) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) dot_part += v[e] * dw[q][e];
                } else if (last) {
                    store_last(a, t, m, n, v);
                } else if (m <= t.last_row) {
                    *reinterpret_cast<bf16x4 *>(t.X + m * t.ld + n) = narrowed(v);
                }
            }
        }
        if (!last) __syncthreads();
    }
}

// The same within 64 registers, for blocks beside others that want all wave slots of a
// compute unit: weights four steps ahead, nothing requested in front of the barriers.  The
// layers of a block of 256-128-64 take about 1 us longer for it (8 tables of 20 ids x 800 samples, where
// nothing else lasts as long, 12.6 -> 13.4 us per forward).
constexpr int LIGHT_AHEAD = 4, LIGHT_XG = 2, LIGHT_BATCH = 4;
template <class Run>
__device__ inline void light_layers(const Run &a, const RunCtx &t)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    for (int L = 0; L < a.n_layers; ++L) {
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));  // else every address below is kept in registers across all layers
        const int m = lane & 31, half = lane >> 5;
        const bool last = L + 1 == a.n_layers, has = wave < a.Npad[L] / 32;
        const int n0 = wave * 32 + 4 * half, KS = a.Kpad[L] / 16;
        f32x16 acc[1][1];
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][0][r] = 0.0f;
        if (has) {
            WeightStream<1, LIGHT_AHEAD> ws(static_cast<const char *>(a.W[t.g][L]) + (size_t)wave * KS * 1024, 0, KS);
            chunk_product<1, 1, LIGHT_AHEAD, LIGHT_XG>(ws, t.X + m * t.ld + half * 8, 0, KS, acc);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (!last) __syncthreads();  // every wave has read the input: the output may replace it
        if (has) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int n = n0 + 8 * q;
                const f32x4 bv = *reinterpret_cast<const f32x4 *>(a.bias[t.g][L] + n);
                f32x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float s = acc[0][0][4 * q + e] + bv[e];
                    v[e] = a.relu[L] != 0 && s < 0.0f ? 0.0f : s;
                }
                if (last)
                    store_last(a, t, m, n, v);
                else
                    *reinterpret_cast<bf16x4 *>(t.X + m * t.ld + n) = narrowed(v);
            }
        }
        if (!last) __syncthreads();
    }
}

// The layers of run `a` on the rows in t.X (the first layer's Kpad columns valid,
// visible to the whole block).  Each layer's output replaces its input in place:
// a wave keeps its sums in registers until every wave has read the input.  A
// wave takes chunks wave, wave + 8, ... of 32 output columns for all RT row tiles,
// or, with two row tiles and at most four chunks, one chunk of one tile.
// red: [CH_WAVES][rows] floats of LDS.
// MAXC: the most chunks a wave has in any layer, 4 (up to 1024 columns) or 1 (up to
// 256: 122 registers instead of 174 to 227, so that two blocks share a compute
// unit and a launch of more blocks than compute units does not take a second
// round for it: towers of 96-72, 264 blocks, 24.0 -> 19.4 us per forward).
// `ahead` holds the first layer's request.
template <int RT, int MAXC, class Run>
__device__ inline void run_layers(const Run &a, const RunCtx &t, Ahead<MAXC> &ahead, float *red)
{
    constexpr int R = rows_of<RT>();
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float dot_part[RT];
#pragma unroll
    for (int j = 0; j < RT; ++j) dot_part[j] = 0.0f;
    int tile = 0;
    bool split = false;  // row tiles dealt to the waves too: a wave's sums belong to row tile `tile`
    if constexpr (MAXC == 1) {
        static_assert(RT == 1, "narrow runs are on one row tile");
        narrow_layers(a, t, ahead, dot_part[0]);
    }
    for (int L = 0; MAXC > 1 && L < a.n_layers; ++L) {
        const int NC = a.Npad[L] / 32;
        split = RT == 2 && NC <= CH_WAVES / 2;
        const int first = split ? wave & (CH_WAVES / 2 - 1) : wave;
        tile = split ? wave / (CH_WAVES / 2) : 0;
        const int cnt = first < NC ? (NC - first + CH_WAVES - 1) / CH_WAVES : 0;
        if (cnt == 0) {
            if (L + 1 < a.n_layers) __syncthreads();  // the one inside layer_pass()
        } else if (split) {
            float part[1] = {0.0f};
            layer_pass<1, 1>(a, t, L, first, tile, part);
            dot_part[0] = part[0];
        } else if (cnt == 1) {
            layer_pass<1, RT>(a, t, L, first, 0, dot_part);
        } else if (cnt == 2) {
            layer_pass<2, RT>(a, t, L, first, 0, dot_part);
        } else if (cnt == 3) {
            layer_pass<3, RT>(a, t, L, first, 0, dot_part);
        } else {
            layer_pass<4, RT>(a, t, L, first, 0, dot_part);
        }
        if (L + 1 < a.n_layers) __syncthreads();
    }
    if (a.out_mode != CHAIN_OUT_DOT) return;
    // Per sample: the two half-waves, then the waves in order.
#pragma unroll
    for (int j = 0; j < RT; ++j) {
        const float d = dot_part[j] + __shfl_xor(dot_part[j], 32, 64);
        // a split layer leaves one tile's part in dot_part[0] and nothing for the other
        if (lane < 32) red[wave * R + ((split ? tile ^ j : j) * 32) + lane] = d;
    }
    __syncthreads();
    if (tid < R && (tid & 31) <= t.last_row && t.row0 + tid < a.M) {
        float sum = 0.0f;
#pragma unroll
        for (int w = 0; w < CH_WAVES; ++w) sum += red[w * R + tid];
        a.dot_out[(long long)(t.row0 + tid) * a.dot_ld + t.g] = sum + a.dot_bias[t.g][0];
    }
}

// Dynamic LDS of a block: the activations and the partial dots of its waves.
template <int RT>
constexpr size_t act_bytes(int ld) { return (size_t)rows_of<RT>() * ld * sizeof(__bf16); }
template <int RT>
constexpr size_t chain_lds_bytes(int ld) { return act_bytes<RT>(ld) + sizeof(float) * CH_WAVES * rows_of<RT>(); }

// Does MAXC = 1 take the run?
inline bool narrow_run(const ChainProblem &a)
{
    for (int L = 0; L < a.n_layers; ++L)
        if (a.Npad[L] > CHAIN_NARROW_WIDTH) return false;
    return true;
}
// Blocks a compute unit is to hold at a time: sets the registers a wave gets.
template <int MAXC>
constexpr int waves_per_simd() { return MAXC == 1 ? 4 : 2; }

// One block's share of the run: samples bx * rows ... of stack g.  The block is
// number `mine` of the `share` that run this stack on one XCD.  `smem` is
// chain_lds_bytes<RT>(a.ld_lds) of dynamic LDS; all CH_THREADS threads take part.
template <bool A_F32, int RT, int MAXC, class Run>
__device__ inline void mlp_chain_block(const Run &a, unsigned char *smem, int bx, int g, int mine, int share)
{
    __bf16 *X = reinterpret_cast<__bf16 *>(smem);
    float *red = reinterpret_cast<float *>(smem + act_bytes<RT>(a.ld_lds));
    const RunCtx t{X, nullptr, a.ld_lds, 0, g, bx * rows_of<RT>(), 31};
    const Touched touched = touch_weights(a, g, mine, share);
    Ahead<MAXC> ahead;
    ahead.request(a, g, 0);
    stage_input<A_F32, RT == 2 ? 16 : 8>(a, g, t.row0, rows_of<RT>(), X, a.ld_lds);
    touched.done();
    __syncthreads();
    run_layers<RT, MAXC>(a, t, ahead, red);
}

// The same for a narrow run into rows (no CHAIN_OUT_DOT), within 64 registers.
template <bool A_F32, class Run>
__device__ inline void light_chain_block(const Run &a, unsigned char *smem, int bx, int g, int mine, int share)
{
    __bf16 *X = reinterpret_cast<__bf16 *>(smem);
    const RunCtx t{X, nullptr, a.ld_lds, 0, g, bx * rows_of<1>(), 31};
    const Touched touched = touch_weights(a, g, mine, share);
    stage_input<A_F32, LIGHT_BATCH>(a, g, t.row0, rows_of<1>(), X, a.ld_lds);
    touched.done();
    __syncthreads();
    light_layers(a, t);
}

}  // namespace chain
}  // namespace rec
#endif
