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
// 16 samples, 1728 -> 1024 four towers 12.2 / 4.4; 300 samples 17.3 / 11.2, 1024 -> 512 8.5 / 6.3,
// 512 -> 256 -> 1 10.5 / 6.2; 256 samples, 884 -> 512 8.5 / 3.5, 512 -> 128 -> 1 6.0 / 4.2;
// one sample of 2560 fp32 -> 1024 16.8 / 4.6.
//
// Where two or more blocks share a compute unit they cover one another's trips, and more waves a
// block or more units in flight a wave change nothing or lose; a block by itself has eight waves for it.
#include "gemm_split_body.h"

namespace rec {

namespace {

using namespace split;

// Of the arguments the leading scalars, up to 14 words, are in registers when a wave
// starts; the rest is a trip to cold memory that loads need not wait for.
template <int TM, int TN, int WN, int WK, int IN, int OUT>
__global__ __launch_bounds__(64 * WN * WK, TM * TN >= 16 || (IN != IN_BF16 && TM * TN >= 8) ? 2 : 4) void fc_split_kernel(
    const void *__restrict__ A0, const void *__restrict__ W0, int lda, int M, int K, int Kpad, int grid_m, int grid_n,
    int m_fast, int per_xcd, int n_groups, int relu, long long a_stride, void *__restrict__ C0, int ldc,
    long long c_stride, float *__restrict__ dot_out, int dot_ld, const SplitGroups<MAX_GROUPS> groups, const FaultReport report)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    if (OUT == CHAIN_OUT_DOT && (int)blockIdx.x == 8 * per_xcd) {
        report_fault(report.err, report.fault);
        return;
    }
    split_block<TM, TN, WN, WK, IN, OUT>(SplitLayer{A0, W0, lda, M, K, Kpad, grid_m, grid_n, m_fast, per_xcd, n_groups, relu,
                                                    a_stride, C0, ldc, c_stride, dot_out, dot_ld, 0, nullptr, 0, 0},
                                         groups, smem, blockIdx.x);
}

template <int TM, int TN, int WN, int WK, int IN, int OUT>
hipError_t launch_as(const FcProblem &a, hipStream_t s)
{
    SplitGroups<MAX_GROUPS> g{};
    for (int i = 0; i < a.groups; ++i) g.s[i] = SplitStack{a.frag[i], a.g.bias[i], a.g.dot_w[i], a.g.dot_bias[i]};
    const SplitLayer p = layer_in_tiles(a, TM, TN, WN);
    hipLaunchKernelGGL((fc_split_kernel<TM, TN, WN, WK, IN, OUT>), dim3(8 * p.per_xcd + report_blocks(a.report)), dim3(64 * WN * WK),
                       (split_lds_bytes<TM, TN, WN, WK>()), s, p.A, p.W0, p.lda, p.M, p.K, p.Kpad, p.grid_m, p.grid_n,
                       p.m_fast, p.per_xcd, p.n_groups, p.relu, p.a_stride, p.C, p.ldc, p.c_stride, p.dot_out, p.dot_ld, g, a.report);
    return hipGetLastError();
}

template <int IN, int OUT>
hipError_t launch_tiles(const FcProblem &a, hipStream_t s)
{
    const FcTile t = fc_split_tile(a);
    switch (t.tm * 100 + t.tn * 10 + t.wk) {
    case 118: return launch_as<1, 1, 1, 8, IN, OUT>(a, s);
    case 128: return launch_as<1, 2, 1, 8, IN, OUT>(a, s);
    case 224: return launch_as<2, 2, 1, 4, IN, OUT>(a, s);
    case 228: return launch_as<2, 2, 1, 8, IN, OUT>(a, s);
    case 244: return launch_as<2, 4, 1, 4, IN, OUT>(a, s);
    case 248: return launch_as<2, 4, 1, 8, IN, OUT>(a, s);
    case 348: return launch_as<3, 4, 1, 8, IN, OUT>(a, s);
    case 444: return launch_as<4, 4, 1, 4, IN, OUT>(a, s);
    case 548: return launch_as<5, 4, 1, 8, IN, OUT>(a, s);
    }
    if constexpr (IN == IN_BF16) {  // fp32 rows cost twice as much: 32 x 64 in two rounds is always less
        if (t.tm == 4 && t.wk == 8) return launch_as<4, 4, 1, 8, IN, OUT>(a, s);
    }
    return hipErrorInvalidValue;
}

// In front of the one-output layer rows are bf16.
hipError_t launch_dot(const FcProblem &a, hipStream_t s)
{
    constexpr int IN = IN_BF16;
    switch (a.Npad + fc_split_dot_tile(a).tm) {
    case 64 + 1: return launch_as<1, 4, 1, 8, IN, CHAIN_OUT_DOT>(a, s);
    case 128 + 1: return launch_as<1, 4, 2, 4, IN, CHAIN_OUT_DOT>(a, s);
    case 128 + 2: return launch_as<2, 4, 2, 4, IN, CHAIN_OUT_DOT>(a, s);
    case 256 + 1: return launch_as<1, 4, 4, 2, IN, CHAIN_OUT_DOT>(a, s);
    case 256 + 2: return launch_as<2, 4, 4, 2, IN, CHAIN_OUT_DOT>(a, s);
    case 256 + 4: return launch_as<4, 4, 4, 2, IN, CHAIN_OUT_DOT>(a, s);
    }
    return hipErrorInvalidValue;
}

template <int IN>
hipError_t launch_in(const FcProblem &a, hipStream_t s)
{
    return a.out_f32 ? launch_tiles<IN, CHAIN_OUT_F32>(a, s) : launch_tiles<IN, CHAIN_OUT_BF16>(a, s);
}

template <int TM, int TN, int WN, int WK, int IN, int OUT>
hipError_t prepare_as()
{
    return grant_lds(fc_split_kernel<TM, TN, WN, WK, IN, OUT>, split_lds_bytes<TM, TN, WN, WK>());
}

template <int TM, int IN>
hipError_t prepare_tiles()
{
    const hipError_t e = prepare_as<TM, 4, 1, 8, IN, CHAIN_OUT_BF16>();
    return e == hipSuccess ? prepare_as<TM, 4, 1, 8, IN, CHAIN_OUT_F32>() : e;
}

template <int IN>
hipError_t prepare_in()
{
    const hipError_t e = prepare_tiles<3, IN>();
    return e == hipSuccess ? prepare_tiles<5, IN>() : e;
}

}  // namespace

// A compute unit spends its time bringing both operands of its blocks through its L1 (25 bytes a
// clock where it has one block of eight waves, 36 where two cover one another) and, once, on the launch and
// the trips of a first block that nothing covers, about 3 us: rounds of blocks plus about one, times the
// rows and columns of a tile.  With one block a
// compute unit eight waves share its k, else four, and two blocks cover one another's trips;
// tiles of 48 and 80 rows, one block a compute unit at a time, pay that once more in every
// round.  us per launch (64 x 64 or 32 x 64 with four waves, the choice without these two /
// now): 300 samples, four of 1728 -> 1024 14.8 / 11.2 (80 rows, 256 blocks), 1024 -> 512
// 7.4 / 6.3 (48 rows, 224), two of 1728 -> 1024 10.7 / 8.4; 2560 fp32 -> 1024, 300 samples 11.8 / 10.2,
// 700 17.7 / 14.6, 1200 24.2 / 20.8.  Blocks of 96 rows never won, and those of 80 only in one
// round: in many each block's loads, sums and stores lie bare (64 rows / 80; 256 -> 192, 40960 samples 20.4
// / 30.2; 1024 -> 704, 32768 96 / 118).
FcTile fc_split_tile(const FcProblem &a)
{
    struct Form {
        int tm, tn, wk1, wk, once1, once;  // waves and uncovered part (tenths of a round), in one round and in several (0: not)
    };
    static const Form forms[] = {{1, 1, 8, 8, 10, 11}, {1, 2, 8, 8, 10, 11}, {2, 2, 8, 4, 10, 11}, {2, 4, 8, 4, 10, 11},
                                 {3, 4, 8, 8, 11, 14}, {4, 4, 8, 4, 11, 11}, {5, 4, 8, 8, 11, 0}};
    const int cus = a.num_cus > 0 ? a.num_cus : 256;
    FcTile best{0, 0, 0};
    long long least = 0;
    for (const Form &f : forms) {
        const long long blocks = (long long)((a.M + 16 * f.tm - 1) / (16 * f.tm)) * (a.Npad / (16 * f.tn)) * a.groups;
        const long long rounds = (blocks + cus - 1) / cus;
        if ((rounds > 1 && f.once == 0) || (a.waves > 0 && f.wk != a.waves)) continue;
        const long long cost = (f.tm * (a.a_f32 ? 2 : 1) + f.tn) * (10 * rounds + (rounds == 1 ? f.once1 : f.once));
        if (best.tm == 0 || cost < least) {
            // Eight waves with a unit each gain nothing, and most fp32 layers run beside pooling,
            // whose waves four leave more room (us per forward, eight / four: 500 samples beside 10 tables, 600 -> 1024
            // 27.0 / 26.1, 2560 33.3 / 31.3; 1000 beside 4, 1000 -> 512 26.4 / 24.2, beside 6, 1536 29.3 / 28.0).
            const bool four = a.Kpad <= 8 * UNIT || (a.a_f32 && f.tn == 4 && 4 * blocks > 3 * cus);
            best = FcTile{f.tm, f.tn, rounds > 1 || a.waves > 0 || (four && f.tm == 2) ? f.wk : f.wk1};
            least = cost;
        }
    }
    return best;
}

// With the one-output layer: a block has all columns, and as many rows as still give
// every compute unit a block.  128 columns in blocks of 16 / 32 rows, us per launch: 1024 inputs, 5120
// samples 11.2 / 9.4, 8192 11.6 / 9.6, 10240 14.5 / 13.2 (k-tile by k-tile 10.7, 10.8, 14.1).
FcTile fc_split_dot_tile(const FcProblem &a)
{
    const long long cus = a.num_cus > 0 ? a.num_cus : 256, blocks16 = (a.M + 15) / 16 * (long long)a.groups;
    if (a.Npad == 64) return FcTile{1, 4, 8};
    if (a.Npad == 128) return FcTile{blocks16 <= cus ? 1 : 2, 8, 4};
    return FcTile{blocks16 <= cus ? 1 : blocks16 <= 2 * cus ? 2 : 4, 16, 2};
}

hipError_t fc_split_prepare()
{
    hipError_t e = prepare_as<4, 4, 4, 2, IN_BF16, CHAIN_OUT_DOT>();
    if (e == hipSuccess) e = prepare_tiles<4, IN_BF16>();
    if (e == hipSuccess) e = prepare_in<IN_BF16>();
    if (e == hipSuccess) e = prepare_in<IN_F32>();
    if (e == hipSuccess) e = prepare_in<IN_F32_ANY>();
    return e;
}

bool fc_split_applies(const FcProblem &a)
{
    for (int g = 0; g < a.groups; ++g)
        if (!a.frag[g]) return false;
    // 32-bit byte offsets inside a block's rows and a stack's weights
    return a.lda <= 1 << 22 && (long long)a.Npad * a.Kpad <= 1ll << 30;
}

bool fc_split_rides(const FcProblem &a)
{
    return a.a_f32 && a.groups == 1 && !a.dot_out && fc_takes_split(a) && rows_in_vectors(a);
}

hipError_t launch_fc_split(const FcProblem &a, hipStream_t s)
{
    if (a.dot_out) return a.a_f32 ? hipErrorInvalidValue : launch_dot(a, s);
    if (!a.a_f32) return launch_in<IN_BF16>(a, s);
    return rows_in_vectors(a) ? launch_in<IN_F32>(a, s) : launch_in<IN_F32_ANY>(a, s);
}

}  // namespace rec
