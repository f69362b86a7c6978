// S2 / S4 as one kernel per stack: a run of fully connected layers whose
// activations never leave the compute unit (the FC stacks of Sec. II-A and
// Table I are narrow: a few hundred to a thousand units per layer).
//
// A block owns 32 samples, or 64 where that still gives (nearly) every compute
// unit a block.  Their input row is brought into LDS as bf16 once; every layer
// then reads its input from there and, once every wave has read it, leaves its
// output (bias, ReLU, narrowed to bf16) in its place, so between the first read
// and the last write only weights move.  The weights come straight from global
// memory (they stay in L2 across blocks) into the MFMA operand registers: they
// are stored fragment by fragment, 64 lanes x 16 bytes each, so every load of a
// wave is one contiguous KiB.  The product is computed transposed,
// D[n][m] = sum_k W[n][k] X[m][k] on v_mfma_f32_32x32x16_bf16: a lane then holds
// four consecutive outputs of one sample and stores them with one instruction.
//
// Wave w of the eight takes the 32-column chunks w, w + 8, ... of a layer, up to
// four at a time.
//
// What bounds it: the weights of the run through each compute unit's L1.  A
// read-only loop over the same fragments gets 53 bytes a clock and compute unit
// on 128 of them and 48 on all; with its products this kernel gets 44.  With the
// activation fragments read right where they are used it got 25 to 36 (0.4 MB of
// weights, 4096 samples: 14.6 -> 10.8 us; the end of a 2560-wide Bottom-FC and
// its Predict-FC as chains 104 -> 89 us per forward).  Two row tiles halve the
// weights a sample asks for: four towers of 1024-512-256, 4096 samples 50 -> 32 us
// behind the first layer (32.8 as launches of their own).
//
// The run ends in fp32 or bf16 rows in global memory, or - the Predict-FC's
// one-output layer - in a dot product of the last activations (fp32, before
// any narrowing) with that layer's weights, summed in a fixed order.
#include "mlp_chain_body.h"

namespace rec {

namespace {

using namespace chain;

template <bool A_F32, int RT, int MAXC>
__global__ __launch_bounds__(CH_THREADS, waves_per_simd<MAXC>()) void mlp_chain_kernel(int blocks, int per_group, const ChainProblem a, const FaultReport report)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    touch_args<8 + sizeof(a) + sizeof(report)>();
    if ((int)blockIdx.x == blocks) {
        report_fault(report.err, report.fault);
        return;
    }
    // Blocks run over the samples of stack 0, then stack 1, ...; XCD x (blocks are
    // dealt round-robin) takes the x-th eighth of that list, so that its L2 holds
    // the weights of one stack or two instead of all of them.
    const bool eighths = (blocks & 7) == 0;
    const int v = eighths ? (blockIdx.x & 7) * (blocks >> 3) + (blockIdx.x >> 3) : blockIdx.x;
    const int g = v / per_group, bx = v - g * per_group;
    const int share = eighths ? min(32, min(per_group, blocks >> 3)) : touch_share(per_group);
    mlp_chain_block<A_F32, RT, MAXC>(a, smem, bx, g, (eighths ? bx : bx >> 3) % share, share);
}

// fp32 [N][K] -> bf16 fragments: element e of lane l of fragment (nc, ks) is
// W[32 nc + l % 32][16 ks + 8 (l / 32) + e], zero outside the matrix.
__global__ __launch_bounds__(256) void pack_chain_kernel(const float *__restrict__ W, int N, int K, int Npad,
                                                         int Kpad, __bf16 *__restrict__ Wp)
{
    const long long lanes = (long long)Npad * Kpad / 8;  // a thread writes a lane's eight elements
    const int KS = Kpad / 16;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < lanes;
         i += (long long)gridDim.x * blockDim.x) {
        const long long frag = i >> 6;
        const int lane = (int)(i & 63);
        const long long nc = frag / KS;
        const int n = (int)nc * 32 + (lane & 31), k0 = (int)(frag - nc * KS) * 16 + (lane >> 5) * 8;
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (__bf16)((n < N && k0 + e < K) ? W[(long long)n * K + k0 + e] : 0.0f);
        *reinterpret_cast<bf16x8 *>(Wp + 8 * i) = o;
    }
}

}  // namespace

bool chain_layer_fits(int Kpad, int Npad, int max_input) { return Kpad <= max_input && Npad <= CHAIN_MAX_WIDTH; }

namespace {

template <bool A_F32, int RT, int MAXC>
hipError_t prepare_as()
{
    return hipFuncSetAttribute(reinterpret_cast<const void *>(mlp_chain_kernel<A_F32, RT, MAXC>),
                               hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)chain_lds_bytes<RT>(CHAIN_MAX_WIDTH + CH_LDS_PAD));
}

template <bool A_F32, int RT, int MAXC>
hipError_t launch_as(const ChainProblem &a, const FaultReport &report, hipStream_t s)
{
    const int per_group = (a.M + rows_of<RT>() - 1) / rows_of<RT>();
    hipLaunchKernelGGL((mlp_chain_kernel<A_F32, RT, MAXC>), dim3(per_group * a.groups + report_blocks(report)), dim3(CH_THREADS),
                       (chain_lds_bytes<RT>(a.ld_lds)), s, per_group * a.groups, per_group, a, report);
    return hipGetLastError();
}

}  // namespace

hipError_t chain_prepare()
{
    hipError_t e = prepare_as<true, 1, 1>();
    if (e == hipSuccess) e = prepare_as<true, 1, 4>();
    if (e == hipSuccess) e = prepare_as<false, 1, 1>();
    if (e == hipSuccess) e = prepare_as<false, 1, 4>();
    if (e == hipSuccess) e = prepare_as<false, 2, 4>();
    return e;
}

hipError_t chain_finalize(const ChainProblem &p, ChainProblem &a, int max_input)
{
    if (p.n_layers < 1 || p.n_layers > CHAIN_MAX_LAYERS || p.groups < 1 || p.groups > MAX_GROUPS)
        return hipErrorInvalidValue;
    int widest = p.Kpad[0];
    for (int L = 0; L < p.n_layers; ++L) {
        if (p.Kpad[L] % PAD != 0 || p.Npad[L] % PAD != 0 || !chain_layer_fits(p.Kpad[L], p.Npad[L], L == 0 ? max_input : CHAIN_MAX_WIDTH))
            return hipErrorInvalidValue;
        if (L > 0 && p.Kpad[L] != p.Npad[L - 1]) return hipErrorInvalidValue;
        if (L + 1 < p.n_layers) widest = widest > p.Npad[L] ? widest : p.Npad[L];
    }
    if (p.K > p.Kpad[0]) return hipErrorInvalidValue;
    a = p;
    a.ld_lds = widest + CH_LDS_PAD;
    // Wide loads of the input rows need aligned rows that end on a vector boundary.
    const int vec = p.a_f32 ? 4 : 8;
    const int esz = p.a_f32 ? 4 : 2;
    a.a_vec = reinterpret_cast<uintptr_t>(p.A) % 16 == 0 && p.lda % vec == 0 && p.a_stride % vec == 0 &&
              (p.a_f32 ? p.K % vec == 0 : true) && (long long)p.lda * esz % 16 == 0;
    if (p.out_mode != CHAIN_OUT_DOT) {
        const int ov = 4;
        if (reinterpret_cast<uintptr_t>(p.C) % 16 != 0 || p.ldc % ov != 0 || p.c_stride % ov != 0)
            return hipErrorInvalidValue;
    }
    return hipSuccess;
}

int chain_two_tile_rounds(int groups, int M, int num_cus)
{
    if (num_cus <= 0) return 0;
    const long long blocks = (long long)groups * ((M + 63) / 64), rounds = (blocks + num_cus - 1) / num_cus;
    return 4 * blocks >= 3 * rounds * num_cus ? (int)rounds : 0;
}

hipError_t launch_mlp_chain(const ChainProblem &p, hipStream_t s, const FaultReport &report)
{
    if (p.M <= 0) return hipSuccess;
    ChainProblem a;
    const hipError_t e = chain_finalize(p, a);
    if (e != hipSuccess) return e;
    if (narrow_run(a)) return a.a_f32 ? launch_as<true, 1, 1>(a, report, s) : launch_as<false, 1, 1>(a, report, s);
    if (a.a_f32) return launch_as<true, 1, 4>(a, report, s);
    return chain_two_tile_rounds(a.groups, a.M, a.num_cus) > 0 ? launch_as<false, 2, 4>(a, report, s) : launch_as<false, 1, 4>(a, report, s);
}

hipError_t launch_pack_chain(const float *W, int N, int K, int Npad, int Kpad, void *W_packed, hipStream_t s)
{
    const long long lanes = (long long)Npad * Kpad / 8;
    const int blocks = (int)((lanes + 255) / 256 < 4096 ? (lanes + 255) / 256 : 4096);
    hipLaunchKernelGGL(pack_chain_kernel, dim3(blocks), dim3(256), 0, s, W, N, K, Npad, Kpad,
                       static_cast<__bf16 *>(W_packed));
    return hipGetLastError();
}

}  // namespace rec
