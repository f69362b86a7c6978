// S3 and S4 in one launch, with the end of S2 in front where that is a stack of
// narrow layers: everything behind pooling for a block of samples, nothing of it
// leaving the compute unit but the buffers a caller may inspect.
//
//   [last layers of Bottom-FC ->] interaction -> Predict-FC -> logits
//
// As launches of their own these cost 3 to 5 us each before they do anything (launch,
// cold weights, one trip through memory between two kernels), more than their
// work on the models here.  A block of 8 waves owns 8, 16 or 32 samples: each wave
// does the interaction of its samples in registers (interact_body.h) and leaves
// their Predict-FC input rows in LDS, where the stack of layers finds them
// (mlp_chain_body.h).  Every block streams all weights of its layers from the L2,
// whatever the number of its samples, so the samples a block takes only decide how
// far the interaction is spread: as few as give each compute unit one block.
//
// What bounds it: 40 tables of 64 columns, 4096 samples, 884-512-128-1: 8 of 27 us
// are the pooled vectors from memory (42 MB, 5.4 TB/s), 10 the first layer's
// weights (0.9 MB through every compute unit's L1, 44 bytes a clock), the rest
// launch, cold lines and the narrow layers; 31.6 us as three launches.  With the
// end of a 2560-1024-256-32 Bottom-FC in front (4096 samples, 10 tables, 0.95 MB of
// weights) 24 against 37.5 us in five launches; 10 tables, 1024 samples (0.1 MB)
// 8.9 against 11.5 in two.  32 samples a block instead of 16 at 4096: 32.1 us
// instead of 29.4, half of the compute units having no block.
#include "interact_body.h"
#include "mlp_chain_body.h"

namespace rec {

namespace {

using namespace chain;

// What the kernel gets of a TailProblem.
struct TailArgs {
    ChainArgs<1> run[2];
    const float *x0;
    const float *pooled;
    void *z;
    int ldx0, T, ldz, rows, ld_lds, blocks;
    FaultReport report;
};

template <int NBLK, int KST, int MAXC>
__global__ __launch_bounds__(CH_THREADS) void tail_kernel(const TailArgs p)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int D = 32 * KST;
    touch_args<sizeof(TailArgs)>();
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rows = p.rows, row0 = blockIdx.x * rows;
    if ((int)blockIdx.x == p.blocks) {
        report_fault(p.report.err, p.report.fault);
        return;
    }
    const int ld = p.ld_lds;
    __bf16 *X = reinterpret_cast<__bf16 *>(smem);                        // [rows][ld]
    float *x0s = reinterpret_cast<float *>(X + (size_t)rows * ld);      // [rows][D], with a Bottom-FC part
    float *red = x0s + (p.run[0].n_layers ? (size_t)rows * D : 0);      // [CH_WAVES][32]

    // Blocks behind those that have samples are there for this alone: cold weights
    // come in as fast as all compute units can ask for them.
    const int share = touch_share(p.blocks), mine = (blockIdx.x >> 3) % share;
    const Touched touched = touch_weights(p.run[1], 0, mine, share);
    if (row0 >= p.run[1].M) {
        touch_weights(p.run[0], 0, mine, share).done();
        touched.done();
        return;
    }
    // Twice through the same code: the Bottom-FC part (if any), then Predict-FC.
    for (int part = p.run[0].n_layers ? 0 : 1; part < 2; ++part) {
        if (part == 0) {
            const Touched first = touch_weights(p.run[0], 0, mine, share);
            stage_input<false, 4>(p.run[0], 0, row0, rows, X, ld);
            first.done();
        } else {
            for (int r = wave; r < rows && row0 + r < p.run[1].M; r += CH_WAVES) {
                const long long b = row0 + r;
                inter::RawRows<NBLK, KST> raw;
                raw.load(p.run[0].n_layers ? nullptr : p.x0 + b * p.ldx0, p.pooled + b * p.T * D, p.T, lane);
                if (p.run[0].n_layers) raw.load_x0(x0s + r * D, lane);
                inter::gram_row<NBLK, KST>(raw, p.T, X + r * ld, p.ldz, lane);
                // the row as a caller may inspect it
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                for (int c = lane; c < p.ldz / 8; c += 64)
                    *reinterpret_cast<u32x4 *>(static_cast<__bf16 *>(p.z) + b * p.ldz + 8 * c) =
                        *reinterpret_cast<const u32x4 *>(X + r * ld + 8 * c);
            }
            touched.done();
        }
        Ahead<MAXC> ahead;
        ahead.request(p.run[part], 0, 0);
        __syncthreads();
        run_layers<1, MAXC>(p.run[part], RunCtx{X, part == 0 ? x0s : nullptr, ld, D, 0, row0, rows - 1}, ahead, red);
        __syncthreads();
    }
}

size_t tail_lds_bytes(const TailProblem &p)
{
    const int D = p.D;
    return (size_t)p.rows * p.ld_lds * sizeof(__bf16) + (p.run[0].n_layers ? sizeof(float) * p.rows * D : 0) +
           sizeof(float) * CH_WAVES * 32;
}
constexpr size_t TAIL_LDS = 32 * (TAIL_MAX_INPUT + CH_LDS_PAD) * sizeof(__bf16) + 32 * 64 * sizeof(float) + sizeof(float) * CH_WAVES * 32;

template <int NBLK, int KST>
hipError_t launch_as(const TailProblem &p, int num_cus, hipStream_t s)
{
    const int blocks = (p.run[1].M + p.rows - 1) / p.rows, grid = blocks < num_cus ? num_cus : blocks;
    auto k = narrow_run(p.run[0]) && narrow_run(p.run[1]) ? tail_kernel<NBLK, KST, 1> : tail_kernel<NBLK, KST, 4>;
    hipLaunchKernelGGL(k, dim3(grid + report_blocks(p.report)), dim3(CH_THREADS), tail_lds_bytes(p), s,
                       TailArgs{{one_stack(p.run[0]), one_stack(p.run[1])}, p.x0, p.pooled, p.z, p.ldx0, p.T, p.ldz, p.rows, p.ld_lds, grid, p.report});
    return hipGetLastError();
}

template <int NBLK, int KST>
hipError_t prepare_as()
{
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(tail_kernel<NBLK, KST, 1>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)TAIL_LDS);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(tail_kernel<NBLK, KST, 4>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)TAIL_LDS);
}

}  // namespace

bool tail_fits(int T, int D) { return inter::fits_wave(T, D); }

int tail_rows(int M, int num_cus)
{
    int rows = 8;
    while (rows < 32 && (M + rows - 1) / rows > num_cus) rows *= 2;
    return rows;
}

int tail_most_samples(int num_cus) { return 32 * num_cus; }

hipError_t tail_prepare()
{
    hipError_t e = prepare_as<1, 1>();
    if (e == hipSuccess) e = prepare_as<2, 1>();
    if (e == hipSuccess) e = prepare_as<3, 1>();
    if (e == hipSuccess) e = prepare_as<4, 1>();
    if (e == hipSuccess) e = prepare_as<1, 2>();
    if (e == hipSuccess) e = prepare_as<2, 2>();
    if (e == hipSuccess) e = prepare_as<3, 2>();
    if (e == hipSuccess) e = prepare_as<4, 2>();
    return e;
}

hipError_t launch_tail(const TailProblem &q, int num_cus, hipStream_t s)
{
    if (q.run[1].M <= 0) return hipSuccess;
    if (!tail_fits(q.T, q.D) || q.run[1].groups != 1 || q.run[1].out_mode != CHAIN_OUT_DOT || q.ldz != q.run[1].Kpad[0])
        return hipErrorInvalidValue;
    TailProblem p = q;
    hipError_t e = chain_finalize(q.run[1], p.run[1], TAIL_MAX_INPUT);
    if (e != hipSuccess) return e;
    p.ld_lds = p.run[1].ld_lds;
    if (q.run[0].n_layers) {
        if (q.run[0].a_f32 || q.run[0].groups != 1 || q.run[0].out_mode != CHAIN_OUT_F32 || q.run[0].M != q.run[1].M ||
            q.run[0].Npad[q.run[0].n_layers - 1] < q.D)
            return hipErrorInvalidValue;
        e = chain_finalize(q.run[0], p.run[0]);
        if (e != hipSuccess) return e;
        p.ld_lds = p.run[0].ld_lds > p.ld_lds ? p.run[0].ld_lds : p.ld_lds;
        p.run[0].ld_lds = p.run[1].ld_lds = p.ld_lds;
    } else if (q.ldx0 % 4 != 0 || reinterpret_cast<uintptr_t>(q.x0) % 16 != 0) {
        return hipErrorInvalidValue;
    }
    p.rows = tail_rows(p.run[1].M, num_cus);
    if (tail_lds_bytes(p) > TAIL_LDS) return hipErrorInvalidValue;
    switch ((p.T + 16) / 16 * 2 + p.D / 32 - 1) {
    case 2: return launch_as<1, 1>(p, num_cus, s);
    case 3: return launch_as<1, 2>(p, num_cus, s);
    case 4: return launch_as<2, 1>(p, num_cus, s);
    case 5: return launch_as<2, 2>(p, num_cus, s);
    case 6: return launch_as<3, 1>(p, num_cus, s);
    case 7: return launch_as<3, 2>(p, num_cus, s);
    case 8: return launch_as<4, 1>(p, num_cus, s);
    default: return launch_as<4, 2>(p, num_cus, s);
    }
}

}  // namespace rec
