// Helpers for measurements and tests (not part of the forward pass).
//
// The rate at which the matrix cores run v_mfma_f32_32x32x16_bf16 on register
// operands, on constant or on pseudo-random values.  With every compute unit
// busy the chip is power-limited and the rate depends on the operand bits; a
// benchmark puts it beside the published peak.
#include "rec_probe.h"
#include "scan_body.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int PROBE_WAVES = 8;

__global__ __launch_bounds__(64 * PROBE_WAVES) void mfma_probe_kernel(int random_operands, int iters,
                                                                      float *__restrict__ sink)
{
    // Two weight-like and four activation-like fragments, as a 128 x 64 wave tile holds per step.
    bf16x8 fw[2], fa[4];
    // Six independent fragments: a GEMM feeds every instruction fresh operands, and the
    // power drawn follows how many operand bits change from one instruction to the next.
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        bf16x8 v;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            unsigned h = ((threadIdx.x * 8u + (unsigned)e) * 6u + (unsigned)f) * 2654435761u + 777u + blockIdx.x * 40503u;
            h ^= h >> 15;
            h *= 2246822519u;
            h ^= h >> 13;
            v[e] = (__bf16)(random_operands ? (float)((int)(h & 0xffffu) - 32768) * (1.0f / 32768.0f) : 1.0f);
        }
        if (f < 2) fw[f] = v;
        else fa[f - 2] = v;
    }
    f32x16 acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[i], fa[j], acc[i][j], 0, 0, 0);
        }
        // Sums stay bounded and the operands keep changing: flip the sign of one fragment.
        if (random_operands) {
            bf16x8 t = fw[0];
#pragma unroll
            for (int e = 0; e < 8; ++e) t[e] = -t[e];
            fw[0] = t;
        }
    }
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) s += acc[i][j][0];
    if (blockIdx.x == 0 && threadIdx.x == 0) sink[0] = s;
}

}  // namespace

extern "C" rec_status rec_probe_mfma(int32_t random_operands, int32_t blocks, int32_t iters,
                                     float *dev_sink, void *stream)
{
    if (!dev_sink || blocks <= 0 || blocks > 65536 || iters <= 0 || iters > (1 << 20)) return REC_ERR_ARG;
    hipLaunchKernelGGL(mfma_probe_kernel, dim3(blocks), dim3(64 * PROBE_WAVES), 0,
                       static_cast<hipStream_t>(stream), random_operands, iters, dev_sink);
    return hipGetLastError() == hipSuccess ? REC_OK : REC_ERR_DEVICE;
}

// The scan's launch as in a forward pass, for tests of the hand-over between its blocks.
extern "C" rec_status rec_probe_scan(const int32_t *dev_lengths, int32_t n, int64_t nnz, int32_t *dev_offsets,
                                     uint64_t *dev_words, int32_t polls, void *dev_err, void *stream)
{
    static_assert(REC_SCAN_POLLS == rec::SCAN_LINK_POLLS && sizeof(rec::ErrRecord) == 64, "as rec_probe.h says");
    if (!dev_lengths || !dev_offsets || !dev_words || !dev_err || n < 1 || nnz < 0 || nnz >= (1ll << 31) || polls < 0 ||
        polls > rec::SCAN_LINK_POLLS)
        return REC_ERR_ARG;
    const hipError_t e = rec::launch_scan(dev_lengths, n, nnz, dev_offsets, reinterpret_cast<unsigned long long *>(dev_words),
                                          static_cast<rec::ErrRecord *>(dev_err), rec::ConcatDense{}, nullptr,
                                          static_cast<hipStream_t>(stream), polls);
    return e == hipSuccess ? REC_OK : REC_ERR_DEVICE;
}

// launch_fc()'s choice, on pointers that nothing follows.
extern "C" rec_status rec_probe_fc_form(int32_t rows, int32_t inputs, int32_t outputs, int32_t stacks, uint32_t flags,
                                        int32_t compute_units, int32_t *form)
{
    using namespace rec;
    static char some[16] __attribute__((aligned(16)));
    const bool dot = (flags & REC_FC_DOT) != 0;
    if (!form || rows < 1 || rows > (1 << 30) || inputs < 1 || outputs < 1 || inputs > (1 << 20) || outputs > (1 << 20) || stacks < 1 ||
        stacks > MAX_GROUPS || compute_units < 1)
        return REC_ERR_ARG;
    FcProblem p{};
    p.A = some; p.a_f32 = (flags & REC_FC_F32_ROWS) != 0;
    p.M = rows; p.K = inputs; p.Kpad = (inputs + 63) / 64 * 64; p.Npad = (outputs + 63) / 64 * 64;
    p.lda = p.a_f32 ? p.K : stacks * p.Kpad;
    p.groups = stacks; p.num_cus = compute_units; p.corun = (flags & REC_FC_BESIDE_POOLING) != 0;
    for (int g = 0; g < stacks && (flags & REC_FC_ANY_ORDER) && !p.corun; ++g) p.frag[g] = some;
    if (dot) p.dot_out = reinterpret_cast<float *>(some);
    if (dot && !fc_can_fuse_dot(p.Npad)) return REC_ERR_ARG;
    FcTile t{0, 0, 0};
    form[0] = REC_FORM_TILES;
    if (fc_takes_split(p)) {
        form[0] = REC_FORM_SPLIT;
        t = dot ? fc_split_dot_tile(p) : fc_split_tile(p);
    } else if (!dot && fc_big_applies(p, compute_units)) {
        form[0] = REC_FORM_WIDE;
        t = fc_big_tile(p, compute_units);
    }
    form[1] = 16 * t.tm; form[2] = 16 * t.tn; form[3] = t.wk;
    return REC_OK;
}

extern "C" rec_status rec_probe_dense_copy(int32_t rows, int32_t columns, int32_t pad, int32_t left, int32_t *deal)
{
    using namespace rec;
    static float some[1];
    if (!deal || rows < 1 || rows > (1 << 24) || columns < 0 || columns > (1 << 16) || pad < 0 || pad >= PAD || left < -1) return REC_ERR_ARG;
    ConcatDense job;
    job.x0 = some; job.w0 = columns; job.B = rows;
    job.width = columns; job.ldz = columns + pad;
    deal[1] = left < 0 ? SCAN_THREADS / 64 : 16;
    deal[0] = left < 0 ? scan::concat_dense_blocks(job, deal[1]) : lookup_dense_blocks(job, left);
    const int all = scan::dense_units(rows, columns, pad).all, waves = deal[0] * deal[1];
    deal[2] = waves > 0 ? (all + waves - 1) / waves : 0;
    return REC_OK;
}
