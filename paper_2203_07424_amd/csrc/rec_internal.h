// Internal declarations shared by the gfx950 kernels and the C boundary.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "rec.h"

namespace rec {

// Device error record (64 bytes, lives at the start of the workspace).
// Positions are kept with atomicMin, so "none" is all ones.
struct ErrRecord {
    unsigned long long first_bad_len;  // smallest position of a negative length
    unsigned long long first_bad_idx;  // smallest position of an id outside its table
    unsigned int flags;                // ERR_* bits
    unsigned int pad[11];
};
enum : unsigned int { ERR_NEG_LENGTH = 1u, ERR_TOTAL_MISMATCH = 2u, ERR_INDEX_RANGE = 4u };

// What the launch that ends a forward may do besides (fault not null): fault[0] = the
// status rec_check() would give, fault[1] = its position.  A launch of one thread for it
// took 2.5 us behind the last one.
struct FaultReport {
    const ErrRecord *err = nullptr;
    long long *fault = nullptr;
};
// In a launch behind pooling's: a block of its own, so that nothing else waits for the record.
inline int report_blocks(const FaultReport &r) { return r.fault ? 1 : 0; }
__device__ inline void report_fault(const ErrRecord *err, long long *fault)
{
    if (threadIdx.x != 0) return;
    const unsigned flags = err->flags;
    long long st = REC_OK, pos = -1;
    if (flags & (ERR_NEG_LENGTH | ERR_TOTAL_MISMATCH)) {
        st = REC_ERR_LENGTHS;
        if (flags & ERR_NEG_LENGTH) pos = (long long)err->first_bad_len;
    } else if (flags & ERR_INDEX_RANGE) {
        st = REC_ERR_INDEX_RANGE;
        pos = (long long)err->first_bad_idx;
    }
    fault[0] = st;
    fault[1] = pos;
}

// A block's LDS beyond 64 KB, what the kernel declares itself included, has to be granted to the
// kernel before its first launch (not under stream capture).
template <class Kernel>
hipError_t grant_lds(Kernel kernel, size_t dynamic)
{
    const void *k = reinterpret_cast<const void *>(kernel);
    hipFuncAttributes has;
    const hipError_t e = hipFuncGetAttributes(&has, k);
    if (e != hipSuccess || has.sharedSizeBytes + dynamic <= 64 * 1024) return e;
    return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dynamic);
}

struct TableDesc {
    const void *base;
    long long rows;
    const int32_t *hot_ids;  // rows worth caching in LDS (may be null)
    int n_hot;
    int pad;
};

// S0: one scan block covers SCAN_TILE lengths.
constexpr int SCAN_THREADS = 256;
constexpr int SCAN_ITEMS = 8;
constexpr int SCAN_TILE = SCAN_THREADS * SCAN_ITEMS;

// All activations and packed weights use leading dimensions that are
// multiples of this many elements.
constexpr int PAD = 64;
inline int pad_up(int x) { return (x + PAD - 1) / PAD * PAD; }

hipError_t launch_clear_err(ErrRecord *err, hipStream_t s);

// S0. offsets[k] = min(sum_{j<k} max(len[j], 0), nnz), k = 0..n.  tile_words is
// scratch of ceil(n / SCAN_TILE) words, zero before the launch, which leaves sums in
// the first scan_linked_words() of them; the pooling launch behind it clears these
// (clear_tile_words()), and whoever owns the words clears them before their first use
// (launch_clear_tile_words()).
// With a ConcatDense job (x0 != null) extra blocks of the launch also do
// the work of launch_concat_dense(), which a model without Bottom-FC can start
// this early: its x0 is the dense input.
struct ConcatDense {
    const float *x0 = nullptr;
    int ldx0 = 0, w0 = 0, B = 0;
    void *z_bf16 = nullptr;
    int width = 0, ldz = 0;
};
// With `rider` (a stack of fully connected layers that fits the on-chip kernel,
// fp32 input, one stack) further blocks of the launch run that stack:
// Bottom-FC does not depend on the sparse side (Sec. III-A), so it can share a
// launch with the scan instead of costing one of its own.
template <int G>
struct ChainArgs;
using ChainProblem = ChainArgs<REC_MAX_TOWERS>;
constexpr int SCAN_LINK_POLLS = 65536;  // of another tile's word before its lengths are added up instead
hipError_t launch_scan(const int32_t *lengths, int n, long long nnz, int32_t *offsets,
                       unsigned long long *tile_words, ErrRecord *err, const ConcatDense &job,
                       const ChainProblem *rider, hipStream_t s, int polls = SCAN_LINK_POLLS);
// The same with the first layer of Bottom-FC instead of a whole stack, where
// scan_layer_rides(); z: its first z_cols columns, narrowed, go there as well.
struct FcProblem;
bool scan_layer_rides(const FcProblem &layer, const void *z);
hipError_t launch_scan_beside_layer(const int32_t *lengths, int n, long long nnz, int32_t *offsets,
                                    unsigned long long *tile_words, ErrRecord *err, const ConcatDense &job,
                                    const FcProblem &layer, void *z, int ldz, int z_cols, hipStream_t s);
int scan_linked_words(int n, bool with_rider);
// What the scan's blocks of a launch get; blocks [0, tiles) are theirs.
struct ScanBlocks {
    const int32_t *lengths;
    int32_t *offsets;
    unsigned long long *words;
    long long nnz;
    int n, tiles, polls;
    ErrRecord *err;
};
hipError_t launch_clear_tile_words(unsigned long long *words, int n, hipStream_t s);
// The words a scan has published, for the pooling launch behind it to clear.
struct TileWords {
    unsigned long long *words;
    int n;
};
// One wave clears the words.
__device__ inline void clear_tile_words(const TileWords &w)
{
    for (int i = threadIdx.x & 63; i < w.n; i += 64)
        __hip_atomic_store(w.words + i, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Once per process and device, before the first launch (not under stream capture).
hipError_t scan_prepare();

// Where S1 leaves the sum of bag (t, b): fp32 pooled[b][t][:], or (z != null,
// concatenation model) narrowed to bf16 at z[b][col0 + t * D ...], row stride ldz.
struct PoolOut {
    float *pooled;
    void *z;
    int ldz, col0;
};

// S1. Sum of the rows of every bag, fp32 accumulation.  nnz (the batch's id
// count) only picks the launch shape: bags of a few ids share a wavefront.  The
// words in `left` are cleared on the way.
// stream_rows: load rows with the non-temporal hint (id streams without reuse).
// max_rows: row count of the largest table (tables under 4 GiB take 32-bit offsets).
// corun: other launches share the device with this one and want wave slots.
hipError_t launch_pool(const TableDesc *tables, int dtype, int T, int D, int B,
                       const int32_t *indices, const int32_t *offsets, PoolOut out, long long nnz,
                       bool stream_rows, long long max_rows, int num_cus, bool corun, const TileWords &left, ErrRecord *err,
                       hipStream_t s);

// Which form launch_pool() takes: bags of a few ids side by side in a wave; two bags in turn in a wave; 32-bit
// byte offsets into the tables.
bool pool_short_applies(int rowbytes, long long nnz, long long bags);
bool pool_two_applies(int rowbytes, long long nnz, long long bags, bool narrow, int num_cus);
bool pool_narrow(long long max_rows, int rowbytes);

// S1 with the tables' hot rows served from an LDS copy (hcap: power of two >= the
// longest hot list, pool_hot_fits(hcap, rowbytes) must hold).
bool pool_hot_fits(int hcap, int rowbytes);
hipError_t launch_pool_hot(const TableDesc *tables, int dtype, int T, int D, int B,
                           const int32_t *indices, const int32_t *offsets, float *pooled, int hcap,
                           int num_cus, const TileWords &left, ErrRecord *err, hipStream_t s);

// S2 / S4. One layer of `groups` stacks that run side by side (the task towers
// of the Predict-FC; 1 for a single stack), stack g being
//   C_g[m][n] = act(sum_k A_g[m][k] * W_g[n][k] + bias_g[n])   on bf16 MFMA, with
//   A_g = A + g * a_stride: bf16 [M][lda] or (a_f32) fp32 [M][lda] with only k < K
//         valid; a_stride = 0 when all stacks read the same input
//   W_g: bf16 [Npad][Kpad], bias_g fp32 [Npad] (zero padded)
//   C_g = C + g * c_stride: bf16 [M][ldc] or (out_f32) fp32 [M][ldc]
// With dot_out != null (allowed when fc_can_fuse_dot(Npad)) C is not stored;
// instead dot_out[m * dot_ld + g] = sum_n act(C_g[m][n]) * dot_w_g[n] + dot_bias_g[0],
// the one-output layer that follows, in fp32.
constexpr int MAX_GROUPS = REC_MAX_TOWERS;
struct FcGroups {
    const void *W[MAX_GROUPS];
    const float *bias[MAX_GROUPS];
    const float *dot_w[MAX_GROUPS];
    const float *dot_bias[MAX_GROUPS];
};
struct FcProblem {
    const void *A; bool a_f32; int lda; long long a_stride;
    int M, K, Kpad, Npad; bool relu;
    void *C; bool out_f32; int ldc; long long c_stride;
    int groups;
    FcGroups g;
    float *dot_out; int dot_ld;
    int num_cus;  // compute units of the device; 0 = unknown (never picks the wide-tile kernels)
    bool corun;   // the launch will share the device with a pooling launch: keep register use low
    FaultReport report;  // with dot_out: made on the way
    // Each stack's weights in the order of launch_pack_chain(), for the kernels that deal
    // a tile's k to the waves of a block (sums in another order); null: not these.
    const void *frag[MAX_GROUPS];
    int waves;    // that share the k of a tile then, where that is prescribed: 4, or 0
};
bool fc_can_fuse_dot(int Npad);
hipError_t launch_fc(const FcProblem &p, hipStream_t s);

// The same layer with the k of a tile dealt to the waves of a block, for launches
// too short to fill the chip; launch_fc() takes this path by itself.
bool fc_split_applies(const FcProblem &p);
struct FcTile {
    int tm, tn;  // 16 tm rows x 16 tn columns
    int wk;      // waves that share its k
};
FcTile fc_split_tile(const FcProblem &p);      // without the one-output layer
FcTile fc_split_dot_tile(const FcProblem &p);  // with it
bool fc_takes_split(const FcProblem &p);   // does launch_fc() take this path?
// May the layer's blocks share a launch with others' (fp32 rows read in vectors)?
bool fc_split_rides(const FcProblem &p);
hipError_t launch_fc_split(const FcProblem &p, hipStream_t s);
// Once per process and device, before the first launch (not under stream capture).
hipError_t fc_split_prepare();

// The same product with 256-row block tiles (bf16 input, C stored), for layers
// wide and batches large enough that such tiles still cover the chip;
// launch_fc() takes this path by itself when fc_big_applies().
bool fc_big_applies(const FcProblem &p, int num_cus);
hipError_t launch_fc_big(const FcProblem &p, int num_cus, hipStream_t s);
FcTile fc_big_tile(const FcProblem &p, int num_cus);  // no tile: does not apply
// Does the layer take tiles of which two blocks fit a compute unit (128 x 128, fp32
// input), so that a scan's blocks may stand in front of them?
bool fc_big_rides(const FcProblem &p, int num_cus);
hipError_t launch_fc_big_behind_scan(const FcProblem &p, const ScanBlocks &scan, hipStream_t s);
// Once per process and device, before the first launch (not under stream
// capture): lets these kernels use their more-than-64-KB LDS tiles.
hipError_t fc_big_prepare();

// A run of layers of every stack in one launch, activations kept on chip:
//   X_0 = A_g (bf16 [M][lda], or fp32 with a_f32; columns >= K read as zero),
//   X_{L+1} = act_L(X_L W_{L,g}^T + bias_{L,g}),  act_L = ReLU where relu[L] != 0,
// each layer narrowing its input to bf16 as the per-layer path does.  Layer L is
// Kpad[L] -> Npad[L] with Kpad[L + 1] == Npad[L], all at most CHAIN_MAX_WIDTH
// (Kpad[0] TAIL_MAX_INPUT in a tail) and multiples of PAD; W[g][L] is the fragment order launch_pack_chain() writes.
// The last X goes to C_g = C + g * c_stride (CHAIN_OUT_BF16 / CHAIN_OUT_F32, row
// stride ldc), or (CHAIN_OUT_DOT) into the one-output layer that follows:
//   dot_out[m * dot_ld + g] = sum_n X[m][n] * dot_w[g][n] + dot_bias[g][0]   in fp32.
constexpr int CHAIN_MAX_LAYERS = 6;
constexpr int CHAIN_MAX_WIDTH = 1024;
constexpr int CHAIN_NARROW_WIDTH = 256;  // up to this many outputs in every layer: the narrow form, two blocks a compute unit
constexpr int TAIL_MAX_INPUT = 2048;  // Kpad of the first Predict-FC layer in launch_tail()
enum { CHAIN_OUT_BF16 = 0, CHAIN_OUT_F32 = 1, CHAIN_OUT_DOT = 2 };
template <int G>  // stacks there is room for: what a launch of one stack passes is a quarter of the size
struct ChainArgs {
    const void *A; bool a_f32; int lda; long long a_stride;
    int M, K;
    int n_layers, groups;
    int Kpad[CHAIN_MAX_LAYERS], Npad[CHAIN_MAX_LAYERS], relu[CHAIN_MAX_LAYERS];
    const void *W[G][CHAIN_MAX_LAYERS];
    const float *bias[G][CHAIN_MAX_LAYERS];
    int out_mode;
    void *C; int ldc; long long c_stride;
    const float *dot_w[G];
    const float *dot_bias[G];
    float *dot_out; int dot_ld;
    int num_cus;
    int ld_lds, a_vec;  // filled in by chain_finalize()
};
inline ChainArgs<1> one_stack(const ChainProblem &p)
{
    ChainArgs<1> a;
    a.A = p.A; a.a_f32 = p.a_f32; a.lda = p.lda; a.a_stride = p.a_stride;
    a.M = p.M; a.K = p.K; a.n_layers = p.n_layers; a.groups = 1;
    for (int L = 0; L < CHAIN_MAX_LAYERS; ++L) {
        a.Kpad[L] = p.Kpad[L]; a.Npad[L] = p.Npad[L]; a.relu[L] = p.relu[L];
        a.W[0][L] = p.W[0][L]; a.bias[0][L] = p.bias[0][L];
    }
    a.out_mode = p.out_mode; a.C = p.C; a.ldc = p.ldc; a.c_stride = p.c_stride;
    a.dot_w[0] = p.dot_w[0]; a.dot_bias[0] = p.dot_bias[0]; a.dot_out = p.dot_out; a.dot_ld = p.dot_ld;
    a.num_cus = p.num_cus; a.ld_lds = p.ld_lds; a.a_vec = p.a_vec;
    return a;
}
bool chain_layer_fits(int Kpad, int Npad, int max_input = CHAIN_MAX_WIDTH);
// The rounds that blocks of 64 samples (two row tiles, one block a compute unit) take,
// 0 where they fill less than three quarters of these.  (256 blocks of four 1024-512-256 towers:
// 107.7 -> 102.4 us per forward; 376, two rounds: 113.1 -> 117.8, so not there.)
int chain_two_tile_rounds(int groups, int M, int num_cus);
// Checks p and completes it (LDS row pitch, whether wide input loads apply) into a.
hipError_t chain_finalize(const ChainProblem &p, ChainProblem &a, int max_input = CHAIN_MAX_WIDTH);
hipError_t launch_mlp_chain(const ChainProblem &p, hipStream_t s, const FaultReport &report = FaultReport{});
// Once per process and device, before the first launch (not under stream capture).
hipError_t chain_prepare();
// fp32 [N][K] -> bf16 [Npad * Kpad] in MFMA fragment order (nearest even, zero padded).
hipError_t launch_pack_chain(const float *W, int N, int K, int Npad, int Kpad, void *W_packed, hipStream_t s);

// Interaction and Predict-FC of a dot model with one tower in one launch, behind
// the last layers of Bottom-FC where run[0].n_layers > 0.
//   run[0]: bf16 input, CHAIN_OUT_F32 into the x0 buffer (M rows)
//   x0:     fp32 rows of Bottom-FC's output, 16-byte aligned, ldx0 % 4 == 0 (run[0].n_layers == 0)
//   run[1]: input z (its A is not read), CHAIN_OUT_DOT
//   z:      the Predict-FC input rows, written for inspection, ldz == run[1].Kpad[0]
struct TailProblem {
    ChainProblem run[2];  // Bottom-FC part, Predict-FC
    const float *x0; int ldx0;
    const float *pooled;
    int T, D;
    void *z; int ldz;
    FaultReport report;  // made on the way
    int rows, ld_lds;  // filled in by launch_tail()
};
bool tail_fits(int T, int D);
// Samples a block takes (8, 16 or 32), and up to how many samples a compute unit
// gets no more than one block.
int tail_rows(int M, int num_cus);
int tail_most_samples(int num_cus);
hipError_t launch_tail(const TailProblem &p, int num_cus, hipStream_t s);
// Once per process and device, before the first launch (not under stream capture).
hipError_t tail_prepare();

// S0 and S1 of a small batch in one launch (front_applies()), into out.pooled or, in a
// concatenation model, out.z.  Beside them
//   rider: a whole Bottom-FC stack front_takes() (fp32 input, one stack); out.pooled only
//   layer: the first Bottom-FC layer, where front_layer_rides(); at most one of the two
//   dense: what launch_concat_dense() does for a model without Bottom-FC; with `layer`
//          only the padding (w0 = 0), the layer's output going to out.z (z_cols columns) as well
struct FrontProblem {
    const int32_t *lengths, *indices;
    long long nnz;
    int32_t *offsets;
    const TableDesc *tables;
    ErrRecord *err;
    int dtype, T, D, B;
    bool stream_rows;
    PoolOut out;
    ConcatDense dense;
    const FcProblem *layer;
    int z_cols;
    int num_cus;
};
bool front_layer_rides(const FcProblem &p, bool concat);
constexpr int FRONT_SHORT_WAVES = 4;  // that share the k of such a layer's tiles in a concatenation model
// Does a whole stack of `input` padded inputs run there within 64 registers?
bool front_takes_light(long long bags, long long nnz, int rowbytes, int input, int num_cus);
// ride_input: padded inputs of the stack that is to ride along, 0: none.
bool front_applies(int T, int B, int D, int dtype, long long nnz, long long max_rows, bool concat, int ride_input);
// More lookups than that, about one id a bag, of a concatenation model without Bottom-FC (no layer).
constexpr int SHORT_FORM_BAGS = 6 * SCAN_TILE;  // up to which bags of a few ids take csrc/front.hip's launch
hipError_t launch_lookups(const FrontProblem &f, hipStream_t s);
int lookup_dense_blocks(const ConcatDense &job, int left);  // its blocks for the dense part, `left` compute units without another
bool front_lookup_applies(int T, int B, int D, int dtype, long long nnz, int num_cus);
// The same beside a layer of 128 x 128 tiles (dot models, bags a wave each).
bool fc_big_beside_pool_applies(const FcProblem &layer, int T, int B, int D, int dtype, long long nnz, long long max_rows);
hipError_t launch_fc_big_beside_pool(const FrontProblem &f, hipStream_t s);
bool front_takes(const ChainProblem &rider);
hipError_t launch_front(const FrontProblem &f, const ChainProblem *rider, hipStream_t s);
// Once per process and device, before the first launch (not under stream capture).
hipError_t front_prepare();

// Last Predict-FC layer of every stack: logits[m * ld + g] = sum_k A_g[m][k] * w_g[k] + bias_g[0]
// in fp32.  A_g = A + g * a_stride is fp32 [M][lda] (a_f32) or bf16 [M][lda];
// w_g = groups.dot_w[g] is fp32 [Kpad], zero padded, bias_g = groups.dot_bias[g].
hipError_t launch_rowdot(const void *A, bool a_f32, int lda, long long a_stride, int M, int Kpad,
                         const FcGroups &groups, int n_groups, float *logits, int ld, hipStream_t s);
hipError_t launch_pack_dot(const float *W, const float *b, int K, int Kpad, float *W_packed,
                           float *bias_packed, hipStream_t s);

// fp32 [N][K] -> bf16 [Npad][Kpad] (nearest even, zero padded), bias -> fp32 [Npad].
hipError_t launch_pack_fc(const float *W, const float *b, int N, int K, int Npad, int Kpad,
                          void *W_packed, float *bias_packed, hipStream_t s);

// S3. out[b] = bf16([x0[b], <v_i, v_j> i > j, 0 ...]) with v = [x0[b], pooled[b][0..T-1]].
size_t interact_lds_bytes_per_sample(int T, int D);
hipError_t launch_interact(const float *x0, int ldx0, const float *pooled, int B, int T, int D,
                           void *out_bf16, int ldo, hipStream_t s);


// Concatenation model: z[b][0 .. w0) = bf16(x0[b][0 .. w0)) and z[b][width .. ldz) = 0;
// the looked-up vectors in between are written by S1.
hipError_t launch_concat_dense(const float *x0, int ldx0, int w0, int B, void *z_bf16, int width,
                               int ldz, hipStream_t s);

}  // namespace rec
