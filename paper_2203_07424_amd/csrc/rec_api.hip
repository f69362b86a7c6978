// C boundary of the forward pass: model bookkeeping on the host and the fixed
// launch sequence  scan -> pool -> Bottom-FC -> interaction -> Predict-FC
// (interaction = pairwise dots, or plain concatenation for the MT-WnD shape of
// Table I, whose Predict-FC is N towers run side by side).
// Bottom-FC does not depend on the SparseNet and Predict-FC waits for both
// (Sec. III-A); on one in-order stream that dependency is the launch order.
#include <algorithm>
#include <mutex>
#include <new>
#include <vector>

#include "rec_internal.h"
#include "rec_probe.h"

using namespace rec;

// Scratch memory of rec_forward_static(): one copy per GPU the library runs on,
// held until the process ends.  In host code this name is only a handle for
// hipGetSymbolAddress(); kernels get the address that call returns.
static __device__ __align__(256) unsigned char scratch[REC_STATIC_SCRATCH_BYTES];

namespace {

constexpr size_t ALIGN = 256;
inline size_t align_up(size_t x) { return (x + ALIGN - 1) / ALIGN * ALIGN; }

struct Layer {
    int K = 0, N = 0, Kpad = 0, Npad = 0;
    const void *W = nullptr;      // bf16 [Npad][Kpad]; fp32 [Kpad] for the one-output layer
    const float *bias = nullptr;  // fp32 [Npad]
    bool dot = false;             // last Predict-FC layer: fp32 dot product, not a GEMM
    bool chain = false;           // narrow enough for the kernel that runs several layers on chip
    const void *Wc = nullptr;     // the weights in MFMA fragment order
    bool loaded = false;
    size_t w_bytes() const { return dot ? sizeof(float) * Kpad : 2 * (size_t)Npad * Kpad; }
    size_t chain_bytes() const { return dot ? 0 : 2 * (size_t)Npad * Kpad; }
};

}  // namespace

// Where the parts of a forward's scratch memory sit inside one block of device
// memory (byte offsets; every part 256-byte aligned).  The error record and the
// table descriptors exist once; what one batch passes through (a frame) once
// up to four times.
constexpr int MAX_FRAMES = 4;
struct Frame {
    size_t off_offsets = 0, off_tile_words = 0, off_pooled = 0, off_x0 = 0, off_act[3] = {0, 0, 0};
};
struct Carve {
    size_t off_err = 0, off_tables = 0, bytes = 0;
    Frame fr[MAX_FRAMES];
};

struct rec_model {
    int T = 0, D = 0, F = 0, dtype = REC_F32;
    int interaction = REC_INTERACT_DOT;
    int towers = 1, n_top = 0;  // top holds towers * n_top layers, tower-major
    int w0 = 0;                 // width of the dense part x0 of the Predict-FC input
    int z_width = 0;            // width of the Predict-FC input
    int max_batch = 0;
    long long max_nnz = 0;
    std::vector<long long> rows;
    long long max_rows = 0;  // of the largest table
    std::vector<Layer> bottom, top;
    std::vector<char> table_loaded;
    std::vector<TableDesc> desc;  // host copy of the device descriptors
    int num_cus = 256;

    Carve lay;               // carve-up of the bound workspace, sized for max_batch
    int z_ld = 0;            // padded width of the interaction output (act[0])
    int act_ld = 0;          // widest padded hidden activation row (elements), act[1], act[2]
    size_t act_row_bytes = 0;  // bytes of one activation row: bf16 everywhere, fp32 into the dot layer
    int x0_ld = 0;           // row stride of the Bottom-FC output in the workspace
    char *ws = nullptr;

    // Bottom-FC runs on a stream of the library's own, beside scan and pooling.
    bool overlap_dense = false;
    bool stream_rows = false;  // pooling loads rows with the non-temporal hint
    int fuse_mlp = 1;          // runs of narrow layers through the on-chip chain kernel: 0 never, 1 where it pays, 2 always
    hipStream_t side = nullptr;
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;

    // Sparse-dense pipeline: a batch owns one of four frames of the workspace
    // until its logits are written.  Scan and Bottom-FC run on the caller's
    // stream, pooling on two streams in turn, interaction and Predict-FC on a
    // fourth; these events order them.
    bool pipeline = false;
    hipStream_t dense_stream = nullptr;              // the caller's choice, else `side`
    hipStream_t pool_stream[2] = {nullptr, nullptr}; // the caller's choice, else own_stream
    hipStream_t own_stream[2] = {nullptr, nullptr};
    hipEvent_t ev_scan[MAX_FRAMES] = {}, ev_bottom[MAX_FRAMES] = {}, ev_pool[MAX_FRAMES] = {}, ev_tail[MAX_FRAMES] = {};
    bool tail_pending[MAX_FRAMES] = {};  // Predict-FC of that frame's batch enqueued, not yet waited for
    bool words_left[MAX_FRAMES] = {};    // a call failed with its scan perhaps enqueued and its pooling not: tile words to be cleared
    int next_frame = 0, last_frame = 0;
    int pool_turn = 0;                   // which pooling stream takes the next batch

    // Stage timing: forward number i records into slot i % slots.
    std::vector<hipEvent_t> ev;  // slots * EV_PER_SLOT
    std::vector<char> slot_mode; // per slot: 1 recorded by a pipelined forward, 2 in order with Bottom-FC inside the scan's launch
    std::vector<uint32_t> slot_shared;  // per slot: stages without a launch of their own (rec_stage_shared())
    int slots = 0, period = 1;
    long long forwards = 0;      // forwards seen since profiling was switched on

    template <class P>
    P *at(size_t off) const { return reinterpret_cast<P *>(ws + off); }
};

namespace {

// Scratch layout of model m for batches of up to `batch` samples, with `frames`
// (1 or MAX_FRAMES) copies of the per-batch part.
Carve carve(const rec_model *m, int batch, int frames)
{
    const bool concat = m->interaction == REC_INTERACT_CONCAT;
    const size_t nb = (size_t)m->T * batch;
    Carve c;
    size_t o = 0;
    c.off_err = o;    o += align_up(sizeof(ErrRecord));
    c.off_tables = o; o += align_up(sizeof(TableDesc) * m->T);
    for (int f = 0; f < frames; ++f) {
        Frame &fr = c.fr[f];
        fr.off_offsets = o;   o += align_up(sizeof(int32_t) * (nb + 1));
        fr.off_tile_words = o; o += align_up(sizeof(long long) * ((nb + SCAN_TILE - 1) / SCAN_TILE));
        fr.off_pooled = o;    o += concat ? 0 : align_up(sizeof(float) * nb * m->D);
        fr.off_x0 = o;        o += !m->bottom.empty() ? align_up(sizeof(float) * (size_t)batch * m->x0_ld) : 0;
        // act[0] holds the Predict-FC input (kept for inspection); the hidden
        // activations of both stacks alternate between act[1] and act[2].
        fr.off_act[0] = o; o += align_up(2 * (size_t)batch * m->z_ld);
        fr.off_act[1] = o; o += align_up((size_t)batch * m->act_row_bytes);
        fr.off_act[2] = o; o += align_up((size_t)batch * m->act_row_bytes);
    }
    for (int f = frames; f < MAX_FRAMES; ++f) c.fr[f] = c.fr[0];
    c.bytes = o;
    return c;
}

}  // namespace

namespace {

// Can S3 + S4 run as the one launch of csrc/tail.hip?
bool tail_possible(const rec_model *m)
{
    const int n = m->n_top - 1;  // layers ahead of the one-output layer
    if (m->interaction != REC_INTERACT_DOT || m->towers != 1 || n < 1 || n > CHAIN_MAX_LAYERS || !tail_fits(m->T, m->D))
        return false;
    for (int i = 0; i < n; ++i)
        if (!chain_layer_fits(m->top[i].Kpad, m->top[i].Npad, i == 0 ? TAIL_MAX_INPUT : CHAIN_MAX_WIDTH)) return false;
    return true;
}

bool all_loaded(const rec_model *m)
{
    for (char c : m->table_loaded)
        if (!c) return false;
    for (const Layer &l : m->bottom)
        if (!l.loaded) return false;
    for (const Layer &l : m->top)
        if (!l.loaded) return false;
    return true;
}

Layer *find_layer(rec_model *m, int which, int layer)
{
    if (which == REC_BOTTOM) {
        if (layer < 0 || layer >= (int)m->bottom.size()) return nullptr;
        return &m->bottom[layer];
    }
    const int tower = which - REC_TOP;
    if (tower < 0 || tower >= m->towers || layer < 0 || layer >= m->n_top) return nullptr;
    return &m->top[(size_t)tower * m->n_top + layer];
}

}  // namespace

namespace {

// The buffers one forward passes through: pointers into a scratch block.
struct Bufs {
    ErrRecord *err;
    const TableDesc *tables;
    int32_t *offsets;
    unsigned long long *tile_words;
    float *pooled;
    float *x0;      // Bottom-FC output (unused without a Bottom-FC)
    void *act[3];
};

Bufs bufs_at(char *base, const Carve &c, int frame)
{
    const Frame &f = c.fr[frame];
    Bufs b;
    b.err = reinterpret_cast<ErrRecord *>(base + c.off_err);
    b.tables = reinterpret_cast<const TableDesc *>(base + c.off_tables);
    b.offsets = reinterpret_cast<int32_t *>(base + f.off_offsets);
    b.tile_words = reinterpret_cast<unsigned long long *>(base + f.off_tile_words);
    b.pooled = reinterpret_cast<float *>(base + f.off_pooled);
    b.x0 = reinterpret_cast<float *>(base + f.off_x0);
    for (int i = 0; i < 3; ++i) b.act[i] = base + f.off_act[i];
    return b;
}

// Scan tiles of the largest batch.
int most_tiles(const rec_model *m) { return (int)(((size_t)m->T * m->max_batch + SCAN_TILE - 1) / SCAN_TILE); }

// Arguments of one forward.
struct Call {
    const float *dense;
    const int32_t *indices;
    const int32_t *lengths;
    int B;
    long long nnz;
    float *logits;
    FaultReport *report;  // rec_forward_static(): where the call's faults go; handed (fault nulled) to the launch that reports them
};

// Stage events of one timed forward (null: not timed).  Slot i of the array is
// recorded by mark(i); which events bracket which stage depends on where the
// stages were enqueued (stage_events()).
enum { EV_BEGIN = 0, EV_SCAN_END = 1, EV_POOL_END = 2, EV_BOTTOM_FIRST_END = 3, EV_BOTTOM_END = 4,
       EV_INTERACT_END = 5, EV_TOP_FIRST_END = 6, EV_END = 7, EV_BOTTOM_BEGIN = 8, EV_INTERACT_BEGIN = 9,
       EV_POOL_BEGIN = 10, EV_PER_SLOT = 11 };

inline hipError_t mark(hipEvent_t *ev, int which, hipStream_t s)
{
    return ev ? hipEventRecord(ev[which], s) : hipSuccess;
}

#define REC_TRY(call)                          \
    do {                                       \
        const hipError_t e_ = (call);          \
        if (e_ != hipSuccess) return e_;       \
    } while (0)

// A run of chain layers [i, j) of one or several stacks side by side, layer l of
// stack k being layers[k * per_stack + l].
void chain_run(const Layer *layers, int per_stack, int G, int i, int j, int num_cus, ChainProblem &c)
{
    c.n_layers = j - i;
    c.groups = G;
    c.K = layers[i].K;
    c.num_cus = num_cus;
    for (int l = i; l < j; ++l) {
        c.Kpad[l - i] = layers[l].Kpad;
        c.Npad[l - i] = layers[l].Npad;
        c.relu[l - i] = 1;
        for (int k = 0; k < G; ++k) {
            c.W[k][l - i] = layers[(size_t)k * per_stack + l].Wc;
            c.bias[k][l - i] = layers[(size_t)k * per_stack + l].bias;
        }
    }
}

// How far a chain that starts at layer i of n reaches (i: no chain here).  Every
// block of a chain streams all weights of its run, which costs more than the
// launches it saves once they no longer are a small fraction of a block's L1
// bandwidth over a launch time: left to itself (fuse_mlp == 1) the library
// chains runs of up to CHAIN_AUTO_BYTES of weights, and only where that saves
// a launch (dot_after: the one-output layer follows layer n - 1).  Where blocks of
// 64 samples fill the chip each sample asks for half of that and runs of any size
// win (four towers of 1024-512-256, 4096 samples: 107.7 -> 102.4 us per forward).
// In more than one round of blocks a launch saved no longer counts, and what is left
// is the activations that stay on chip: not enough for several towers that save one
// launch and up to 512 columns (two rounds, separate / chained: four of 1024-512-256
// 183.0 / 192.0, eight of 512-256 59.9 / 67.5; but eight of 1024-256 101.0 / 97.5, two
// of 512-256 110.3 / 107.2, four of 512-512-512 141.6 / 126.9).
// Runs of narrow layers keep blocks of 32, two a compute unit, so for them it is that
// many bytes for each launch saved (us per forward of four towers in separate launches /
// chained; 192 KiB a launch: 256-256-256 behind a wide layer, 4096 samples 53.7 / 50.8,
// 512-256-256-256-256-256 84.4 / 73.3; 384: 1024-256-256-256 95.0 / 94.8, 12288 samples
// 252.1 / 255.3; 640: 1024-256-256 89.3 / 90.6, 8192 samples 159.6 / 167.7).
// G stacks side by side, B samples; a_f32: the run starts from the dense input.
int chain_end(const rec_model *m, const Layer *layers, int i, int n, int G, int B, bool a_f32, bool dot_after)
{
    constexpr size_t CHAIN_AUTO_BYTES = 256 * 1024;
    if (m->fuse_mlp == 0 || (m->pipeline && m->fuse_mlp == 1)) return i;
    int j = i;
    size_t bytes = 0;
    bool narrow = true;
    for (; j < n && layers[j].chain && j - i < CHAIN_MAX_LAYERS; ++j) {
        bytes += layers[j].chain_bytes();
        narrow = narrow && layers[j].Npad <= CHAIN_NARROW_WIDTH;
    }
    if (m->fuse_mlp == 2 || j == i) return j;
    const int saved = (j - i - 1) + (dot_after && j == n && !fc_can_fuse_dot(layers[j - 1].Npad) ? 1 : 0);
    if (saved < 1) return i;
    if (const int rounds = a_f32 ? 0 : chain_two_tile_rounds(G, B, m->num_cus); rounds > 0) {
        if (narrow) return bytes > saved * CHAIN_AUTO_BYTES ? i : j;
        if (saved > 1 || rounds == 1 || G < 4 || layers[i].Npad > 512) return j;
    }
    return bytes > CHAIN_AUTO_BYTES ? i : j;
}

// May a layer's launch deal the k of a tile to the waves of a block?  With the forms
// prescribed (fuse_mlp 0 or 2) and beside pooling sums run over k in order, so that
// a layer's result is the same bits in a pipelined model as in an in-order one.
bool splits(const rec_model *m) { return m->fuse_mlp == 1 && !m->pipeline; }

// Layer i of Bottom-FC as a launch of its own, on rows A.
FcProblem bottom_layer(const rec_model *m, int i, const Call &c, const void *A, bool a_f32, int lda, void *C, int ldc)
{
    const Layer &l = m->bottom[i];
    FcProblem p{};
    p.A = A; p.a_f32 = a_f32; p.lda = lda;
    p.M = c.B; p.relu = true; p.groups = 1; p.num_cus = m->num_cus; p.corun = m->pipeline;
    p.K = l.K; p.Kpad = l.Kpad; p.Npad = l.Npad;
    p.g.W[0] = l.W; p.g.bias[0] = l.bias;
    if (splits(m)) p.frag[0] = l.Wc;
    p.C = C; p.out_f32 = i + 1 == (int)m->bottom.size(); p.ldc = ldc;
    // Beside the short bags of a small batch a layer is in blocks of four waves; where it has a
    // launch to itself all the same (a timed forward, REC_OPT_OVERLAP_DENSE) its sums are to be the same bits.
    if (m->interaction == REC_INTERACT_CONCAT && m->bottom.size() == 1 &&
        front_applies(m->T, c.B, m->D, m->dtype, c.nnz, m->max_rows, true, 0) && front_layer_rides(p, true))
        p.waves = FRONT_SHORT_WAVES;
    return p;
}
// Its first layer.
FcProblem first_bottom_layer(const rec_model *m, const Bufs &u, const Call &c)
{
    const bool last = m->bottom.size() == 1;
    return bottom_layer(m, 0, c, c.dense, true, m->F, last ? static_cast<void *>(u.x0) : u.act[1], last ? m->x0_ld : m->act_ld);
}

// S2: ReLU after every layer; the last one leaves fp32 for the interaction.  Of
// the layers only the first `upto_layer`, the tail kernel taking the others
// (their input: *rest, row stride *rest_ld); first_done: without the first, which
// first_bottom_layer() has described to the launch that took it.
hipError_t enqueue_bottom(const rec_model *m, const Bufs &u, const Call &c, hipStream_t s, hipEvent_t *ev,
                          int upto_layer, bool first_done, const void **rest, int *rest_ld)
{
    const int all = (int)m->bottom.size(), n = upto_layer;
    const Layer *layers = m->bottom.data();
    const void *A = c.dense;
    bool a_f32 = true;
    int lda = m->F, launches = 0, i = 0;
    if (first_done) {
        const FcProblem p = first_bottom_layer(m, u, c);
        A = p.C; lda = p.ldc; a_f32 = false;
        launches = i = 1;  // of a forward that is not timed
    }
    while (i < n) {
        const int j = chain_end(m, layers, i, n, 1, c.B, a_f32, false);
        const int upto = j > i ? j : i + 1;
        const bool last = upto == all;
        void *C = last ? static_cast<void *>(u.x0) : u.act[1 + (launches & 1)];
        const int ldc = last ? m->x0_ld : m->act_ld;
        if (j > i) {
            ChainProblem cp{};
            cp.A = A; cp.a_f32 = a_f32; cp.lda = lda; cp.a_stride = 0; cp.M = c.B;
            chain_run(layers, all, 1, i, j, m->num_cus, cp);
            cp.out_mode = last ? CHAIN_OUT_F32 : CHAIN_OUT_BF16;
            cp.C = C; cp.ldc = ldc; cp.c_stride = 0;
            REC_TRY(launch_mlp_chain(cp, s));
        } else {
            REC_TRY(launch_fc(bottom_layer(m, i, c, A, a_f32, lda, C, ldc), s));
        }
        A = C; lda = ldc; a_f32 = false;
        if (launches++ == 0) REC_TRY(mark(ev, EV_BOTTOM_FIRST_END, s));  // the first launch is timed on its own
        i = upto;
    }
    if (launches == 0) REC_TRY(mark(ev, EV_BOTTOM_FIRST_END, s));
    if (rest) { *rest = A; *rest_ld = lda; }
    return mark(ev, EV_BOTTOM_END, s);
}
hipError_t enqueue_bottom(const rec_model *m, const Bufs &u, const Call &c, hipStream_t s, hipEvent_t *ev)
{
    return enqueue_bottom(m, u, c, s, ev, (int)m->bottom.size(), false, nullptr, nullptr);
}

// Bottom-FC does not depend on the sparse side (Sec. III-A): when the whole
// stack is one run of the on-chip kernel, an in-order forward lets it ride on
// the scan's launch instead of giving it a launch of its own (9-11 us on
// every workload here, whatever its size).
bool bottom_rides_on_scan(const rec_model *m)
{
    const int n = (int)m->bottom.size();
    return n > 0 && !m->pipeline && !m->overlap_dense && chain_end(m, m->bottom.data(), 0, n, 1, 1, true, false) == n;
}

// The first layer of Bottom-FC that the tail kernel would take (none: the number of
// layers): a run of narrow layers at its end, behind at least one layer that
// narrows the input, when the stack does not ride on the scan as a whole.  A layer
// with more weights than a launch is worth stays one of its own, all compute units
// fetching them: 320, 960, 1920 KiB in blocks of 8, 16, 32 samples (us per forward with
// the layer in the joint launch / on its own; 512 KiB: 1 sample 27.3 / 25.2, 300 39.7 / 38.0, 2048
// 63.6 / 62.9, 3000 67.4 / 70.2; 800 KiB: 300 36.2 / 32.5, 4096 65.3 / 69.5; 1 MiB: 300 44.9 / 39.7,
// 3000 67.3 / 61.3, 4096 68.0 / 68.0; 2 MiB: 4096 77.4 / 67.9).
size_t tail_layer_bytes(const rec_model *m, int B)
{
    const int rows = tail_rows(B, m->num_cus);
    return (rows == 8 ? 320 : rows == 16 ? 960 : 1920) * 1024;
}
int tail_bottom_from(const rec_model *m, int B)
{
    const int n = (int)m->bottom.size();
    if (m->overlap_dense || m->pipeline || bottom_rides_on_scan(m)) return n;
    int i = n;
    while (i > 1 && m->bottom[i - 1].chain && n - i < CHAIN_MAX_LAYERS &&
           (m->fuse_mlp == 2 || m->bottom[i - 1].chain_bytes() <= tail_layer_bytes(m, B)))
        --i;
    return i;
}

// Do S3 and S4 of this call run as the one launch of csrc/tail.hip?  A block streams
// all weights whatever its samples, 10 us a MB, so it is a question of the weights
// for each launch it takes the place of.  us per forward as separate launches / as
// one; at small batches (B = 256) 1 MiB for 2: 45.4 / 47.2, 0.9 for 4: 57.8 / 48.7,
// so 320 KiB a launch.  From a dozen samples a compute unit the separate layers are
// past their launch cost as well, but blocks of 16 samples leave half of each
// matrix instruction idle: at 12 and 16 samples a compute unit (40 tables of 64,
// Predict-FC of two or more layers; 10 tables of 32, 2560-wide Bottom-FC)
//   1 MiB for 2     72.6 / 72.5    86.3 / 85.7     2.5 for 4   88.0 / 83.5   101.1 / 98.9
//   1.5 for 2       78.2 / 77.3    88.3 / 90.7     2.8 for 4   91.6 / 90.6   103.8 / 106.5
//   2 for 2         75.9 / 83.2    90.7 / 96.8     4.4 for 4  102.2 / 104.7  113.9 / 121.6
//   9.8 for 5      126.1 / 168.0  147.7 / 194.4    6.4 for 5  115.9 / 133.3  127.7 / 150.3
// so 640 KiB a launch; in blocks of 32 (20 and 32 samples a compute unit)
//   1.5 for 2      101.5 / 105.3  152.6 / 147.4    2.5 for 4  126.4 / 116.6  151.0 / 146.4
//   3.8 for 2      130.8 / 129.8  183.6 / 173.7    6.4 for 5  168.8 / 162.9  197.3 / 194.9
//   5 for 2        180.6 / 181.6  256.2 / 250.9    9.8 for 5  191.7 / 199.9  249.3 / 270.6
// 1920.  With more samples than compute units can take in one round of blocks it
// loses (64 a unit, 1 MiB for 2: 892 / 900, 0.9 for 4: 251 / 260).
bool tail_applies(const rec_model *m, const Call &c)
{
    if (m->fuse_mlp == 0 || !tail_possible(m)) return false;
    if (m->bottom.empty() && (m->F % 4 != 0 || reinterpret_cast<uintptr_t>(c.dense) % 16 != 0)) return false;
    if (m->fuse_mlp == 2) return true;
    if (m->pipeline || c.B > tail_most_samples(m->num_cus)) return false;
    const int n = m->n_top - 1, nb = (int)m->bottom.size();
    size_t bytes = 0, launches = 0;  // of the layers the launch would take
    for (int i = 0; i < n;) {
        const int j = chain_end(m, m->top.data(), i, n, 1, c.B, false, true);
        for (int l = i; l < std::max(j, i + 1); ++l) bytes += m->top[l].chain_bytes();
        i = std::max(j, i + 1);
        ++launches;
    }
    for (int i = tail_bottom_from(m, c.B); i < nb; ++i, ++launches) bytes += m->bottom[i].chain_bytes();
    const size_t kib = c.B < 12 * m->num_cus ? 320 : tail_rows(c.B, m->num_cus) < 32 ? 640 : 1920;
    return bytes <= launches * kib * 1024;
}

// A concatenation model without Bottom-FC has the dense part of its Predict-FC
// input rows written by spare blocks of the scan: one launch less in front of S4.
bool concat_rides_on_scan(const rec_model *m)
{
    return m->interaction == REC_INTERACT_CONCAT && m->bottom.empty();
}

// Bottom-FC as a run that rides along with the sparse side.
ChainProblem bottom_run(const rec_model *m, const Bufs &u, const Call &c)
{
    const int n = (int)m->bottom.size();
    ChainProblem cp{};
    cp.A = c.dense; cp.a_f32 = true; cp.lda = m->F; cp.a_stride = 0; cp.M = c.B;
    chain_run(m->bottom.data(), n, 1, 0, n, m->num_cus, cp);
    cp.out_mode = CHAIN_OUT_F32;
    cp.C = u.x0; cp.ldc = m->x0_ld; cp.c_stride = 0;
    return cp;
}

ConcatDense concat_job(const rec_model *m, const Bufs &u, const Call &c)
{
    ConcatDense job;
    job.x0 = c.dense; job.ldx0 = m->F; job.w0 = m->w0; job.B = c.B;
    job.z_bf16 = u.act[0]; job.width = m->z_width; job.ldz = m->z_ld;
    return job;
}

int longest_hot_list(const rec_model *m, bool use_hot)
{
    int hmax = 0;
    if (use_hot)
        for (const TableDesc &d : m->desc) hmax = d.n_hot > hmax ? d.n_hot : hmax;
    return hmax;
}

PoolOut pool_out(const rec_model *m, const Bufs &u)
{
    return m->interaction == REC_INTERACT_CONCAT ? PoolOut{nullptr, u.act[0], m->z_ld, m->w0}
                                                 : PoolOut{u.pooled, nullptr, 0, 0};
}

// Which stages of a forward share a launch; decided once per call.
struct Plan {
    bool ride = false;   // Bottom-FC in the scan's launch
    bool front = false;  // scan (and Bottom-FC, with ride) in the pooling launch
    bool layer = false;  // Bottom-FC's first layer in the launch of the scan
    bool joined = false;  // scan and pooling in the launch of that layer, in large tiles
    bool tail = false;   // interaction, Predict-FC and the Bottom-FC layers [tail_from, ...) in one launch
    int tail_from = 0;
};

// S0 and S1 (and Bottom-FC, with_bottom) of a small in-order batch as one launch,
// where csrc/front.hip has one for it (timed: of the more bags that a stack's light form is for, scan
// and pooling are to have an interval each).  With layer by layer prescribed (fuse_mlp 0) only
// where no layer is involved, in a concatenation model without Bottom-FC.
bool front_applies_to(const rec_model *m, const Call &c, bool use_hot, bool with_bottom, bool timed)
{
    const bool concat = m->interaction == REC_INTERACT_CONCAT;
    if (m->pipeline || (m->overlap_dense && !m->bottom.empty()) || (concat && with_bottom)) return false;
    if (m->fuse_mlp == 0 && !concat_rides_on_scan(m)) return false;
    if (!concat && longest_hot_list(m, use_hot) > 0) return false;
    if (concat_rides_on_scan(m) && m->fuse_mlp != 0 && !timed && front_lookup_applies(m->T, c.B, m->D, m->dtype, c.nnz, m->num_cus))
        return true;
    if (with_bottom)
        for (const Layer &l : m->bottom)
            if (l.Npad > CHAIN_NARROW_WIDTH) return false;
    return front_applies(m->T, c.B, m->D, m->dtype, c.nnz, m->max_rows, concat, with_bottom && !timed ? m->bottom[0].Kpad : 0);
}

// Does Bottom-FC's first layer, which waits for nothing, run beside the scan (and
// pooling, p.front)?  (In a concatenation model as the only layer, its output being
// part of the Predict-FC input rows.)
bool first_layer_rides(const rec_model *m, const Bufs &u, const Call &c, const Plan &p)
{
    const bool concat = m->interaction == REC_INTERACT_CONCAT;
    if (m->fuse_mlp == 0 || m->pipeline || m->overlap_dense || p.ride || m->bottom.empty() || (concat && m->bottom.size() > 1))
        return false;
    if (chain_end(m, m->bottom.data(), 0, p.tail_from, 1, c.B, true, false) > 0) return false;
    const FcProblem first = first_bottom_layer(m, u, c);
    return p.front ? front_layer_rides(first, concat) : scan_layer_rides(first, concat ? u.act[0] : nullptr);
}

// Does pooling join the launch of the scan and a first layer of large tiles?
bool pool_joins_layer(const rec_model *m, const Bufs &u, const Call &c, bool use_hot)
{
    if (m->interaction == REC_INTERACT_CONCAT || longest_hot_list(m, use_hot) > 0) return false;
    const FcProblem first = first_bottom_layer(m, u, c);
    return !fc_split_rides(first) && fc_big_beside_pool_applies(first, m->T, c.B, m->D, m->dtype, c.nnz, m->max_rows);
}

hipError_t enqueue_front(const rec_model *m, const Bufs &u, const Call &c, const Plan &plan, hipStream_t s)
{
    FrontProblem f{};
    f.lengths = c.lengths; f.indices = c.indices; f.nnz = c.nnz;
    f.offsets = u.offsets; f.tables = u.tables; f.err = u.err;
    f.dtype = m->dtype; f.T = m->T; f.D = m->D; f.B = c.B;
    f.stream_rows = m->stream_rows;
    f.num_cus = m->num_cus;
    f.out = pool_out(m, u);
    if (m->interaction == REC_INTERACT_CONCAT) {
        f.dense = concat_job(m, u, c);
        if (!concat_rides_on_scan(m)) f.dense.w0 = 0;  // the padding only
    }
    FcProblem first{};
    if (plan.layer) {
        first = first_bottom_layer(m, u, c);
        f.layer = &first;
        f.z_cols = m->w0;
    }
    ChainProblem cp{};
    if (plan.ride) cp = bottom_run(m, u, c);
    return launch_front(f, plan.ride ? &cp : nullptr, s);
}

// timed: a forward whose stages are timed gives those an interval of their own that have
// a launch to themselves layer by layer; the joint launches of the first layer only pay
// where nothing stands between the launches.
Plan plan_of(const rec_model *m, const Bufs &u, const Call &c, bool use_hot, bool timed)
{
    Plan p;
    p.ride = bottom_rides_on_scan(m);
    p.front = front_applies_to(m, c, use_hot, p.ride, timed);
    if (timed && !p.ride && !concat_rides_on_scan(m)) p.front = false;
    p.tail = tail_applies(m, c);
    p.tail_from = p.tail ? tail_bottom_from(m, c.B) : (int)m->bottom.size();
    p.layer = !timed && first_layer_rides(m, u, c, p);
    if (p.front && !p.layer && !timed) {  // a layer too large to run beside pooling still may beside the scan
        Plan q = p;
        q.front = false;
        q.layer = first_layer_rides(m, u, c, q);
        if (q.layer) p = q;
    }
    p.joined = p.layer && !p.front && pool_joins_layer(m, u, c, use_hot);
    return p;
}

hipError_t enqueue_scan(const rec_model *m, const Bufs &u, const Call &c, const Plan &plan, hipStream_t s)
{
    ConcatDense job;
    if (plan.layer) {
        const bool concat = m->interaction == REC_INTERACT_CONCAT;
        if (concat) {
            job = concat_job(m, u, c);
            job.w0 = 0;  // the padding only
        }
        return launch_scan_beside_layer(c.lengths, m->T * c.B, c.nnz, u.offsets, u.tile_words, u.err, job,
                                        first_bottom_layer(m, u, c), concat ? u.act[0] : nullptr, m->z_ld, m->w0, s);
    }
    if (concat_rides_on_scan(m)) job = concat_job(m, u, c);
    ChainProblem cp{};
    if (plan.ride) cp = bottom_run(m, u, c);
    return launch_scan(c.lengths, m->T * c.B, c.nnz, u.offsets, u.tile_words, u.err, job, plan.ride ? &cp : nullptr, s);
}

// Launches of layers [0, n) of G stacks side by side.
int launches_of(const rec_model *m, const Layer *layers, int n, int G, int B, bool a_f32, bool dot_after)
{
    int launches = 0;
    for (int i = 0; i < n; ++launches) i = std::max(chain_end(m, layers, i, n, G, B, a_f32 && i == 0, dot_after), i + 1);
    return launches;
}

// The stages that have no launch of their own under plan p (bits REC_STAGE_*).
uint32_t shared_stages(const rec_model *m, const Plan &p, int B)
{
    const int n = m->n_top - 1;
    uint32_t s = 0;
    const auto in_another = [&s](int stage) { s |= 1u << stage; };
    if (p.front) in_another(REC_STAGE_SCAN);
    const int bottom = p.ride ? 0 : launches_of(m, m->bottom.data(), p.tail_from, 1, B, true, false);
    if (bottom < 1) in_another(REC_STAGE_BOTTOM_FIRST);
    if (bottom < 2) in_another(REC_STAGE_BOTTOM_REST);
    if (p.tail || concat_rides_on_scan(m)) in_another(REC_STAGE_INTERACT);
    // Does the one-output layer fold into the launch of the layers in front of it?
    int top = launches_of(m, m->top.data(), n, m->towers, B, false, true);
    bool folded = n > 0 && fc_can_fuse_dot(m->top[n - 1].Npad);
    for (int i = 0; i < n && !folded;) {
        const int j = chain_end(m, m->top.data(), i, n, m->towers, B, false, true);
        folded = j > i && j == n;
        i = std::max(j, i + 1);
    }
    if (!folded) ++top;
    if (p.tail || top < 2) in_another(REC_STAGE_TOP_REST);
    return s;
}

// S1.  With hot lists registered (and use_hot), hot rows are served from LDS.  In the
// concatenation model the sums go straight into the Predict-FC input rows.
// with_bottom: Bottom-FC or its first layer shared the scan's launch.
hipError_t enqueue_pool(const rec_model *m, const Bufs &u, const Call &c, bool use_hot, hipStream_t s, bool with_bottom)
{
    const TileWords left{u.tile_words, scan_linked_words(m->T * c.B, with_bottom)};
    const int B = c.B, T = m->T, D = m->D;
    const bool concat = m->interaction == REC_INTERACT_CONCAT;
    const int hmax = longest_hot_list(m, use_hot);
    if (hmax > 0 && !concat) {
        // Capacity: at least the longest list; a sparse hash (128 slots of rows
        // or more, where LDS allows) keeps the per-wave probe chains short.
        const int rowbytes = D * (m->dtype == REC_F16 ? 2 : 4);
        int hcap = 16;
        while (hcap < hmax) hcap *= 2;
        while (hcap < 128 && pool_hot_fits(hcap * 2, rowbytes)) hcap *= 2;
        REC_TRY(launch_pool_hot(u.tables, m->dtype, T, D, B, c.indices, u.offsets, u.pooled, hcap,
                                m->num_cus, left, u.err, s));
    } else {
        REC_TRY(launch_pool(u.tables, m->dtype, T, D, B, c.indices, u.offsets, pool_out(m, u), c.nnz, m->stream_rows,
                            m->max_rows, m->num_cus, m->pipeline || m->overlap_dense, left, u.err, s));
    }
    return hipSuccess;
}

hipError_t enqueue_sparse(const rec_model *m, const Bufs &u, const Call &c, const Plan &plan, bool use_hot,
                          hipStream_t s, hipEvent_t *ev)
{
    if (plan.front || plan.joined) {  // all of it in the pooling stage; the scan's reads an empty interval
        REC_TRY(mark(ev, EV_SCAN_END, s));
        REC_TRY(enqueue_front(m, u, c, plan, s));
        return mark(ev, EV_POOL_END, s);
    }
    REC_TRY(enqueue_scan(m, u, c, plan, s));
    REC_TRY(mark(ev, EV_SCAN_END, s));
    REC_TRY(enqueue_pool(m, u, c, use_hot, s, plan.ride || plan.layer));
    return mark(ev, EV_POOL_END, s);
}

// The report of call c, for the launch that is to make it.
FaultReport take_report(const Call &c)
{
    if (!c.report) return FaultReport{};
    const FaultReport r = *c.report;
    c.report->fault = nullptr;
    return r;
}

// S3 and S4 in one launch, behind the Bottom-FC layers [from, ...) on `rest`.
hipError_t enqueue_fused_tail(const rec_model *m, const Bufs &u, const Call &c, hipStream_t s, hipEvent_t *ev,
                              int from, const void *rest, int rest_ld)
{
    const int nb = (int)m->bottom.size(), n = m->n_top - 1;
    TailProblem t{};
    if (from < nb) {
        ChainProblem &b = t.run[0];
        b.A = rest; b.a_f32 = false; b.lda = rest_ld; b.M = c.B;
        chain_run(m->bottom.data(), nb, 1, from, nb, m->num_cus, b);
        b.out_mode = CHAIN_OUT_F32;
        b.C = u.x0; b.ldc = m->x0_ld;
    }
    // Without a Bottom-FC the dense part of the Predict-FC input is the dense input.
    t.x0 = nb ? u.x0 : c.dense;
    t.ldx0 = nb ? m->x0_ld : m->F;
    t.pooled = u.pooled; t.T = m->T; t.D = m->D;
    t.z = u.act[0]; t.ldz = m->z_ld;
    t.report = take_report(c);
    t.run[1].A = u.act[0]; t.run[1].lda = m->z_ld; t.run[1].M = c.B;
    chain_run(m->top.data(), m->n_top, 1, 0, n, m->num_cus, t.run[1]);
    t.run[1].out_mode = CHAIN_OUT_DOT;
    t.run[1].dot_w[0] = static_cast<const float *>(m->top[n].W);
    t.run[1].dot_bias[0] = m->top[n].bias;
    t.run[1].dot_out = c.logits; t.run[1].dot_ld = 1;
    REC_TRY(mark(ev, EV_INTERACT_END, s));
    REC_TRY(launch_tail(t, m->num_cus, s));
    REC_TRY(mark(ev, EV_TOP_FIRST_END, s));
    return mark(ev, EV_END, s);
}

// S3 and S4.
hipError_t enqueue_tail(const rec_model *m, const Bufs &u, const Call &c, const Plan &plan, hipStream_t s,
                        hipEvent_t *ev)
{
    if (plan.tail) return enqueue_fused_tail(m, u, c, s, ev, (int)m->bottom.size(), nullptr, 0);
    const int B = c.B, T = m->T, D = m->D;
    const bool concat = m->interaction == REC_INTERACT_CONCAT;
    // Without a Bottom-FC the dense part of the Predict-FC input is the dense input.
    const float *x0 = m->bottom.empty() ? c.dense : u.x0;
    const int x0_ld = m->bottom.empty() ? m->F : m->x0_ld;
    // S3 -> act[0], row stride z_ld, zero filled up to it
    if (concat) {
        if (!concat_rides_on_scan(m) && !plan.layer)
            REC_TRY(launch_concat_dense(x0, x0_ld, m->w0, B, u.act[0], m->z_width, m->z_ld, s));
    } else
        REC_TRY(launch_interact(x0, x0_ld, u.pooled, B, T, D, u.act[0], m->z_ld, s));
    REC_TRY(mark(ev, EV_INTERACT_END, s));
    // S4: the towers run side by side, their hidden activations in adjacent
    // column blocks of one row.  ReLU on all layers but the last.  The last layer
    // is one fp32 dot per sample and tower: folded into the epilogue of the layer
    // before it when that layer's block tile spans whole rows, else that layer
    // leaves fp32 for a dot kernel.
    const int G = m->towers, n_top = m->n_top;
    FcProblem p{};
    p.A = u.act[0]; p.a_f32 = false; p.lda = m->z_ld; p.a_stride = 0;
    p.M = B; p.relu = true; p.groups = G; p.num_cus = m->num_cus; p.corun = m->pipeline;
    for (int k = 0; k < G; ++k) {
        const Layer &dotl = m->top[(size_t)k * n_top + n_top - 1];
        p.g.dot_w[k] = static_cast<const float *>(dotl.W);
        p.g.dot_bias[k] = dotl.bias;
    }
    bool cur_f32 = false, done = false, first_marked = false;
    const Layer *layers = m->top.data();
    const int n = n_top - 1;  // layers ahead of the one-output layer
    int launches = 0;
    for (int i = 0; i < n && !done;) {
        const Layer &l = layers[i];  // shape of layer i in every tower
        const int j = chain_end(m, layers, i, n, G, B, false, true);
        if (j > i) {
            ChainProblem cp{};
            cp.A = p.A; cp.a_f32 = false; cp.lda = p.lda; cp.a_stride = p.a_stride; cp.M = B;
            chain_run(layers, n_top, G, i, j, m->num_cus, cp);
            if (j == n) {
                cp.out_mode = CHAIN_OUT_DOT;
                for (int k = 0; k < G; ++k) { cp.dot_w[k] = p.g.dot_w[k]; cp.dot_bias[k] = p.g.dot_bias[k]; }
                cp.dot_out = c.logits; cp.dot_ld = G;
                done = true;
            } else {
                cp.out_mode = CHAIN_OUT_BF16;
                cp.C = u.act[1 + (launches & 1)]; cp.ldc = G * layers[j - 1].Npad; cp.c_stride = layers[j - 1].Npad;
                p.A = cp.C; p.lda = cp.ldc; p.a_stride = cp.c_stride; p.a_f32 = false;
            }
            REC_TRY(launch_mlp_chain(cp, s, done ? take_report(c) : FaultReport{}));
            i = j;
        } else {
            for (int k = 0; k < G; ++k) {
                p.g.W[k] = m->top[(size_t)k * n_top + i].W;
                p.g.bias[k] = m->top[(size_t)k * n_top + i].bias;
                p.frag[k] = splits(m) ? m->top[(size_t)k * n_top + i].Wc : nullptr;
            }
            p.K = l.K; p.Kpad = l.Kpad; p.Npad = l.Npad;
            const bool feeds_dot = i + 1 == n;
            if (feeds_dot && fc_can_fuse_dot(l.Npad)) {
                p.C = nullptr; p.out_f32 = false; p.ldc = 0; p.c_stride = 0;
                p.dot_out = c.logits; p.dot_ld = G;
                p.report = take_report(c);
                REC_TRY(launch_fc(p, s));
                done = true;
            } else {
                p.C = u.act[1 + (launches & 1)]; p.out_f32 = feeds_dot; p.ldc = G * l.Npad; p.c_stride = l.Npad;
                REC_TRY(launch_fc(p, s));
                p.A = p.C; p.lda = p.ldc; p.a_stride = p.c_stride; p.a_f32 = false;
                cur_f32 = feeds_dot;
            }
            ++i;
        }
        ++launches;
        if (!first_marked) {  // the first launch (the widest layer, or the run it starts) is timed on its own
            REC_TRY(mark(ev, EV_TOP_FIRST_END, s));
            first_marked = true;
        }
    }
    if (!done)
        REC_TRY(launch_rowdot(p.A, cur_f32, p.lda, p.a_stride, B, m->top[n_top - 1].Kpad, p.g, G, c.logits, G, s));
    if (!first_marked) REC_TRY(mark(ev, EV_TOP_FIRST_END, s));
    return mark(ev, EV_END, s);
}

// The whole pass in order on one stream: S0, S1, S2, S3, S4.
hipError_t enqueue_in_order(const rec_model *m, const Bufs &u, const Call &c, const Plan &plan, bool use_hot,
                            hipStream_t s, hipEvent_t *ev)
{
    REC_TRY(mark(ev, EV_BEGIN, s));
    REC_TRY(enqueue_sparse(m, u, c, plan, use_hot, s, ev));
    if (plan.ride) {  // S2 ran inside S0's launch: its stages read zero
        REC_TRY(mark(ev, EV_BOTTOM_FIRST_END, s));
        REC_TRY(mark(ev, EV_BOTTOM_END, s));
    } else if (plan.tail_from < (int)m->bottom.size()) {
        const void *rest = nullptr;
        int rest_ld = 0;
        REC_TRY(enqueue_bottom(m, u, c, s, ev, plan.tail_from, plan.layer, &rest, &rest_ld));
        return enqueue_fused_tail(m, u, c, s, ev, plan.tail_from, rest, rest_ld);
    } else {
        REC_TRY(enqueue_bottom(m, u, c, s, ev, (int)m->bottom.size(), plan.layer, nullptr, nullptr));
    }
    return enqueue_tail(m, u, c, plan, s, ev);
}

// Device address of `scratch` on each GPU, looked up once per device with that
// device current.
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
char *g_scratch_ptr[MAX_DEVICES] = {};

rec_status static_scratch(char **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return REC_ERR_DEVICE;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return REC_ERR_DEVICE;
        if (fc_big_prepare() != hipSuccess || fc_split_prepare() != hipSuccess || chain_prepare() != hipSuccess || scan_prepare() != hipSuccess ||
            tail_prepare() != hipSuccess || front_prepare() != hipSuccess)
            return REC_ERR_DEVICE;
        g_scratch_ptr[dev] = static_cast<char *>(p);
    }
    *out = g_scratch_ptr[dev];
    return REC_OK;
}

// Table descriptors by value: what rec_forward_static() writes into its scratch
// at the start of every call.
struct StaticTables {
    const void *base[REC_STATIC_MAX_TABLES];
    long long rows[REC_STATIC_MAX_TABLES];
};

__global__ __launch_bounds__(256) void static_begin_kernel(const StaticTables st, int T, TableDesc *dst,
                                                           ErrRecord *err, unsigned long long *tile_words, int tiles)
{
    const int t = threadIdx.x;
    for (int i = t; i < tiles; i += 256) tile_words[i] = 0;
    if (t < T) {
        dst[t].base = st.base[t];
        dst[t].rows = st.rows[t];
        dst[t].hot_ids = nullptr;
        dst[t].n_hot = 0;
        dst[t].pad = 0;
    }
    if (t == 0) {
        err->first_bad_len = ~0ull;
        err->first_bad_idx = ~0ull;
        err->flags = 0u;
    }
}

__global__ __launch_bounds__(64) void static_end_kernel(const ErrRecord *err, long long *fault)
{
    report_fault(err, fault);
}

// Host-checkable faults of a forward call.
rec_status check_call(const rec_model *m, const float *dev_dense, const int32_t *dev_indices,
                      const int32_t *dev_lengths, int32_t batch, int64_t nnz, const float *dev_logits)
{
    if (!m) return REC_ERR_ARG;
    if (batch < 0 || batch > m->max_batch || nnz < 0 || nnz > m->max_nnz) return REC_ERR_ARG;
    if (!m->ws || !all_loaded(m)) return REC_ERR_STATE;
    if (batch == 0) return REC_OK;
    if (!dev_dense || !dev_lengths || !dev_logits || (nnz > 0 && !dev_indices)) return REC_ERR_ARG;
    return REC_OK;
}

}  // namespace

extern "C" {

const char *rec_status_string(int status)
{
    // An int, not the enum: a caller may pass a number that is no enumerator, and
    // reading such a value through the enum type is undefined in C++.
    switch (status) {
    case REC_OK: return "ok";
    case REC_ERR_ARG: return "bad argument";
    case REC_ERR_SHAPE: return "layer widths or embedding size do not fit the model";
    case REC_ERR_STATE: return "call made before what it depends on";
    case REC_ERR_LENGTHS: return "negative length or sum(lengths) != nnz";
    case REC_ERR_INDEX_RANGE: return "row id outside its table";
    case REC_ERR_OVERFLOW: return "count exceeds 32-bit index range";
    case REC_ERR_DEVICE: return "HIP call failed";
    case REC_ERR_CAPACITY: return "call needs more scratch than the static array holds";
    }
    return "unknown status";
}

rec_status rec_create(const rec_config *cfg, rec_model **out)
{
    if (!out) return REC_ERR_ARG;
    *out = nullptr;
    if (!cfg || !cfg->rows || !cfg->bottom_widths || !cfg->top_widths) return REC_ERR_ARG;
    if (cfg->num_tables <= 0 || cfg->emb_dim <= 0 || cfg->num_dense <= 0 || cfg->n_bottom < 0 ||
        cfg->n_top <= 0 || cfg->max_batch <= 0 || cfg->max_nnz < 0)
        return REC_ERR_ARG;
    if (cfg->table_dtype != REC_F32 && cfg->table_dtype != REC_F16) return REC_ERR_ARG;
    if (cfg->interaction != REC_INTERACT_DOT && cfg->interaction != REC_INTERACT_CONCAT) return REC_ERR_ARG;
    if (cfg->num_towers < 0 || cfg->num_towers > REC_MAX_TOWERS) return REC_ERR_ARG;
    const int towers = cfg->num_towers > 0 ? cfg->num_towers : 1;
    const bool concat = cfg->interaction == REC_INTERACT_CONCAT;

    const int T = cfg->num_tables, D = cfg->emb_dim;
    // A row must be 16 * 2^k bytes (k = 0..6) for the 128-bit gather.
    const long long rowbytes = (long long)D * (cfg->table_dtype == REC_F16 ? 2 : 4);
    if (rowbytes % 16 != 0) return REC_ERR_SHAPE;
    const long long lpr = rowbytes / 16;
    if (lpr > 64 || (lpr & (lpr - 1)) != 0) return REC_ERR_SHAPE;

    for (int t = 0; t < T; ++t) {
        if (cfg->rows[t] <= 0) return REC_ERR_ARG;
        if (cfg->rows[t] >= (1ll << 31)) return REC_ERR_OVERFLOW;
    }
    if (cfg->max_nnz >= (1ll << 31)) return REC_ERR_OVERFLOW;
    if ((long long)T * cfg->max_batch >= (1ll << 31)) return REC_ERR_OVERFLOW;

    for (int i = 0; i <= cfg->n_bottom; ++i)
        if (cfg->bottom_widths[i] <= 0 || cfg->bottom_widths[i] >= (1 << 24)) return REC_ERR_SHAPE;
    for (int i = 0; i <= cfg->n_top; ++i)
        if (cfg->top_widths[i] <= 0 || cfg->top_widths[i] >= (1 << 24)) return REC_ERR_SHAPE;
    const int w0 = cfg->bottom_widths[cfg->n_bottom];
    const long long width = concat ? w0 + (long long)T * D : D + (long long)T * (T + 1) / 2;
    if (width >= (1ll << 24)) return REC_ERR_OVERFLOW;
    if (cfg->bottom_widths[0] != cfg->num_dense || (!concat && w0 != D)) return REC_ERR_SHAPE;
    if (cfg->top_widths[0] != width || cfg->top_widths[cfg->n_top] != 1) return REC_ERR_SHAPE;
    if (!concat && interact_lds_bytes_per_sample(T, D) > 64 * 1024) return REC_ERR_SHAPE;

    rec_model *m = new (std::nothrow) rec_model();
    if (!m) return REC_ERR_ARG;
    m->T = T; m->D = D; m->F = cfg->num_dense; m->dtype = cfg->table_dtype;
    m->interaction = cfg->interaction; m->towers = towers; m->n_top = cfg->n_top;
    m->w0 = w0; m->z_width = (int)width;
    m->max_batch = cfg->max_batch; m->max_nnz = cfg->max_nnz;
    m->rows.assign(cfg->rows, cfg->rows + T);
    for (int t = 0; t < T; ++t) m->max_rows = std::max<long long>(m->max_rows, cfg->rows[t]);
    m->table_loaded.assign(T, 0);
    m->desc.assign(T, TableDesc{nullptr, 0, nullptr, 0, 0});
    for (int t = 0; t < T; ++t) m->desc[t].rows = cfg->rows[t];
    m->x0_ld = pad_up(w0);
    m->z_ld = pad_up((int)width);
    m->act_ld = PAD;
    // Hidden activations of the towers sit side by side in one row.
    auto fill = [&](Layer *v, const int32_t *w, int n, int side_by_side) {
        for (int i = 0; i < n; ++i) {
            v[i].K = w[i]; v[i].N = w[i + 1];
            v[i].Kpad = pad_up(w[i]); v[i].Npad = pad_up(w[i + 1]);
            v[i].chain = chain_layer_fits(v[i].Kpad, v[i].Npad);
            if (i + 1 < n || side_by_side == 1)  // the one-output layer leaves no activation row
                m->act_ld = std::max(m->act_ld, side_by_side * v[i].Npad);
        }
    };
    m->bottom.resize(cfg->n_bottom);
    fill(m->bottom.data(), cfg->bottom_widths, cfg->n_bottom, 1);
    m->top.resize((size_t)towers * cfg->n_top);
    for (int k = 0; k < towers; ++k) {
        fill(&m->top[(size_t)k * cfg->n_top], cfg->top_widths, cfg->n_top, towers);
        m->top[(size_t)k * cfg->n_top + cfg->n_top - 1].dot = true;
        m->top[(size_t)k * cfg->n_top + cfg->n_top - 1].chain = false;
    }
    m->act_row_bytes = 2 * (size_t)m->act_ld;
    if (cfg->n_top > 1)  // the layer feeding the dot leaves fp32
        m->act_row_bytes = std::max(m->act_row_bytes, sizeof(float) * towers * m->top[cfg->n_top - 2].Npad);

    m->lay = carve(m, m->max_batch, 1);
    *out = m;
    return REC_OK;
}

void rec_destroy(rec_model *m)
{
    if (!m) return;
    for (hipEvent_t e : m->ev)
        if (e) (void)hipEventDestroy(e);
    if (m->ev_fork) (void)hipEventDestroy(m->ev_fork);
    if (m->ev_join) (void)hipEventDestroy(m->ev_join);
    for (int k = 0; k < MAX_FRAMES; ++k)
        for (hipEvent_t e : {m->ev_scan[k], m->ev_pool[k], m->ev_tail[k], m->ev_bottom[k]})
            if (e) (void)hipEventDestroy(e);
    for (hipStream_t o : m->own_stream)
        if (o) (void)hipStreamDestroy(o);
    if (m->side) (void)hipStreamDestroy(m->side);
    delete m;
}

size_t rec_workspace_bytes(const rec_model *m) { return m ? m->lay.bytes : 0; }

rec_status rec_bind_workspace(rec_model *m, void *dev_ptr, size_t bytes, void *stream)
{
    if (!m || !dev_ptr) return REC_ERR_ARG;
    if (bytes < m->lay.bytes || reinterpret_cast<uintptr_t>(dev_ptr) % ALIGN != 0) return REC_ERR_ARG;
    if (!m->side) {
        // Default priority; the two events only order work, they carry no timing.
        if (hipStreamCreateWithFlags(&m->side, hipStreamNonBlocking) != hipSuccess ||
            hipEventCreateWithFlags(&m->ev_fork, hipEventDisableTiming) != hipSuccess ||
            hipEventCreateWithFlags(&m->ev_join, hipEventDisableTiming) != hipSuccess)
            return REC_ERR_DEVICE;
        for (int k = 0; k < MAX_FRAMES; ++k)
            if (hipEventCreateWithFlags(&m->ev_scan[k], hipEventDisableTiming) != hipSuccess ||
                hipEventCreateWithFlags(&m->ev_pool[k], hipEventDisableTiming) != hipSuccess ||
                hipEventCreateWithFlags(&m->ev_tail[k], hipEventDisableTiming) != hipSuccess ||
                hipEventCreateWithFlags(&m->ev_bottom[k], hipEventDisableTiming) != hipSuccess)
                return REC_ERR_DEVICE;
    }
    if (m->pipeline)
        for (hipStream_t &o : m->own_stream)
            if (!o && hipStreamCreateWithFlags(&o, hipStreamNonBlocking) != hipSuccess) return REC_ERR_DEVICE;
    for (bool &b : m->tail_pending) b = false;
    m->next_frame = m->last_frame = 0;
    m->pool_turn = 0;
    {   // set-up is also where the kernels are granted their LDS and the static scratch
        // of this device is looked up, once per device
        char *unused = nullptr;
        if (static_scratch(&unused) != REC_OK) return REC_ERR_DEVICE;
    }
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0)
        m->num_cus = cus;
    m->ws = static_cast<char *>(dev_ptr);
    // The descriptors live in the workspace: tables and hot lists are to be registered again.
    std::fill(m->table_loaded.begin(), m->table_loaded.end(), 0);
    for (TableDesc &d : m->desc) { d.base = nullptr; d.hot_ids = nullptr; d.n_hot = 0; }
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (launch_clear_err(m->at<ErrRecord>(m->lay.off_err), s) != hipSuccess) return REC_ERR_DEVICE;
    for (int f = 0; f < (m->pipeline ? MAX_FRAMES : 1); ++f) {
        const Bufs u = bufs_at(m->ws, m->lay, f);
        if (launch_clear_tile_words(u.tile_words, most_tiles(m), s) != hipSuccess) return REC_ERR_DEVICE;
        m->words_left[f] = false;
    }
    if (hipStreamSynchronize(s) != hipSuccess) return REC_ERR_DEVICE;
    return REC_OK;
}

rec_status rec_load_tables(rec_model *m, int32_t table, const void *dev_rows)
{
    if (!m || !dev_rows || table < 0 || table >= m->T) return REC_ERR_ARG;
    if (reinterpret_cast<uintptr_t>(dev_rows) % 16 != 0) return REC_ERR_ARG;
    if (!m->ws) return REC_ERR_STATE;
    m->desc[table].base = dev_rows;
    if (hipMemcpy(m->at<TableDesc>(m->lay.off_tables) + table, &m->desc[table], sizeof(TableDesc),
                  hipMemcpyHostToDevice) != hipSuccess)
        return REC_ERR_DEVICE;
    m->table_loaded[table] = 1;
    return REC_OK;
}

rec_status rec_load_hot_rows(rec_model *m, int32_t table, const int32_t *dev_ids, int32_t n)
{
    if (!m || table < 0 || table >= m->T || n < 0 || n > REC_MAX_HOT_ROWS || (n > 0 && !dev_ids))
        return REC_ERR_ARG;
    if (!m->ws) return REC_ERR_STATE;
    int hcap = 16;
    while (hcap < n) hcap *= 2;
    const int rowbytes = m->D * (m->dtype == REC_F16 ? 2 : 4);
    if (n > 0 && !pool_hot_fits(hcap, rowbytes)) return REC_ERR_ARG;
    m->desc[table].hot_ids = n > 0 ? dev_ids : nullptr;
    m->desc[table].n_hot = n;
    if (hipMemcpy(m->at<TableDesc>(m->lay.off_tables) + table, &m->desc[table], sizeof(TableDesc),
                  hipMemcpyHostToDevice) != hipSuccess)
        return REC_ERR_DEVICE;
    return REC_OK;
}

size_t rec_mlp_packed_bytes(const rec_model *m, int32_t which, int32_t layer)
{
    if (!m) return 0;
    const Layer *l = find_layer(const_cast<rec_model *>(m), which, layer);
    if (!l) return 0;
    return align_up(l->w_bytes()) + align_up(sizeof(float) * l->Npad) + align_up(l->chain_bytes());
}

rec_status rec_load_mlp(rec_model *m, int32_t which, int32_t layer, const float *dev_W,
                        const float *dev_b, void *dev_packed, void *stream)
{
    if (!m || !dev_W || !dev_b || !dev_packed) return REC_ERR_ARG;
    Layer *l = find_layer(m, which, layer);
    if (!l) return REC_ERR_ARG;
    if (reinterpret_cast<uintptr_t>(dev_packed) % ALIGN != 0) return REC_ERR_ARG;
    char *p = static_cast<char *>(dev_packed);
    float *bias = reinterpret_cast<float *>(p + align_up(l->w_bytes()));
    hipStream_t s = static_cast<hipStream_t>(stream);
    const hipError_t e = l->dot ? launch_pack_dot(dev_W, dev_b, l->K, l->Kpad, reinterpret_cast<float *>(p), bias, s)
                                : launch_pack_fc(dev_W, dev_b, l->N, l->K, l->Npad, l->Kpad, p, bias, s);
    if (e != hipSuccess) return REC_ERR_DEVICE;
    if (!l->dot) {
        char *pc = p + align_up(l->w_bytes()) + align_up(sizeof(float) * l->Npad);
        if (launch_pack_chain(dev_W, l->N, l->K, l->Npad, l->Kpad, pc, s) != hipSuccess) return REC_ERR_DEVICE;
        l->Wc = pc;
    }
    l->W = p;
    l->bias = bias;
    l->loaded = true;
    return REC_OK;
}

rec_status rec_forward(rec_model *m, const float *dev_dense, const int32_t *dev_indices,
                       const int32_t *dev_lengths, int32_t batch, int64_t nnz, float *dev_logits,
                       void *stream)
{
    const rec_status st = check_call(m, dev_dense, dev_indices, dev_lengths, batch, nnz, dev_logits);
    if (st != REC_OK || batch == 0) return st;

    hipStream_t s = static_cast<hipStream_t>(stream);
    const Call c{dev_dense, dev_indices, dev_lengths, batch, nnz, dev_logits, nullptr};
    // Forward number i is timed when i is a multiple of the period; it is the
    // (i / period)-th timed one.
    const bool prof = m->slots > 0 && m->forwards % m->period == 0;
    const size_t slot = prof ? (size_t)((m->forwards / m->period) % m->slots) : 0;
    hipEvent_t *ev = prof ? &m->ev[slot * EV_PER_SLOT] : nullptr;
    const int frame = m->pipeline ? m->next_frame : 0;
    const Bufs u = bufs_at(m->ws, m->lay, frame);
    const Plan plan = plan_of(m, u, c, true, prof);
#define REC_DEV(call)                                  \
    do {                                               \
        if ((call) != hipSuccess) return REC_ERR_DEVICE; \
    } while (0)

    if (m->pipeline) {
        // Four queues (Sec. IV-A, S-D pipeline; dependencies of Sec. III-A): scan
        // (S0) and Bottom-FC (S2) on the caller's stream, pooling (S1) on two
        // streams in turn, interaction and Predict-FC (S3, S4) on a fourth.  Two
        // pooling launches are in flight at any time, so neither the packets between
        // launches nor the ramps of a launch leave the memory system idle; a batch
        // owns one of four frames until its logits are written.
        const int k = frame;
        hipStream_t p = m->pool_stream[m->pool_turn] ? m->pool_stream[m->pool_turn] : m->own_stream[m->pool_turn];
        hipStream_t d = m->dense_stream ? m->dense_stream : m->side;
        if (m->tail_pending[k]) {  // the batch that used this frame four calls ago
            REC_DEV(hipStreamWaitEvent(s, m->ev_tail[k], 0));
            m->tail_pending[k] = false;
        }
        if (m->words_left[k]) REC_DEV(launch_clear_tile_words(u.tile_words, most_tiles(m), s));
        m->words_left[k] = true;
        REC_DEV(mark(ev, EV_BEGIN, s));
        REC_DEV(enqueue_scan(m, u, c, Plan{}, s));
        REC_DEV(mark(ev, EV_SCAN_END, s));
        REC_DEV(hipEventRecord(m->ev_scan[k], s));
        REC_DEV(hipStreamWaitEvent(p, m->ev_scan[k], 0));
        REC_DEV(mark(ev, EV_POOL_BEGIN, p));
        REC_DEV(enqueue_pool(m, u, c, true, p, false));
        REC_DEV(mark(ev, EV_POOL_END, p));
        REC_DEV(hipEventRecord(m->ev_pool[k], p));
        if (!m->bottom.empty()) {
            REC_DEV(mark(ev, EV_BOTTOM_BEGIN, s));
            REC_DEV(enqueue_bottom(m, u, c, s, ev));
        }
        REC_DEV(hipEventRecord(m->ev_bottom[k], s));
        REC_DEV(hipStreamWaitEvent(d, m->ev_bottom[k], 0));
        REC_DEV(hipStreamWaitEvent(d, m->ev_pool[k], 0));
        REC_DEV(mark(ev, EV_INTERACT_BEGIN, d));
        REC_DEV(enqueue_tail(m, u, c, plan, d, ev));
        REC_DEV(hipEventRecord(m->ev_tail[k], d));
        m->tail_pending[k] = true;
        m->last_frame = k;
        m->next_frame = (k + 1) % MAX_FRAMES;
        m->pool_turn ^= 1;
        if (prof) m->slot_mode[slot] = 1;
    } else {
        m->last_frame = 0;
        if (m->words_left[0]) REC_DEV(launch_clear_tile_words(u.tile_words, most_tiles(m), s));
        m->words_left[0] = true;
        // S2 does not depend on S0/S1: with overlap it is enqueued on the side
        // stream, forked from and joined back into the caller's stream.
        if (m->overlap_dense && !m->bottom.empty()) {
            REC_DEV(mark(ev, EV_BEGIN, s));
            REC_DEV(hipEventRecord(m->ev_fork, s));
            REC_DEV(hipStreamWaitEvent(m->side, m->ev_fork, 0));
            REC_DEV(enqueue_bottom(m, u, c, m->side, nullptr));
            REC_DEV(hipEventRecord(m->ev_join, m->side));
            REC_DEV(enqueue_sparse(m, u, c, plan, true, s, ev));
            // the "bottom" stage then times only what pooling did not hide
            REC_DEV(hipStreamWaitEvent(s, m->ev_join, 0));
            REC_DEV(mark(ev, EV_BOTTOM_FIRST_END, s));
            REC_DEV(mark(ev, EV_BOTTOM_END, s));
            REC_DEV(enqueue_tail(m, u, c, plan, s, ev));
        } else {
            REC_DEV(enqueue_in_order(m, u, c, plan, true, s, ev));
        }
        if (prof) m->slot_mode[slot] = plan.ride ? 2 : 0;
    }
#undef REC_DEV
    m->words_left[frame] = false;
    if (prof) m->slot_shared[slot] = shared_stages(m, plan, batch);
    if (m->slots > 0) ++m->forwards;
    return REC_OK;
}

rec_status rec_forward_static(rec_model *m, const float *dev_dense, const int32_t *dev_indices,
                              const int32_t *dev_lengths, int32_t batch, int64_t nnz, float *dev_logits,
                              int64_t *dev_fault, void *stream)
{
    const rec_status st = check_call(m, dev_dense, dev_indices, dev_lengths, batch, nnz, dev_logits);
    if (st != REC_OK) return st;
    if (m->T > REC_STATIC_MAX_TABLES) return REC_ERR_CAPACITY;
    const Carve lay = carve(m, batch > 0 ? batch : 1, 1);
    if (lay.bytes > REC_STATIC_SCRATCH_BYTES) return REC_ERR_CAPACITY;
    char *base = nullptr;
    const rec_status sp = static_scratch(&base);
    if (sp != REC_OK) return sp;

    hipStream_t s = static_cast<hipStream_t>(stream);
    const Bufs u = bufs_at(base, lay, 0);
    // The array keeps what the last call left: descriptors and error record are
    // written afresh; every other part is fully overwritten before it is read.
    StaticTables tabs{};
    for (int t = 0; t < m->T; ++t) {
        tabs.base[t] = m->desc[t].base;
        tabs.rows[t] = m->desc[t].rows;
    }
    hipLaunchKernelGGL(static_begin_kernel, dim3(1), dim3(256), 0, s, tabs, m->T, const_cast<TableDesc *>(u.tables),
                       u.err, u.tile_words, (int)(((size_t)m->T * batch + SCAN_TILE - 1) / SCAN_TILE));
    if (hipGetLastError() != hipSuccess) return REC_ERR_DEVICE;
    FaultReport report{u.err, reinterpret_cast<long long *>(dev_fault)};
    if (batch > 0) {
        const Call c{dev_dense, dev_indices, dev_lengths, batch, nnz, dev_logits, &report};
        if (enqueue_in_order(m, u, c, plan_of(m, u, c, false, false), false, s, nullptr) != hipSuccess) return REC_ERR_DEVICE;
    }
    if (report.fault) {  // no launch took it
        hipLaunchKernelGGL(static_end_kernel, dim3(1), dim3(64), 0, s, report.err, report.fault);
        if (hipGetLastError() != hipSuccess) return REC_ERR_DEVICE;
    }
    return REC_OK;
}

rec_status rec_drain(rec_model *m, void *stream)
{
    if (!m) return REC_ERR_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    // Every batch's last stage runs on the one dense stream, in order: the event
    // of the latest call stands for all of them.
    if (m->tail_pending[m->last_frame] &&
        hipStreamWaitEvent(s, m->ev_tail[m->last_frame], 0) != hipSuccess)
        return REC_ERR_DEVICE;
    for (bool &p : m->tail_pending) p = false;
    return REC_OK;
}

rec_status rec_check(rec_model *m, void *stream, int64_t *first_bad_pos)
{
    if (!m) return REC_ERR_ARG;
    if (!m->ws) return REC_ERR_STATE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    ErrRecord h;
    ErrRecord *d = m->at<ErrRecord>(m->lay.off_err);
    if (rec_drain(m, stream) != REC_OK) return REC_ERR_DEVICE;
    if (hipStreamSynchronize(s) != hipSuccess) return REC_ERR_DEVICE;
    if (hipMemcpy(&h, d, sizeof(h), hipMemcpyDeviceToHost) != hipSuccess) return REC_ERR_DEVICE;
    if (first_bad_pos) *first_bad_pos = -1;
    if (h.flags == 0) return REC_OK;
    if (launch_clear_err(d, s) != hipSuccess) return REC_ERR_DEVICE;
    if (hipStreamSynchronize(s) != hipSuccess) return REC_ERR_DEVICE;
    if (h.flags & (ERR_NEG_LENGTH | ERR_TOTAL_MISMATCH)) {
        if (first_bad_pos && (h.flags & ERR_NEG_LENGTH)) *first_bad_pos = (int64_t)h.first_bad_len;
        return REC_ERR_LENGTHS;
    }
    if (first_bad_pos) *first_bad_pos = (int64_t)h.first_bad_idx;
    return REC_ERR_INDEX_RANGE;
}

rec_status rec_debug_get(rec_model *m, int32_t what, const void **dev_ptr, int64_t *ld_out)
{
    if (!m || !dev_ptr) return REC_ERR_ARG;
    if (!m->ws) return REC_ERR_STATE;
    int64_t ld = 0;
    const Frame &f = m->lay.fr[m->last_frame];
    switch (what) {
    case REC_DBG_OFFSETS: *dev_ptr = m->at<void>(f.off_offsets); ld = 0; break;
    case REC_DBG_POOLED:
        if (m->interaction != REC_INTERACT_DOT) return REC_ERR_STATE;
        *dev_ptr = m->at<void>(f.off_pooled); ld = m->D; break;
    case REC_DBG_BOTTOM_OUT:
        if (m->bottom.empty()) return REC_ERR_STATE;
        *dev_ptr = m->at<void>(f.off_x0); ld = m->x0_ld; break;
    case REC_DBG_INTERACT: *dev_ptr = m->at<void>(f.off_act[0]); ld = m->z_ld; break;
    default: return REC_ERR_ARG;
    }
    if (ld_out) *ld_out = ld;
    return REC_OK;
}

rec_status rec_set_option(rec_model *m, int32_t option, int32_t value)
{
    if (!m) return REC_ERR_ARG;
    switch (option) {
    case REC_OPT_OVERLAP_DENSE: m->overlap_dense = value != 0; return REC_OK;
    case REC_OPT_STREAM_ROWS: m->stream_rows = value != 0; return REC_OK;
    case REC_OPT_FUSE_MLP:
        if (value < 0 || value > 2) return REC_ERR_ARG;
        m->fuse_mlp = value;
        return REC_OK;
    case REC_OPT_PIPELINE:
        // Decides the size of the workspace: only while none is bound.
        if (m->ws) return REC_ERR_STATE;
        m->pipeline = value != 0;
        m->lay = carve(m, m->max_batch, m->pipeline ? MAX_FRAMES : 1);
        return REC_OK;
    default: return REC_ERR_ARG;
    }
}

rec_status rec_set_dense_stream(rec_model *m, void *stream)
{
    if (!m) return REC_ERR_ARG;
    for (int k = 0; k < MAX_FRAMES; ++k)
        if (m->tail_pending[k]) return REC_ERR_STATE;  // work is still ordered on the old one
    m->dense_stream = static_cast<hipStream_t>(stream);
    return REC_OK;
}

rec_status rec_set_pool_streams(rec_model *m, void *stream_a, void *stream_b)
{
    if (!m) return REC_ERR_ARG;
    for (int k = 0; k < MAX_FRAMES; ++k)
        if (m->tail_pending[k]) return REC_ERR_STATE;
    m->pool_stream[0] = static_cast<hipStream_t>(stream_a);
    m->pool_stream[1] = static_cast<hipStream_t>(stream_b);
    return REC_OK;
}

rec_status rec_set_profiling(rec_model *m, int32_t slots, int32_t period)
{
    if (!m || slots < 0 || slots > 65536 || (slots > 0 && period < 1)) return REC_ERR_ARG;
    for (hipEvent_t e : m->ev)
        if (e) (void)hipEventDestroy(e);
    m->ev.assign((size_t)slots * EV_PER_SLOT, nullptr);
    m->slot_mode.assign((size_t)slots, 0);
    m->slot_shared.assign((size_t)slots, 0);
    m->slots = 0;
    m->forwards = 0;
    for (hipEvent_t &e : m->ev)
        if (hipEventCreate(&e) != hipSuccess) return REC_ERR_DEVICE;
    m->slots = slots;
    m->period = slots > 0 ? period : 1;
    return REC_OK;
}

rec_status rec_stage_ms(rec_model *m, int32_t slot, float *ms)
{
    if (!m || !ms) return REC_ERR_ARG;
    const long long timed = (m->forwards + m->period - 1) / m->period;  // timed forwards so far
    if (m->slots <= 0 || slot < 0 || slot >= m->slots || slot >= timed) return REC_ERR_STATE;
    hipEvent_t *ev = &m->ev[(size_t)slot * EV_PER_SLOT];
    // Stage i ran between events begin[i] and end[i]; in a pipelined forward the
    // dense stages sit on another stream and have begin events of their own.
    static const int end[REC_NUM_STAGES] = {EV_SCAN_END, EV_POOL_END, EV_BOTTOM_FIRST_END, EV_BOTTOM_END,
                                            EV_INTERACT_END, EV_TOP_FIRST_END, EV_END};
    static const int begin_in_order[REC_NUM_STAGES] = {EV_BEGIN, EV_SCAN_END, EV_POOL_END, EV_BOTTOM_FIRST_END,
                                                       EV_BOTTOM_END, EV_INTERACT_END, EV_TOP_FIRST_END};
    static const int begin_pipelined[REC_NUM_STAGES] = {EV_BEGIN, EV_POOL_BEGIN, EV_BOTTOM_BEGIN,
                                                        EV_BOTTOM_FIRST_END, EV_INTERACT_BEGIN,
                                                        EV_INTERACT_END, EV_TOP_FIRST_END};
    const int *begin = m->slot_mode[slot] == 1 ? begin_pipelined : begin_in_order;
    if (hipEventSynchronize(ev[EV_END]) != hipSuccess) return REC_ERR_DEVICE;
    for (int i = 0; i < REC_NUM_STAGES; ++i) {
        ms[i] = 0.0f;
        const bool bottom_stage = i == REC_STAGE_BOTTOM_FIRST || i == REC_STAGE_BOTTOM_REST;
        if (bottom_stage && ((m->slot_mode[slot] == 1 && m->bottom.empty()) || m->slot_mode[slot] == 2))
            continue;  // no launch of its own: nothing to time
        if (hipEventElapsedTime(&ms[i], ev[begin[i]], ev[end[i]]) != hipSuccess) return REC_ERR_DEVICE;
    }
    return REC_OK;
}

rec_status rec_stage_shared(const rec_model *m, int32_t slot, uint32_t *mask)
{
    if (!m || !mask) return REC_ERR_ARG;
    const long long timed = (m->forwards + m->period - 1) / m->period;
    if (m->slots <= 0 || slot < 0 || slot >= m->slots || slot >= timed) return REC_ERR_STATE;
    *mask = m->slot_shared[slot];
    return REC_OK;
}

static rec_status probe_plan(const rec_model *m, int32_t batch, int64_t nnz, Plan *p)
{
    if (!m || batch < 1 || batch > m->max_batch || nnz < 0 || nnz > m->max_nnz) return REC_ERR_ARG;
    alignas(16) float some[4] = {};  // nothing follows these pointers
    try {
        rec_model loaded = *m;
        for (std::vector<Layer> *stack : {&loaded.bottom, &loaded.top})
            for (Layer &l : *stack) l.Wc = some;
        Bufs u{};
        u.x0 = some;
        for (void *&a : u.act) a = some;
        const Call c{some, nullptr, nullptr, batch, nnz, some, nullptr};
        *p = plan_of(&loaded, u, c, true, false);
    } catch (const std::bad_alloc &) {
        return REC_ERR_STATE;
    }
    return REC_OK;
}

rec_status rec_probe_plan(const rec_model *m, int32_t batch, int64_t nnz, uint32_t *mask, int32_t *tail_from)
{
    if (!mask || !tail_from) return REC_ERR_ARG;
    Plan p;
    const rec_status st = probe_plan(m, batch, nnz, &p);
    if (st != REC_OK) return st;
    *mask = (p.ride ? REC_PLAN_RIDE : 0) | (p.front ? REC_PLAN_FRONT : 0) | (p.layer ? REC_PLAN_LAYER : 0) |
            (p.tail ? REC_PLAN_TAIL : 0);
    *tail_from = p.tail_from;
    return REC_OK;
}

rec_status rec_probe_plan_pooling(const rec_model *m, int32_t batch, int64_t nnz, int32_t *form)
{
    if (!form) return REC_ERR_ARG;
    Plan p;
    const rec_status st = probe_plan(m, batch, nnz, &p);
    if (st != REC_OK) return st;
    const long long bags = (long long)m->T * batch;
    const int rowbytes = m->D * (m->dtype == REC_F16 ? 2 : 4);
    const bool concat = m->interaction == REC_INTERACT_CONCAT;
    if (p.joined)
        *form = REC_POOL_BESIDE_WIDE;
    else if (p.front && concat)
        *form = bags > SHORT_FORM_BAGS ? REC_POOL_MANY_LOOKUPS : REC_POOL_FEW_LOOKUPS;
    else if (p.front)
        *form = p.ride && front_takes_light(bags, nnz, rowbytes, m->bottom[0].Kpad, m->num_cus) ? REC_POOL_FRONT_LIGHT : REC_POOL_FRONT;
    else if (longest_hot_list(m, true) > 0 && !concat)
        *form = REC_POOL_HOT;
    else if (pool_short_applies(rowbytes, nnz, bags))
        *form = REC_POOL_SHORT;
    else
        *form = !concat && pool_two_applies(rowbytes, nnz, bags, pool_narrow(m->max_rows, rowbytes), m->num_cus) ? REC_POOL_TWO : REC_POOL_BAG;
    return REC_OK;
}

rec_status rec_probe_plan_joined(const rec_model *m, int32_t batch, int64_t nnz, int32_t *joined)
{
    if (!joined) return REC_ERR_ARG;
    Plan p;
    const rec_status st = probe_plan(m, batch, nnz, &p);
    if (st == REC_OK) *joined = p.joined ? 1 : 0;
    return st;
}

}  // extern "C"
