/*
 * rec_probe.h - helpers for measurements and tests.  Not part of the forward pass.
 *
 * What the matrix cores of this device sustain:
 * The published bf16 matrix rate of the chip (the MLP roofline of this build)
 * assumes every compute unit issuing matrix instructions at the top clock.
 * Whether a device sustains that depends on the operand values: with all compute
 * units busy the chip is power-limited, and bit patterns that toggle more of the
 * multiplier array lower the rate it settles at.  rec_probe_mfma() runs nothing
 * but v_mfma_f32_32x32x16_bf16 on register operands, so that a benchmark can
 * put the rate the hardware reaches on constant and on random operands beside
 * the published peak and beside its own GEMMs.
 *
 * The offsets scan by itself, with the bound on its waits in the caller's hand.
 *
 * Which kernel a layer's launch takes, and which stages of a forward share a launch
 * (host code, no device).
 */
#ifndef REC_PROBE_H
#define REC_PROBE_H

#include <stdint.h>
#include "rec.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Enqueues on `stream` one launch of `blocks` workgroups of 8 wavefronts; every
 * wavefront issues iters * 32 matrix instructions (32 x 32 x 16, bf16 in, fp32
 * accumulate, 8 independent accumulator tiles): 2 * 32 * 32 * 16 flops each,
 * blocks * 8 * iters * 32 * 32768 flops per launch.  random_operands = 0: every
 * operand element is 1.0; otherwise pseudo-random values in [-1, 1), different
 * per lane and changed every iteration by a sign flip of one operand.
 * dev_sink (device float[1]) receives a checksum.
 * REC_ERR_ARG on null sink or non-positive counts (blocks <= 65536, iters <= 2^20). */
REC_API rec_status rec_probe_mfma(int32_t random_operands, int32_t blocks, int32_t iters,
                          float *dev_sink, void *stream);

/* Most polls rec_probe_scan() takes, and what rec_forward() uses. */
#define REC_SCAN_POLLS 65536

/* Enqueues the scan of one forward pass alone: dev_offsets (int32 [n + 1]) from
 * dev_lengths (int32 [n]) as rec_forward() computes them.  A block of the scan
 * covers 2048 lengths, publishes their sum in a word of dev_words (uint64
 * [ceil(n / 2048)], zero on entry; the last word is not touched) and reads the
 * words of earlier blocks, at most `polls` times each before it adds up those
 * lengths itself.  The published words are left in place (in a forward pass the
 * pooling launch clears them).  dev_err: 64 bytes, 8-byte aligned, of scratch.
 * REC_ERR_ARG on a null pointer, n < 1, nnz < 0 or >= 2^31, polls outside
 * [0, REC_SCAN_POLLS]. */
REC_API rec_status rec_probe_scan(const int32_t *dev_lengths, int32_t n, int64_t nnz, int32_t *dev_offsets,
                          uint64_t *dev_words, int32_t polls, void *dev_err, void *stream);

/* What rec_probe_fc_form() asks about (bits of `flags`) ... */
enum {
    REC_FC_F32_ROWS = 1,       /* the dense input: fp32 rows, 16-byte aligned */
    REC_FC_DOT = 2,            /* the one-output layer folded into the launch */
    REC_FC_BESIDE_POOLING = 4, /* a pipelined model's */
    REC_FC_ANY_ORDER = 8       /* sums over k in any order: REC_OPT_FUSE_MLP 1 (beside pooling never) */
};
/* ... and form[0] of its answer: k-tile by k-tile; in tiles of 128 columns and more; the
 * k of a tile dealt to the waves of a block. */
enum { REC_FORM_TILES = 0, REC_FORM_WIDE = 1, REC_FORM_SPLIT = 2 };

/* The form a launch of one FC layer takes: `rows` samples, `inputs` -> `outputs`
 * features, `stacks` of them side by side, on a device of `compute_units`.
 * form[1..2]: rows and columns of a block's tile, form[3]: waves that share its k
 * (REC_FORM_TILES: zeros).  REC_ERR_ARG on a null pointer or counts that no layer has. */
REC_API rec_status rec_probe_fc_form(int32_t rows, int32_t inputs, int32_t outputs, int32_t stacks, uint32_t flags,
                          int32_t compute_units, int32_t *form);

/* Bits of rec_probe_plan()'s mask. */
enum {
    REC_PLAN_RIDE = 1,  /* Bottom-FC in the launch of the scan */
    REC_PLAN_FRONT = 2, /* scan and pooling in one launch */
    REC_PLAN_LAYER = 4, /* Bottom-FC's first layer in the launch of the scan */
    REC_PLAN_TAIL = 8   /* interaction and Predict-FC in one launch */
};
/* What an untimed rec_forward() of `batch` samples and nnz ids, its buffers 16-byte
 * aligned, would run with the options as set (no workspace needed): *mask, and in
 * *tail_from the first Bottom-FC layer that the launch of REC_PLAN_TAIL takes (the number
 * of layers: none).  REC_ERR_ARG on a null pointer or a batch that the model does not take. */
REC_API rec_status rec_probe_plan(const rec_model *m, int32_t batch, int64_t nnz, uint32_t *mask, int32_t *tail_from);
/* The same, *joined = 1 where pooling is in the launch of REC_PLAN_LAYER too, a layer of large tiles. */
REC_API rec_status rec_probe_plan_joined(const rec_model *m, int32_t batch, int64_t nnz, int32_t *joined);

/* Forms of pooling: launches of their own (a bag a wave, two bags a wave, several bags of a few ids a wave, hot
 * rows from LDS) ... */
enum {
    REC_POOL_BAG = 0, REC_POOL_TWO = 1, REC_POOL_SHORT = 2, REC_POOL_HOT = 3,
    /* ... and with the scan in one: beside Bottom-FC or its first layer in small tiles, a whole Bottom-FC within 64
     * registers, a few lookups of a concatenation model, many of them, beside a first layer of large tiles. */
    REC_POOL_FRONT = 4, REC_POOL_FRONT_LIGHT = 5, REC_POOL_FEW_LOOKUPS = 6, REC_POOL_MANY_LOOKUPS = 7, REC_POOL_BESIDE_WIDE = 8
};
/* The one that rec_forward() would take, as rec_probe_plan(). */
REC_API rec_status rec_probe_plan_pooling(const rec_model *m, int32_t batch, int64_t nnz, int32_t *form);

/* How a launch that copies the dense part of a concatenation model without Bottom-FC (`rows`
 * samples of `columns` features, then `pad` zeros a row) deals it: deal[0] blocks of deal[1]
 * waves, deal[2] units a wave at most, a unit four wave-wide accesses.  left: -1, the launch of the scan or of
 * scan and a few lookups; else compute units without a block of the launch of many lookups. */
REC_API rec_status rec_probe_dense_copy(int32_t rows, int32_t columns, int32_t pad, int32_t left, int32_t *deal);

#ifdef __cplusplus
}
#endif
#endif /* REC_PROBE_H */
