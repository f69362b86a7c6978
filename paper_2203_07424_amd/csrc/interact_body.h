// Pairwise-dot interaction of one sample by one wavefront, operands in registers
// (csrc/interact.hip describes the split into bf16 planes).
//
// The Gram matrix X X^T takes the same fragment for both operands: lane l holds
// row 16 I + l % 16, columns 32 ks + 8 (l / 16) ... + 8 of X, which is two 16-byte
// loads of the fp32 row.  So a wave loads every row block of its sample straight
// into operand registers, splits it there, and multiplies block I by the blocks
// J <= I: no staging, no barrier, all loads of the sample in flight at once.
#ifndef REC_INTERACT_BODY_H
#define REC_INTERACT_BODY_H
#include "rec_internal.h"

namespace rec {
namespace inter {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// NBLK blocks of 16 rows (V = T + 1 <= 16 NBLK), rows of 32 KST columns.
template <int NBLK, int KST>
struct RawRows {
    f32x4 v[NBLK][KST][2];
    // Row 0 is x0 (loaded here, or null and left to load_x0()), rows 1 .. T the
    // pooled vectors (contiguous), the rest zero.
    __device__ inline void load(const float *x0, const float *pooled, int T, int lane)
    {
        const int r16 = lane & 15, kq = lane >> 4;
        const int first = x0 ? 0 : 1;
#pragma unroll
        for (int I = 0; I < NBLK; ++I) {
            const int r = 16 * I + r16;
            const float *p = (r == 0 ? x0 : pooled + (size_t)(r - 1) * (32 * KST)) + 8 * kq;
#pragma unroll
            for (int ks = 0; ks < KST; ++ks) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    v[I][ks][h] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                    if (r >= first && r <= T) v[I][ks][h] = *reinterpret_cast<const f32x4 *>(p + 32 * ks + 4 * h);
                }
            }
        }
    }
    // Row 0 from LDS.
    __device__ inline void load_x0(const float *x0, int lane)
    {
        if ((lane & 15) != 0) return;
#pragma unroll
        for (int ks = 0; ks < KST; ++ks)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                v[0][ks][h] = *reinterpret_cast<const f32x4 *>(x0 + 32 * ks + 8 * (lane >> 4) + 4 * h);
    }
};

// Predict-FC input row of one sample into `z` (LDS, 16-byte aligned, ldz bf16, zero
// behind the width): [bf16(x0), <X_i, X_j> for i > j].
template <int NBLK, int KST>
__device__ inline void gram_row(const RawRows<NBLK, KST> &raw, int T, __bf16 *z, int ldz, int lane)
{
    constexpr int D = 32 * KST;
    const int r16 = lane & 15, kq = lane >> 4;
    bf16x8 hi[NBLK][KST], lo[NBLK][KST];
#pragma unroll
    for (int I = 0; I < NBLK; ++I)
#pragma unroll
        for (int ks = 0; ks < KST; ++ks)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float x = raw.v[I][ks][e >> 2][e & 3];
                hi[I][ks][e] = (__bf16)x;
                lo[I][ks][e] = (__bf16)(x - (float)hi[I][ks][e]);
            }
    if (r16 == 0) {  // row 0's hi plane is bf16(x0)
#pragma unroll
        for (int ks = 0; ks < KST; ++ks) *reinterpret_cast<bf16x8 *>(z + 32 * ks + 8 * kq) = hi[0][ks];
    }
    const int width = D + T * (T + 1) / 2;
    for (int c = width + lane; c < ldz; c += 64) z[c] = (__bf16)0.0f;
#pragma unroll
    for (int I = 0; I < NBLK; ++I) {
        int at[4];  // where row i's terms start
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = 16 * I + 4 * kq + v;
            at[v] = D + i * (i - 1) / 2;
        }
#pragma unroll
        for (int J = 0; J <= I; ++J) {
            f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int ks = 0; ks < KST; ++ks) {
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo[I][ks], hi[J][ks], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi[I][ks], lo[J][ks], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi[I][ks], hi[J][ks], acc, 0, 0, 0);
            }
            // acc[v] = <X_i, X_j>, i = 16 I + 4 (lane / 16) + v, j = 16 J + lane % 16.
            const int j = 16 * J + r16;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = 16 * I + 4 * kq + v;
                if (i <= T && j < i) z[at[v] + j] = (__bf16)acc[v];
            }
        }
    }
}

// Does a wave's register file take a sample of this shape?
inline bool fits_wave(int T, int D) { return (D == 32 || D == 64) && T + 1 <= 64; }

}  // namespace inter
}  // namespace rec
#endif
