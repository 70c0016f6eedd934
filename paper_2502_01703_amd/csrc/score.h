// Shared between the scoring kernels (score.hip, score_wide.hip, score_split.hip).
#pragma once
#include "common.h"

namespace qless {

struct ScoreArgs {
    const unsigned char *tc[QLESS_MAX_CHECKPOINTS];
    const unsigned char *vc[QLESS_MAX_CHECKPOINTS];
    const float *tr[QLESS_MAX_CHECKPOINTS];
    const float *vr[QLESS_MAX_CHECKPOINTS];
    float eta[QLESS_MAX_CHECKPOINTS];
    int C;
    int64_t N;
    int32_t M, k;                              // bfloat16 rows: k is their length in bytes
    float *score, *full;
};

__device__ inline float neg_inf() { return __uint_as_float(0xFF800000u); }
// unsigned keys that order like the fp32 values; 0 lies below every value's key
__device__ inline unsigned int f32_order_key(float f) {
    const unsigned int u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
inline float nan_below_all() { return __builtin_bit_cast(float, 0xFFFFFFFFu); }      // the value of key 0
__device__ inline float f32_from_order_key(unsigned int k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

constexpr size_t kLdsPerCU = 160 * 1024;       // LDS of one compute unit
int compute_units();                           // of the current device (256 on MI355X)

// score.hip: score[i] = the value of key smax[i], keys cleared
void launch_score_finish(unsigned int *smax, int64_t N, float *score, hipStream_t st);

// score_wide.hip: 8-bit codes and bfloat16 rows (bits = 16) against more than 64 validation vectors.
size_t wide_workspace(int64_t N, int32_t M, int64_t row_bytes, int C);
// prepare = false: the workspace still holds the pre-pass of an earlier launch with the same validation
// side, laid out for plan_rows >= a.N train rows (the finish kernel leaves the row maxima cleared).  shape: of the tile (here and below,
// for the tests; otherwise the one that serves the call best)
qless_status launch_wide(const ScoreArgs &a, int bits, void *ws, hipStream_t st, bool prepare = true, int64_t plan_rows = 0,
                         int shape = -1);

// score_codes.hip: 4-bit codes against more than 64 validation vectors.
size_t codes_workspace(int64_t N, int32_t M, int64_t row_bytes, int C);
qless_status launch_codes(const ScoreArgs &a, void *ws, hipStream_t st, int shape = -1);

// score_fp4.hip: 1- and 2-bit codes (k a multiple of 128) against more than 64 validation vectors.
// use_fp4: whether it serves a call faster than the 128 x 64 tiles of score.hip; share: with the planes of a call whose checkpoints
// are shared out over workgroups
bool use_fp4(int64_t N, int32_t M, int32_t k, int bits, int C);
size_t fp4_workspace(int64_t N, int32_t M, int32_t k, int bits, int C, bool share);
qless_status launch_fp4(const ScoreArgs &a, int bits, void *ws, size_t ws_bytes, hipStream_t st);
size_t fp4_workspace_as(int64_t N, int32_t M, int32_t k, int C, int parts);
qless_status launch_fp4_as(const ScoreArgs &a, int bits, int shape, int parts, void *ws, hipStream_t st);

// score_split.hip: few pairs (bits = 16: bfloat16 rows).  use_split: whether the path serves a call faster than the others.
// Rows hold at least 16 bytes (16 per plane for the ternary codes).
bool use_split(int64_t N, int32_t M, int64_t row_bytes, int bits, int C);
size_t split_workspace(int64_t N, int32_t M, int64_t row_bytes, int bits, int C);
// none: the score of a row none of whose sums lies above -infinity
// launch_split_finish: joins planes [C * parts][N][M] of partial dot products (int32, or fp32 of bfloat16 rows)
qless_status launch_split_finish(const ScoreArgs &a, int parts, const uint32_t *planes, bool bf16, float none, hipStream_t st);
qless_status launch_split(const ScoreArgs &a, int bits, float none, void *ws, hipStream_t st);

}  // namespace qless
