// What the tile kernels share: the epilogues of a wavefront that owns WR x WC accumulators of
// 32 x 32 (train rows x validation columns).  acc[b][c][v]: train row 32 b + 8 (v / 4) + 4 half + v % 4, column 32 c + lane % 32.
#pragma once
#include "score.h"

namespace qless {

typedef __attribute__((ext_vector_type(16))) float f32x16;

// Checkpoint epilogue: facc += ((unit acc) rnorm) w', rounded after every operation.  row_first: the wavefront's first train row,
// vw: weights of its first column on; rnorm may be null (1).  Lane L holds rnorm of train rows 64 q + L; rows are fetched by shuffle.
template <int WR, int WC, class Acc>
__device__ inline void tile_add_checkpoint(const Acc (&acc)[WR][WC], float unit, const float *rnorm, int64_t row_first, int64_t N,
                                           const float *vw, float (&facc)[WR][WC][16]) {
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    float rt_lane[(WR + 1) / 2];
#pragma unroll
    for (int q = 0; q < (WR + 1) / 2; ++q) {
        int64_t r = row_first + 64 * q + lane;
        if (r > N - 1) r = N - 1;
        rt_lane[q] = rnorm ? rnorm[r] : 1.0f;
    }
    int row_lane = 4 * half;                              // opaque: the 16 lane numbers below are formed here, not kept over the loop
    asm volatile("" : "+v"(row_lane));
    float wv[WC];
#pragma unroll
    for (int c = 0; c < WC; ++c) wv[c] = vw[32 * c + l32];
#pragma unroll
    for (int b = 0; b < WR; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float rt = __shfl(rt_lane[b >> 1], 32 * (b & 1) + 8 * (v >> 2) + row_lane + (v & 3), 64);
#pragma unroll
            for (int c = 0; c < WC; ++c) {
                const float D = unit == 1.0f ? (float)acc[b][c][v] : unit * (float)acc[b][c][v];
                facc[b][c][v] = __fadd_rn(facc[b][c][v], __fmul_rn(__fmul_rn(D, rt), wv[c]));
            }
        }
}

// The value of another lane of its row of 16 (row_mirror, row_half_mirror, quad_perm)
template <int CTRL> __device__ inline float lane_moved(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}
// One step of a reduction that scatters its results: of 2 H values a lane keeps H (the upper ones where `upper`), each joined with the
// same value of the lane that CTRL names, which keeps the others.
template <int H, int CTRL> __device__ inline void max_scatter(float *m, bool upper) {
#pragma unroll
    for (int j = 0; j < H; ++j) {
        const float keep = upper ? m[j + H] : m[j], send = upper ? m[j] : m[j + H];
        m[j] = fmaxf(keep, lane_moved<CTRL>(send));
    }
}

// Tile epilogue: optional full matrix, row maxima over this tile's columns into s_rowmax (per train row of the tile; the caller takes
// them on behind a barrier).  trow: the wavefront's first row in the tile, col_first its first column.  The 16 rows of a lane's
// accumulator are reduced over 16 lanes in four scattering steps, 15 moves, after which lane l holds row l % 16, and over the other 16 lanes
// with one more (five shuffles and a branch per row: 5 to 7 us more per tile, 270 000 x 1024 x 4 at 2 bits 3.80 against 3.60 ms).
template <int WR, int WC>
__device__ inline void tile_finish(const ScoreArgs &a, const float (&facc)[WR][WC][16], int64_t row0, int trow, int col_first, unsigned int *s_rowmax) {
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
#pragma unroll
    for (int b = 0; b < WR; ++b) {
        float m[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int64_t r = row0 + trow + 32 * b + 8 * (v >> 2) + 4 * half + (v & 3);
            m[v] = neg_inf();
#pragma unroll
            for (int c = 0; c < WC; ++c) {
                const int col = col_first + 32 * c + l32;
                if (col < a.M) {
                    m[v] = fmaxf(m[v], facc[b][c][v]);
                    if (a.full && r < a.N) a.full[r * a.M + col] = facc[b][c][v];
                }
            }
        }
        if (a.score) {                                // uniform
            max_scatter<8, 0x140>(m, lane & 8);           // lanes i, 15 - i
            max_scatter<4, 0x141>(m, lane & 4);           // i, 7 - i of 8
            max_scatter<2, 0x4E>(m, lane & 2);            // i, i ^ 2
            max_scatter<1, 0xB1>(m, lane & 1);            // i, i ^ 1
            const float best = fmaxf(m[0], __shfl_xor(m[0], 16, 64));
            const int v = lane & 15;
            if (!(lane & 16) && best > neg_inf()) atomicMax(&s_rowmax[trow + 32 * b + 8 * (v >> 2) + 4 * half + (v & 3)], f32_order_key(best));
        }
    }
}

}  // namespace qless
