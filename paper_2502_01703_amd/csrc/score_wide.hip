// qless_score / qless_score16 / qless_score_mixed against more than 64 validation vectors: the tile kernel of
// the 8-bit codes (int8 products) and of bfloat16 rows.
//
// Bound: the matrix cores under the card's power limit.  At 270 000 x 1024 x 4 checkpoints, k = 8192, 8 bits, the
// matrix instructions alone (random operands) take 4.8 ms at 2.0 GHz; LDS operand reads add 1.6 ms, the
// copies into LDS 2 ms -- and most of that as clock (the card falls to 1.7 - 1.8 GHz while the matrix pipes
// are busy 54 % of the cycles), so what counts is bytes moved per product, then latency at the barriers.
//   * Tiles of 192 x 256, 256 x 192, 256 x 128 or 512 x 96 (train x validation), eight wavefronts of 96 x 64,
//     64 x 96 or 64 x 64: the fp32 checkpoint sums and the accumulators of a larger tile do not fit in
//     registers next to each other.  choose_shape() picks by padded work.
//   * A stage is 128 bytes (a whole cache line) of every train and validation row of the tile, copied
//     global -> LDS asynchronously into a ring of two or three stages.  The pre-pass lays the validation rows out
//     stage by stage as they lie in LDS, so their copies are linear.
//   * One barrier per stage, between the matrix instructions of its last K step: everything of the stage is in
//     registers by then, so the copies of the stage after the ring and the operand reads of the next stage
//     start behind it while the remaining instructions run, and no wavefront waits for its first operands
//     after a barrier (the kernel before: barrier, then reads, then instructions).
//   * Every matrix instruction is followed by one operand read or copy of the next K step.
//   * 16-byte chunk c of row r lies at position c ^ ((r / 2) % 8): 16 consecutive rows read together use all 64
//     banks (c ^ (r % 8), conflict-free for 32 banks, cost 5 %).
// Measured, same card, N = 270 000, k = 8192, C = 4 (before -> now): 8 bits, M = 1024: 10.0 -> 8.5 ms; bfloat16 65536 x 512:
// 2.51 -> 2.15 ms.
#include "score.h"

namespace qless {

typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(16))) int i32x16;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;

struct WidePrep {                              // workspace views (device pointers)
    unsigned char *vexp;                       // [C][val tile][stage][VT rows x 128 bytes], zero past the rows and their ends
    float *vw;                                 // [C][Mp] eta * rnorm'
    unsigned int *smax;                        // [N] order-preserving keys of the row maxima
    int32_t Mp, cb, nst;                       // padded validation rows, bytes per row, stages per row
};

template <bool BF16> struct WideAcc { typedef i32x16 type; };
template <> struct WideAcc<true> { typedef f32x16 type; };
template <bool BF16>
__device__ inline typename WideAcc<BF16>::type wide_mma(i32x4 a, i32x4 b, typename WideAcc<BF16>::type c);
template <>
__device__ inline i32x16 wide_mma<false>(i32x4 a, i32x4 b, i32x16 c) { return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0); }
template <>
__device__ inline f32x16 wide_mma<true>(i32x4 a, i32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// One workgroup per (padded validation row, checkpoint); the first checkpoint's also clear the row-maximum keys.
__global__ void __launch_bounds__(256)
score_wide_prepare_kernel(ScoreArgs a, WidePrep w, int VT, int bf16) {
    const int row = blockIdx.x, ci = blockIdx.y, vt = row / VT, r = row % VT;
    unsigned char *dst = w.vexp + ((size_t)ci * w.Mp + (size_t)vt * VT) * (size_t)w.nst * 128 + (size_t)r * 128;
    const unsigned char *src = a.vc[ci] + (int64_t)(row < a.M ? row : 0) * w.cb;
    for (int t = threadIdx.x; t < w.nst * 8; t += 256) {
        const int st = t >> 3, c = t & 7;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (row < a.M && st * 128 + c * 16 < w.cb) v = *(const uint4 *)(src + st * 128 + c * 16);
        *(uint4 *)(dst + (size_t)st * VT * 128 + ((c ^ ((r >> 1) & 7)) << 4)) = v;
    }
    if (threadIdx.x == 0) w.vw[ci * w.Mp + row] = row < a.M ? (bf16 ? a.eta[ci] : __fmul_rn(a.eta[ci], a.vr[ci][row])) : 0.0f;
    if (ci == 0) {
        const int64_t per = (a.N + gridDim.x - 1) / gridDim.x, lo = (int64_t)row * per;
        for (int64_t i = lo + threadIdx.x; i < lo + per && i < a.N; i += 256) w.smax[i] = 0u;
    }
}

// A wavefront owns WR x WC accumulators of 32 x 32, WY x WX wavefronts make a tile of 32 WR WY train rows x 32 WC WX
// validation rows; NBUF stages in the ring.
template <int BITS_, int WR_, int WC_, int WY_, int WX_, int NBUF_>
struct WideShape {
    static constexpr int BITS = BITS_, WR = WR_, WC = WC_, WY = WY_, WX = WX_, NBUF = NBUF_, NW = WY * WX;
    static constexpr int MT = 32 * WR * WY, VT = 32 * WC * WX;
    static constexpr int TBYTES = MT * 128, VBYTES = VT * 128, BUF = TBYTES + VBYTES;
    static constexpr int TCP = TBYTES / 1024, VCP = VBYTES / 1024;              // 1 KB copies per stage
    static constexpr int TU = (TCP + NW - 1) / NW, VU = (VCP + NW - 1) / NW, LPW = TU + VU;      // per wavefront
    static_assert(TCP % NW == 0, "a copy's parity follows from its number");
    static constexpr int LDS = NBUF * BUF;
    static_assert(NBUF >= 2 && LDS + 4 * MT <= (int)kLdsPerCU, "the ring and the row maxima fit in LDS");
    static_assert((NBUF - 1) * LPW < 64, "vmcnt is a 6-bit counter");
};

// Where the copies of train rows read, in bytes from the tile's first row (and the stage's 128 q bytes into it): copy q takes
// rows 8 q + lane / 8, chunk (lane % 8) ^ ((row / 2) % 8).
//   wide_lane_offset     the lane's part beside the wave-uniform 8 q cb.  Chunks past a row's end read on into the rows
//                        after it (the validation bytes there are zero).
//   wide_reads_past      whether that leaves the store: its last rows are shorter than a stage, and one row of 32 bytes
//                        (4 bits, k = 64) reaches three rows on, so this can be the tile before the last one as well.
//   wide_clamped_offset  for such tiles: rows past N re-read the last row (masked later), chunks past the row end its last
//                        16 bytes.  over: bytes of this stage past the end of a row.
__host__ __device__ inline unsigned wide_lane_offset(unsigned lane, int q, int cb) {
    return (lane >> 3) * (unsigned)cb + (((lane & 7) ^ ((4u * (unsigned)q + (lane >> 4)) & 7)) << 4);
}
__host__ __device__ inline bool wide_reads_past(int64_t row0, int MT, int64_t N, int cb, int nst) {
    return (row0 + MT - 1) * cb + (int64_t)nst * 128 > N * cb;
}
__host__ __device__ inline unsigned wide_clamped_offset(unsigned lane, int q, int64_t row0, int64_t N, int cb, int over) {
    const int64_t r = row0 + q * 8 + (int)(lane >> 3), gr = r < N ? r : N - 1;
    int at = (int)(((lane & 7) ^ ((4u * (unsigned)q + (lane >> 4)) & 7)) << 4);
    if (over > 0 && at > 112 - over) at = 112 - over;
    return (unsigned)((gr - row0) * cb) + (unsigned)at;
}

// EDGE = false: every tile has MT rows that exist (the last one starts at N - MT and repeats rows of the tile before
// it, with the same results) and rows are whole stages.  EDGE = true: fewer train rows than a tile, or rows that
// end inside a stage, whose last tiles may not read past the store; the branch this takes per copy costs 10 % in the
// 256 x 128 shape (2.42 against 2.20 ms, bfloat16 65536 x 512).
template <class Sh, bool EDGE>
__global__ void __launch_bounds__(64 * Sh::NW, Sh::NW / 4)
score_wide_kernel(ScoreArgs a, WidePrep w, int64_t ttiles, int vtiles) {
    constexpr bool BF16 = Sh::BITS == 16;
    constexpr int WR = Sh::WR, WC = Sh::WC, WX = Sh::WX, NBUF = Sh::NBUF, NW = Sh::NW, MT = Sh::MT, VT = Sh::VT;
    constexpr int TBYTES = Sh::TBYTES, VBYTES = Sh::VBYTES, BUF = Sh::BUF, VCP = Sh::VCP, TU = Sh::TU, VU = Sh::VU, LPW = Sh::LPW;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ unsigned int s_rowmax[MT];
    // XCD-aware decode: the vtiles workgroups of one train tile get ids 8 apart (same XCD, same L2)
    const int64_t id = blockIdx.x, jj = id >> 3;
    const int vt = (int)(jj % vtiles);
    const int64_t tt = (jj / vtiles) * 8 + (id & 7);
    if (tt >= ttiles) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int trow = wave / WX * 32 * WR, vcol = wave % WX * 32 * WC;           // this wavefront's corner inside the tile
    const int64_t row0 = EDGE || tt * MT + MT <= a.N ? tt * MT : a.N - MT;
    for (int i = tid; i < MT; i += 64 * NW) s_rowmax[i] = 0u;
    const unsigned lds0 = (unsigned)(uintptr_t)((__attribute__((address_space(3))) unsigned char *)smem);

    // ---- copies, 1 KB each: TU of train rows (8 rows x 128 bytes) and VU of validation rows (linear) per wavefront and
    // stage; past the end of the validation side a wavefront repeats its last copy, so that all count the same number.
    // The address is a wave-uniform base plus a lane part that the copies share: the tiles fill the register file,
    // and a spilled register is read back through the same counter as the copies.
    const int T = a.C * w.nst;                            // stages of all checkpoints, one pipeline
    const int over = EDGE ? w.nst * 128 - w.cb : 0;       // bytes of the last stage past the end of a train row
    const bool clamped = EDGE && wide_reads_past(row0, MT, a.N, w.cb, w.nst);
    const int q0 = wave * TU, v0 = wave * VU < VCP ? wave * VU : VCP - 1;     // first copy of either side
    unsigned train_lane[2];                               // of copies of even and odd distance from q0
#pragma unroll
    for (int e = 0; e < 2; ++e) train_lane[e] = wide_lane_offset((unsigned)lane, q0 + e, w.cb);
    const unsigned val_lane = (unsigned)(lane * 16);
    int i_it = 0, i_ci = 0, i_s = 0, i_buf = 0;           // the next stage to request
    const unsigned char *tb = a.tc[0] + row0 * w.cb;
    const unsigned char *vb = w.vexp + (size_t)vt * w.nst * VBYTES;
    auto copy = [&](int u) {
        if (u >= TU) {
            const int q = v0 + u - TU < VCP ? v0 + u - TU : VCP - 1;
            global_to_lds16(vb + q * 1024, val_lane, lds0 + (unsigned)(i_buf * BUF + TBYTES + q * 1024));
            return;
        }
        const int q = q0 + u;
        const unsigned lds = lds0 + (unsigned)(i_buf * BUF + q * 1024);
        if (!clamped) {
            global_to_lds16(tb + (unsigned)(q * 8 * w.cb), train_lane[u & 1], lds);
        } else {
            unsigned l = (unsigned)lane;                  // opaque, so that this stays in its branch
            asm volatile("" : "+v"(l));
            global_to_lds16(tb, wide_clamped_offset(l, q, row0, a.N, w.cb, i_s == w.nst - 1 ? over : 0), lds);
        }
    };
    auto copy_next = [&]() {
        tb += 128; vb += VBYTES; ++i_it;
        if (++i_buf == NBUF) i_buf = 0;
        if (++i_s == w.nst) {
            i_s = 0;
            if (++i_ci < a.C) { tb = a.tc[i_ci] + row0 * w.cb; vb = w.vexp + ((size_t)i_ci * vtiles + vt) * (size_t)w.nst * VBYTES; }
        }
    };

    // ---- operand reads: the lane (row l32, half) takes chunk 2 ks + half; both sides share the lane's part of the address
    const unsigned lane_base = (unsigned)(l32 * 128 + ((half ^ ((l32 >> 1) & 7)) << 4));
    const unsigned a_base = (unsigned)(trow * 128), b_base = (unsigned)(TBYTES + vcol * 128);        // wave-uniform
    i32x4 fa[WR], fb[2][WC];
    auto load_a = [&](int b, int buf, int ks) {
        fa[b] = *(const i32x4 *)(smem + ((lane_base ^ (ks << 5)) + (unsigned)(buf * BUF) + a_base) + b * 4096);
    };
    auto load_b = [&](int c, int slot, int buf, int ks) {
        fb[slot][c] = *(const i32x4 *)(smem + ((lane_base ^ (ks << 5)) + (unsigned)(buf * BUF) + b_base) + c * 4096);
    };
    auto pin = []() { __builtin_amdgcn_sched_barrier(0); };   // keeps the order below

    float facc[WR][WC][16];
#pragma unroll
    for (int b = 0; b < WR; ++b)
#pragma unroll
        for (int c = 0; c < WC; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) facc[b][c][v] = 0.0f;

    for (int i = 0; i < NBUF && i < T; ++i) {
#pragma unroll
        for (int u = 0; u < LPW; ++u) copy(u);
        copy_next();
    }
    if (NBUF <= T) wait_vmcnt<(NBUF - 1) * LPW>(); else wait_vmcnt<0>();
    __syncthreads();
#pragma unroll
    for (int c = 0; c < WC; ++c) load_b(c, 0, 0, 0);
#pragma unroll
    for (int b = 0; b < WR; ++b) load_a(b, 0, 0);
    __builtin_amdgcn_s_waitcnt(0xC07F);                   // lgkmcnt(0): no read is outstanding at the head of the loop
    int buf = 0, g = 0;
    for (int ci = 0; ci < a.C; ++ci) {
        typename WideAcc<BF16>::type acc[WR][WC];
#pragma unroll
        for (int b = 0; b < WR; ++b)
#pragma unroll
            for (int c = 0; c < WC; ++c)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[b][c][v] = 0;
        for (int s = 0; s < w.nst; ++s, ++g) {
            const int next = buf + 1 == NBUF ? 0 : buf + 1;
            const bool more = g + 1 < T, refill = i_it < T;
            // K step ks multiplies what the step before read; the train fragment of a row block is re-read as soon as
            // its instructions are issued.  In the last step the stage's buffer has been read completely
            // after the first instructions: there the barrier, and behind it the next stage's reads and the
            // copies into the buffer.
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const int cur = ks & 1, nxt = cur ^ 1;
                const int lbuf = ks < 3 ? buf : next, lks = (ks + 1) & 3;
                constexpr int K0 = WC - 1;                                      // instruction of the last step before the barrier
                constexpr int SLOTS = WR * WC - K0;                             // instructions the copies are spread over
#pragma unroll
                for (int b = 0; b < WR; ++b) {
#pragma unroll
                    for (int c = 0; c < WC; ++c) {
                        pin();
                        acc[b][c] = wide_mma<BF16>(fa[b], fb[cur][c], acc[b][c]);
                        pin();
                        if (ks < 3 && b == 0) load_b(c, nxt, lbuf, lks);
                        const int i = b * WC + c;
                        if (ks == 3 && more && i >= K0) {
                            if (i == K0) {
                                // this wavefront's reads of the stage have returned and its share of the next
                                // stage has landed; the barrier says so of all wavefronts
                                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                                if (refill) wait_vmcnt<(NBUF - 2) * LPW>(); else wait_vmcnt<0>();
                                __builtin_amdgcn_s_barrier();
                                asm volatile("" ::: "memory");
                                pin();
#pragma unroll
                                for (int q = 0; q < WC; ++q) load_b(q, nxt, lbuf, lks);
                                pin();
                            }
                            if (refill) {
#pragma unroll
                                for (int u = 0; u < LPW; ++u)
                                    if (u * SLOTS / LPW == i - K0) copy(u);
                            }
                        }
                    }
                    pin();
                    if (ks < 3 || more) load_a(b, lbuf, lks);
                }
            }
            if (refill) copy_next();
            pin();
            __builtin_amdgcn_s_waitcnt(0xC07F);
            pin();
            buf = next;
        }
        // checkpoint epilogue.  acc[b][c][v]: train row 32 b + 8 (v / 4) + 4 half + v % 4, val column 32 c + l32.
        // Lane L holds rnorm of train rows trow + L and trow + 64 + L; rows are fetched by shuffle.
        float rt_lane[(WR + 1) / 2];
#pragma unroll
        for (int q = 0; q < (WR + 1) / 2; ++q) {
            int64_t r = row0 + trow + 64 * q + lane;
            if (r > a.N - 1) r = a.N - 1;
            rt_lane[q] = (BF16 && !a.tr[ci]) ? 1.0f : a.tr[ci][r];
        }
        int row_lane = 4 * half;                          // opaque: the 16 lane numbers below are formed here, not kept over the loop
        asm volatile("" : "+v"(row_lane));
        float wv[WC];
#pragma unroll
        for (int c = 0; c < WC; ++c) wv[c] = w.vw[ci * w.Mp + vt * VT + vcol + 32 * c + l32];
#pragma unroll
        for (int b = 0; b < WR; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float rt = __shfl(rt_lane[b >> 1], 32 * (b & 1) + 8 * (v >> 2) + row_lane + (v & 3), 64);
#pragma unroll
                for (int c = 0; c < WC; ++c) {
                    const float D = (float)acc[b][c][v];
                    facc[b][c][v] = __fadd_rn(facc[b][c][v], __fmul_rn(__fmul_rn(D, rt), wv[c]));
                }
            }
    }
    // tile epilogue: optional full matrix, row maxima over this val tile
#pragma unroll
    for (int b = 0; b < WR; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int rloc = trow + 32 * b + 8 * (v >> 2) + 4 * half + (v & 3);
            const int64_t r = row0 + rloc;
            float m = neg_inf();
#pragma unroll
            for (int c = 0; c < WC; ++c) {
                const int col = vt * VT + vcol + 32 * c + l32;
                if (col < a.M) {
                    m = fmaxf(m, facc[b][c][v]);
                    if (a.full && r < a.N) a.full[r * a.M + col] = facc[b][c][v];
                }
            }
            if (a.score) {
#pragma unroll
                for (int o = 16; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
                if (l32 == 0 && m > neg_inf()) atomicMax(&s_rowmax[rloc], f32_order_key(m));
            }
        }
    if (a.score) {
        __syncthreads();
        for (int i = tid; i < MT; i += 64 * NW)
            if (row0 + i < a.N && s_rowmax[i] != 0u) atomicMax(&w.smax[row0 + i], s_rowmax[i]);
    }
}

// Padded validation rows of any shape: at most M + 255.
static size_t wide_val_rows(int32_t M) { return (size_t)(M + 255); }
static void wide_offsets(int64_t N, int32_t M, int64_t cb, int C, size_t *off_vw, size_t *off_smax, size_t *total) {
    auto up = [](size_t o) { return (o + 255) & ~(size_t)255; };
    *off_vw = up((size_t)C * wide_val_rows(M) * (size_t)((cb + 127) / 128 * 128));
    *off_smax = up(*off_vw + (size_t)C * wide_val_rows(M) * 4);
    *total = *off_smax + (size_t)(N > 0 ? N : 1) * 4;
}
size_t wide_workspace(int64_t N, int32_t M, int64_t row_bytes, int C) {
    size_t v, s, t;
    wide_offsets(N, M, row_bytes, C, &v, &s, &t);
    return t;
}

template <class Sh>
static qless_status launch_wide_shape(const ScoreArgs &a, WidePrep w, bool prepare, hipStream_t st) {
    QLESS_LDS_KERNEL((score_wide_kernel<Sh, false>), Sh::LDS);
    QLESS_LDS_KERNEL((score_wide_kernel<Sh, true>), Sh::LDS);
    w.Mp = (a.M + Sh::VT - 1) / Sh::VT * Sh::VT;
    const int vtiles = w.Mp / Sh::VT;
    const int64_t ttiles = (a.N + Sh::MT - 1) / Sh::MT, grid = 8 * (int64_t)vtiles * ((ttiles + 7) / 8);
    if (grid > 0x7FFFFFFF) return QLESS_ERR_UNSUPPORTED;
    if (prepare)
        hipLaunchKernelGGL(score_wide_prepare_kernel, dim3((unsigned)w.Mp, (unsigned)a.C), dim3(256), 0, st, a, w, Sh::VT, Sh::BITS == 16);
    if (a.N >= Sh::MT && w.cb % 128 == 0)
        hipLaunchKernelGGL((score_wide_kernel<Sh, false>), dim3((unsigned)grid), dim3(64 * Sh::NW), Sh::LDS, st, a, w, ttiles, vtiles);
    else
        hipLaunchKernelGGL((score_wide_kernel<Sh, true>), dim3((unsigned)grid), dim3(64 * Sh::NW), Sh::LDS, st, a, w, ttiles, vtiles);
    return QLESS_OK;
}

// The shape with the least padded work: rounds of one workgroup per compute unit, times the tile's pairs, times what a
// pair costs in the shape (measured at N = 270 000, M = 285 and 1024, relative to the 96 x 64 wavefronts:
// 256 x 128 6 %, 512 x 96 16 % more per pair -- more operand bytes per product).  The validation tiles of a train tile run
// on one XCD, so the rounds are those of the XCD with the most train tiles: 25 316 x 773 in tiles of 256 x 192 is 495
// workgroups, but 65 of them on three of the XCDs, a third round (6016 codes of 4 bits: 202 us; 256 x 128: 169).
static int choose_shape(int64_t N, int32_t M) {
    static const struct { int mt, vt; double cost; } s[4] = {{192, 256, 1.0}, {256, 192, 1.0}, {256, 128, 1.06}, {512, 96, 1.16}};
    const int64_t cus = (compute_units() + 7) / 8;                   // per XCD
    int best = 0;
    double least = 0;
    for (int i = 0; i < 4; ++i) {
        const int64_t ttiles = (N + s[i].mt - 1) / s[i].mt, tiles = (ttiles + 7) / 8 * ((M + s[i].vt - 1) / s[i].vt);
        const double c = (double)((tiles + cus - 1) / cus) * s[i].mt * s[i].vt * s[i].cost;
        if (i == 0 || c < least) { best = i; least = c; }
    }
    return best;
}

template <int BITS>
static qless_status launch_wide_bits(const ScoreArgs &a, const WidePrep &w, int shape, bool prepare, hipStream_t st) {
    switch (shape) {
        case 0: return launch_wide_shape<WideShape<BITS, 3, 2, 2, 4, 2>>(a, w, prepare, st);
        case 1: return launch_wide_shape<WideShape<BITS, 2, 3, 4, 2, 2>>(a, w, prepare, st);
        case 2: return launch_wide_shape<WideShape<BITS, 2, 2, 4, 2, 3>>(a, w, prepare, st);
        default: return launch_wide_shape<WideShape<BITS, 2, 3, 8, 1, 2>>(a, w, prepare, st);
    }
}

qless_status launch_wide(const ScoreArgs &a, int bits, void *ws, hipStream_t st, bool prepare, int64_t plan_rows) {
    const int64_t rows = plan_rows > 0 ? plan_rows : a.N;
    WidePrep w{};
    w.cb = bits == 16 ? a.k : a.k * bits / 8;
    w.nst = (w.cb + 127) / 128;
    size_t off_vw, off_smax, total;
    wide_offsets(rows, a.M, w.cb, a.C, &off_vw, &off_smax, &total);
    unsigned char *base = (unsigned char *)ws;
    w.vexp = base; w.vw = (float *)(base + off_vw); w.smax = (unsigned int *)(base + off_smax);
    const int shape = choose_shape(rows, a.M);            // of plan_rows: the pre-pass is laid out for it
    qless_status rc;
    if (bits == 16) rc = launch_wide_bits<16>(a, w, shape, prepare, st);
    else rc = launch_wide_bits<8>(a, w, shape, prepare, st);
    if (rc != QLESS_OK) return rc;
    if (a.score) launch_score_finish(w.smax, a.N, a.score, st);
    return launch_status();
}

template <class Sh>
static int64_t wide_reach(int64_t N, int cb) {
    const int nst = (cb + 127) / 128, over = nst * 128 - cb;
    const int64_t ttiles = (N + Sh::MT - 1) / Sh::MT;
    const bool edge = !(N >= Sh::MT && cb % 128 == 0);
    int64_t most = 0;
    for (int64_t tt = ttiles > 3 ? ttiles - 3 : 0; tt < ttiles; ++tt) {
        const int64_t row0 = edge || tt * Sh::MT + Sh::MT <= N ? tt * Sh::MT : N - Sh::MT;
        const bool clamped = edge && wide_reads_past(row0, Sh::MT, N, cb, nst);
        for (int s = 0; s < nst; ++s)
            for (int q = 0; q < Sh::TCP; ++q)
                for (unsigned lane = 0; lane < 64; ++lane) {
                    const int64_t off = clamped ? (int64_t)wide_clamped_offset(lane, q, row0, N, cb, s == nst - 1 ? over : 0)
                                                : (int64_t)q * 8 * cb + wide_lane_offset(lane, q, cb);
                    const int64_t end = row0 * cb + (int64_t)s * 128 + off + 16;
                    most = end > most ? end : most;
                }
    }
    return most;
}

}  // namespace qless

// For the tests, host only: the end of the last byte of the train rows that any copy of tile shape `shape` reads (at most
// N * row_bytes), from the kernel's own address arithmetic.
extern "C" int64_t qless_internal_wide_reach(int64_t N, int row_bytes, int shape) {
    using namespace qless;
    switch (shape) {
        case 0: return wide_reach<WideShape<8, 3, 2, 2, 4, 2>>(N, row_bytes);
        case 1: return wide_reach<WideShape<8, 2, 3, 4, 2, 2>>(N, row_bytes);
        case 2: return wide_reach<WideShape<8, 2, 2, 4, 2, 3>>(N, row_bytes);
        default: return wide_reach<WideShape<8, 2, 3, 8, 1, 2>>(N, row_bytes);
    }
}

// For the tests, host only: the tile shape that a call with N train rows and M validation vectors takes.
extern "C" int qless_internal_wide_shape(int64_t N, int32_t M) { return qless::choose_shape(N, M); }
