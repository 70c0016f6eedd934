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
//   * Two rings, as in score_codes.hip: lines (128 bytes) of every train row in a ring of three (512 rows: two), half lines of every
//     validation row in a ring of three; the pre-pass lays the validation rows out in the order in which the lanes read them.  One ring
//     of two whole-line stages of both had every copy start behind one barrier and land before the next.
//   * One barrier per half line, behind the second matrix instruction of its last K step: everything of the half line is in
//     registers by then.  Validation fragments are requested again as soon as their last instruction is issued, train fragments
//     of the next K step go to registers of their own.
// Measured, same card, k = 8192, C = 4 (one ring of whole-line stages, row maxima by shuffles -> now): 8 bits, N = 270 000, M = 1024 8.63 -> 7.86 ms,
// M = 285 3.43 -> 3.19; 30 000 x 285 x 3, k = 4160 184 -> 155 us; bfloat16 65 536 x 512 2.16 -> 2.02 ms, 65 536 x 285, k = 4096 848 -> 750 us.
// Rings of four half lines: the same.
#include "score_tile.h"

namespace qless {

typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(16))) int i32x16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;

struct WidePrep {                              // workspace views (device pointers)
    unsigned char *vexp;                       // [C][val tile][half line][2 K steps][2 halves][VT rows][16 bytes], zero past the rows and their ends
    float *vw;                                 // [C][Mp] eta * rnorm'
    unsigned int *smax;                        // [N] order-preserving keys of the row maxima
    int32_t Mp, cb, nst;                       // padded validation rows, bytes and lines per row
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

// grid (32 padded validation rows, checkpoint, part of the row): a thread takes one row's 16-byte chunks j, j + 8, .. of the part; the first
// checkpoint's workgroups clear the row-maximum keys.
__global__ void __launch_bounds__(256)
score_wide_prepare_kernel(ScoreArgs a, WidePrep w, int VT, int bf16) {
    const int ci = blockIdx.y, rl = threadIdx.x & 31, j = threadIdx.x >> 5, row = (int)blockIdx.x * 32 + rl, r = row % VT;
    // chunk t: half line t / 4; 2 * (K step) + half = t % 4
    unsigned char *dst = w.vexp + ((size_t)ci * w.Mp + row - r) * (size_t)w.nst * 128;
    const unsigned char *src = a.vc[ci] + (int64_t)(row < a.M ? row : 0) * w.cb;
    const int chunks = w.cb / 16, per = (w.nst + (int)gridDim.z - 1) / (int)gridDim.z * 8, t0 = (int)blockIdx.z * per;
    for (int t = t0 + j; t < t0 + per && t < w.nst * 8; t += 8) {
        uint4 v = make_uint4(0, 0, 0, 0);
        if (row < a.M && t < chunks) v = *(const uint4 *)(src + t * 16);
        *(uint4 *)(dst + ((size_t)t * VT + r) * 16) = v;
    }
    if (blockIdx.z == 0 && j == 0) w.vw[ci * w.Mp + row] = row < a.M ? (bf16 ? a.eta[ci] : __fmul_rn(a.eta[ci], a.vr[ci][row])) : 0.0f;
    if (ci == 0) {
        const int64_t groups = (int64_t)gridDim.x * gridDim.z, g = (int64_t)blockIdx.z * gridDim.x + blockIdx.x;
        const int64_t share = (a.N + groups - 1) / groups, lo = g * share;
        for (int64_t i = lo + threadIdx.x; i < lo + share && i < a.N; i += 256) w.smax[i] = 0u;
    }
}

// A wavefront owns WR x WC accumulators of 32 x 32, WY x WX wavefronts make a tile of 32 WR WY train rows x 32 WC WX
// validation rows; NT lines of train rows and NV half lines of validation rows in the rings.
template <int BITS_, int WR_, int WC_, int WY_, int WX_, int NT_, int NV_>
struct WideShape {
    static constexpr int BITS = BITS_, WR = WR_, WC = WC_, WY = WY_, WX = WX_, NT = NT_, NV = NV_, NW = WY * WX;
    static constexpr int MT = 32 * WR * WY, VT = 32 * WC * WX;
    static constexpr int TBYTES = MT * 128, VBYTES = VT * 64;
    static constexpr int TCP = TBYTES / 1024, VCP = VBYTES / 1024;              // 1 KB copies
    static constexpr int TU = TCP / NW, VU = (VCP + NW - 1) / NW;               // per wavefront
    static constexpr int LDS = NT * TBYTES + NV * VBYTES;
    static_assert(TCP % NW == 0 && VBYTES % 1024 == 0, "whole copies");
    static_assert((NT == 2 || NT == 3) && NV >= 3 && LDS + 4 * MT <= (int)kLdsPerCU, "the rings and the row maxima fit in LDS");
    static_assert((NV - 1) * VU + 2 * TU < 64, "vmcnt is a 6-bit counter");
};

// Where the copies of train rows read, in bytes from the tile's first row (and the line's 128 bytes into it): copy q takes rows
// 8 q + lane / 8, of each the chunk (lane % 8) ^ ((row / 2) % 8): 16 consecutive rows read together use all 64 banks.  EDGE: rows past
// `last_row` re-read that one (masked later), chunks past `last_chunk` bytes re-read that one (the validation bytes there are zero).
template <bool EDGE>
__host__ __device__ inline unsigned wide_offset(unsigned lane, int q, int cb, unsigned last_row, unsigned last_chunk) {
    unsigned row = (lane >> 3) * (unsigned)cb + 8u * (unsigned)q * (unsigned)cb, at = ((lane & 7) ^ ((4u * (unsigned)q + (lane >> 4)) & 7)) << 4;
    if (EDGE) { row = row < last_row ? row : last_row; at = at < last_chunk ? at : last_chunk; }
    return row + at;
}

// EDGE = false: every tile has MT rows that exist (the last one starts at N - MT and repeats rows of the tile before
// it, with the same results) and rows are whole lines.  EDGE = true: fewer train rows than a tile, or rows that
// end inside a line.  The straight-line stage: see score_codes_kernel.
template <class Sh, bool EDGE>
__global__ void __launch_bounds__(64 * Sh::NW, Sh::NW / 4)
score_wide_kernel(ScoreArgs a, WidePrep w, int64_t ttiles, int vtiles) {
    constexpr bool BF16 = Sh::BITS == 16;
    constexpr int WR = Sh::WR, WC = Sh::WC, WX = Sh::WX, NT = Sh::NT, NV = Sh::NV, NW = Sh::NW, MT = Sh::MT, VT = Sh::VT;
    constexpr int TBYTES = Sh::TBYTES, VBYTES = Sh::VBYTES, VCP = Sh::VCP, TU = Sh::TU, VU = Sh::VU;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];        // [NT][TBYTES], [NV][VBYTES]
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

    // ---- copies: TU of a line of train rows, VU of half a line's validation rows (linear) per wavefront; past the end of the
    // validation side a wavefront repeats its last copy, so that all count the same number
    const int nst = w.nst, T = a.C * nst;                 // lines per row, and of all checkpoints
    const int over = nst * 128 - w.cb;                    // bytes of the last line past the end of a train row
    const unsigned last_row = EDGE ? (unsigned)((a.N - 1 - row0 < MT ? a.N - 1 - row0 : MT) * w.cb) : 0u;
    const int q0 = wave * TU;
    unsigned train_lane[2];                               // of copies of even and odd distance from q0, beside the wave-uniform 8 q cb
#pragma unroll
    for (int e = 0; e < 2; ++e) train_lane[e] = wide_offset<false>((unsigned)lane, q0 + e, w.cb, 0, 0) - 8u * (unsigned)(q0 + e) * (unsigned)w.cb;
    const unsigned val_lane = (unsigned)(lane * 16);
    // the checkpoints' train rows: lane i holds the tile's first row of checkpoint i
    const uint64_t tile_row = (uint64_t)(a.tc[lane < a.C ? lane : 0] + row0 * w.cb);
    auto train_of = [&](int ci) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)tile_row, ci);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(tile_row >> 32), ci);
        return (const unsigned char *)(((uint64_t)hi << 32) | lo);
    };
    int t_it = 0, t_ci = 0, t_s = 0, t_slot = 0;          // the next line of train rows to request
    int v_it = 0, v_s = 0, v_slot = 0;                    // and the next half line of validation rows
    const unsigned char *tb = train_of(0);
    const unsigned char *vb = w.vexp + (size_t)vt * (2 * nst) * VBYTES;
    const size_t v_wrap = (size_t)(vtiles - 1) * (2 * nst) * VBYTES;
    auto copy_train = [&](int u) {
        const int q = q0 + u;
        const unsigned lds = lds0 + (unsigned)(t_slot * TBYTES + q * 1024);
        if (EDGE) {
            unsigned l = (unsigned)lane;                  // opaque: formed here, not kept in a register per copy
            asm volatile("" : "+v"(l));
            global_to_lds16(tb, wide_offset<true>(l, q, w.cb, last_row, t_s == nst - 1 ? (unsigned)(112 - over) : 112u), lds);
        } else {
            global_to_lds16(tb + (unsigned)(q * 8 * w.cb), train_lane[u & 1], lds);
        }
    };
    auto copy_val = [&](int u) {
        const int at = wave * VU + u, q = VCP % (NW * VU) == 0 || at < VCP ? at : VCP - 1;
        global_to_lds16(vb + q * 1024, val_lane, lds0 + (unsigned)(NT * TBYTES + v_slot * VBYTES + q * 1024));
    };
    auto next_train = [&]() {
        const bool end = t_it + 1 >= T, wrap = !end && t_s + 1 == nst;
        t_ci += wrap ? 1 : 0;
        const unsigned char *first = train_of(t_ci);
        tb = wrap ? first : tb + (end ? 0 : 128);
        t_s = wrap ? 0 : t_s + (end ? 0 : 1);
        ++t_it;
        t_slot = t_slot + 1 == NT ? 0 : t_slot + 1;
    };
    auto next_val = [&]() {
        const bool end = v_it + 1 >= 2 * T, wrap = !end && v_s + 1 == 2 * nst;
        vb += (end ? 0 : VBYTES) + (wrap ? v_wrap : 0);
        v_s = wrap ? 0 : v_s + (end ? 0 : 1);
        ++v_it;
        v_slot = v_slot + 1 == NV ? 0 : v_slot + 1;
    };

    // ---- operands.  Train: the lane (row l32, half) takes chunk 2 * (K step of the line) + half; validation: 16 bytes at
    // [K step of the half line][half][row].
    const unsigned a_lane = (unsigned)(l32 * 128 + ((half ^ ((l32 >> 1) & 7)) << 4)), a_base = (unsigned)(trow * 128);
    const unsigned b_lane = (unsigned)((half * VT + vcol + l32) * 16);
    i32x4 fa[2][WR], fb[WC];
    auto load_a = [&](int set, int b, int slot, int ks) {
        fa[set][b] = *(const i32x4 *)(smem + (a_lane ^ (unsigned)(ks << 5)) + (unsigned)(slot * TBYTES) + a_base + b * 4096);
    };
    auto load_b = [&](int c, int slot, int ks) {
        fb[c] = *(const i32x4 *)(smem + NT * TBYTES + (unsigned)(slot * VBYTES) + b_lane + (2 * ks * VT + 32 * c) * 16);
    };
    auto pin = []() { __builtin_amdgcn_sched_barrier(0); };   // keeps the order below

    float facc[WR][WC][16];
#pragma unroll
    for (int b = 0; b < WR; ++b)
#pragma unroll
        for (int c = 0; c < WC; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) facc[b][c][v] = 0.0f;

    // The first requests, in the order in which the loop goes on: at the barrier of half line h validation rows h + NV, behind them
    // (odd h) the line of train rows NT lines on from the one that is done.
    for (int i = 0; i < NT; ++i) {
        if (i == NT - 1)
            for (int j = 0; j < NV; ++j) {
#pragma unroll
                for (int u = 0; u < VU; ++u) copy_val(u);
                next_val();
            }
#pragma unroll
        for (int u = 0; u < TU; ++u) copy_train(u);
        next_train();
    }
    wait_vmcnt<(NV - 1) * VU + TU>();                     // the first line and half line
    __syncthreads();
#pragma unroll
    for (int c = 0; c < WC; ++c) load_b(c, 0, 0);
#pragma unroll
    for (int b = 0; b < WR; ++b) load_a(0, b, 0, 0);
    int tslot = 0, vslot = 0;
    for (int ci = 0; ci < a.C; ++ci) {
        typename WideAcc<BF16>::type acc[WR][WC];
#pragma unroll
        for (int b = 0; b < WR; ++b)
#pragma unroll
            for (int c = 0; c < WC; ++c)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[b][c][v] = 0;
        for (int s = 0; s < nst; ++s) {
            const int tnext = tslot + 1 == NT ? 0 : tslot + 1;
            // Column block by column block: a validation fragment is requested again (for the next K step) as soon as its last
            // instruction is issued; the train fragments of the next K step go to registers of their own.
#pragma unroll
            for (int k4 = 0; k4 < 4; ++k4) {                                    // K steps of the line: h = k4 / 2 the half line
                const int h = k4 >> 1, cur = k4 & 1;
                const bool last = k4 & 1;                                       // of its half line
                const int vnext = vslot + 1 == NV ? 0 : vslot + 1;
                const int rt = k4 == 3 ? tnext : tslot, rv = last ? vnext : vslot, ra = (k4 + 1) & 3, rb = last ? 0 : 1;   // the next K step's
                constexpr int I = WR * WC, K0 = 1;                              // instructions of a K step; the last one's before the barrier
#pragma unroll
                for (int i = 0; i < I; ++i) {
                    const int c = i / WR, b = i % WR;
                    pin();
                    acc[b][c] = wide_mma<BF16>(fa[cur][b], fb[c], acc[b][c]);
                    asm volatile("" : "+v"(acc[b][c]) :: "memory");              // stays here, between the reads before and behind it
                    pin();
                    if (last && i == K0) {
                        // this wavefront's reads of the half line (and line) have returned and its share of the next one has
                        // landed; the barrier says so of all wavefronts.  Younger: validation rows of the half lines after it and,
                        // with three lines in the ring or none needed now, a line of train rows.
                        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                        if (h == 0 || NT == 3) wait_vmcnt<(NV - 2) * VU + TU>(); else wait_vmcnt<VU>();
                        __builtin_amdgcn_s_barrier();
                        asm volatile("" ::: "memory");
                        pin();
                    }
                    if (last ? i >= K0 && i < K0 + WR : i < WR) load_a(cur ^ 1, last ? i - K0 : i, rt, ra);
                    if (b == WR - 1) load_b(c, rv, rb);
                    if (last && i >= K0) {
                        const int n = VU + (h == 1 ? TU : 0);                   // copies, spread over the instructions behind the barrier
#pragma unroll
                        for (int u = 0; u < VU + TU; ++u)
                            if (u < n && u * (I - K0) / n == i - K0) { if (u < VU) copy_val(u); else copy_train(u - VU); }
                    }
                }
                if (last) { next_val(); vslot = vnext; }
            }
            next_train();
            tslot = tnext;
        }
        tile_add_checkpoint<WR, WC>(acc, 1.0f, a.tr[ci], row0 + trow, a.N, w.vw + ci * w.Mp + vt * VT + vcol, facc);
    }
    wait_vmcnt<0>();                                      // no copy is under way when the workgroup gives its LDS back
    tile_finish<WR, WC>(a, facc, row0, trow, vt * VT + vcol, s_rowmax);
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
    if (prepare) {
        const unsigned rows32 = (unsigned)(w.Mp / 32);
        unsigned parts = (512 + rows32 * (unsigned)a.C - 1) / (rows32 * (unsigned)a.C);      // two workgroups per compute unit
        if (parts > (unsigned)w.nst) parts = (unsigned)w.nst;
        hipLaunchKernelGGL(score_wide_prepare_kernel, dim3(rows32, (unsigned)a.C, parts), dim3(256), 0, st, a, w, Sh::VT, Sh::BITS == 16);
    }
    if (a.N >= Sh::MT && w.cb % 128 == 0)
        hipLaunchKernelGGL((score_wide_kernel<Sh, false>), dim3((unsigned)grid), dim3(64 * Sh::NW), Sh::LDS, st, a, w, ttiles, vtiles);
    else
        hipLaunchKernelGGL((score_wide_kernel<Sh, true>), dim3((unsigned)grid), dim3(64 * Sh::NW), Sh::LDS, st, a, w, ttiles, vtiles);
    return QLESS_OK;
}

// The shape with the fastest rounds of one workgroup per compute unit.  A round takes so many microseconds per line of the rows, per checkpoint (its epilogue) and
// whatever its length, 8-bit codes and bfloat16 rows each: fitted to 115 and 170 random calls (N = 500 .. 270 000, M = 65 .. 1024, k = 64 .. 16384, C = 1 .. 6),
// each run with all four shapes.  Over these and another 98 and 140 the chosen one is 0.3 and 0.1 % behind the fastest, 10 and 5 % at most (with one price per
// padded pair, of the kernel before this one at 8 bits, 1.2 and 0.7 %, 16 and 15 %; two calls of the 523 are 8 and 10 % slower for it): short rows want few
// epilogues, 29 863 x 832 x 3, k = 128 bfloat16 66.8 us in 192 x 256 tiles, 59.4 in 256 x 192; long ones
// the 192 x 256 tiles: 65 536 x 512 x 4, k = 8192 2020 and 2153 us).  The validation tiles of a train tile run
// on one XCD, so the rounds are those of the XCD with the most train tiles: 25 316 x 773 in tiles of 256 x 192 is 495
// workgroups, but 65 of them on three of the XCDs, a third round.
struct WidePrice { int mt, vt; struct { double line, checkpoint, round; } us[2]; };
constexpr int kWideShapes = 4;
constexpr WidePrice kWidePrice[kWideShapes] = {{192, 256, {{1.164, 2.05, 8.6}, {0.985, 3.40, 9.0}}}, {256, 192, {{1.204, 1.85, 8.0}, {1.047, 1.60, 8.35}}},
                                               {256, 128, {{0.945, 1.48, 5.5}, {0.805, 1.17, 6.2}}}, {512, 96, {{1.504, 1.65, 7.7}, {1.400, 1.22, 8.6}}}};
static int choose_shape(int64_t N, int32_t M, int lines, int C, bool bf16) {
    const int64_t cus = (compute_units() + 7) / 8;                   // per XCD
    int best = 0;
    double least = 0;
    for (int i = 0; i < kWideShapes; ++i) {
        const WidePrice &s = kWidePrice[i];
        const int64_t ttiles = (N + s.mt - 1) / s.mt, tiles = (ttiles + 7) / 8 * ((M + s.vt - 1) / s.vt);
        const double us = (double)((tiles + cus - 1) / cus) * (C * (lines * s.us[bf16].line + s.us[bf16].checkpoint) + s.us[bf16].round);
        if (i == 0 || us < least) { best = i; least = us; }
    }
    return best;
}

template <int BITS> struct Wide {
    typedef WideShape<BITS, 3, 2, 2, 4, 3, 3> T192x256;
    typedef WideShape<BITS, 2, 3, 4, 2, 3, 3> T256x192;
    typedef WideShape<BITS, 2, 2, 4, 2, 3, 3> T256x128;
    typedef WideShape<BITS, 2, 3, 8, 1, 2, 3> T512x96;
};
template <int BITS>
static qless_status launch_wide_bits(const ScoreArgs &a, const WidePrep &w, int shape, bool prepare, hipStream_t st) {
    switch (shape) {
        case 0: return launch_wide_shape<typename Wide<BITS>::T192x256>(a, w, prepare, st);
        case 1: return launch_wide_shape<typename Wide<BITS>::T256x192>(a, w, prepare, st);
        case 2: return launch_wide_shape<typename Wide<BITS>::T256x128>(a, w, prepare, st);
        default: return launch_wide_shape<typename Wide<BITS>::T512x96>(a, w, prepare, st);
    }
}

qless_status launch_wide(const ScoreArgs &a, int bits, void *ws, hipStream_t st, bool prepare, int64_t plan_rows, int shape) {
    const int64_t rows = plan_rows > 0 ? plan_rows : a.N;
    WidePrep w{};
    w.cb = bits == 16 ? a.k : a.k * bits / 8;
    w.nst = (w.cb + 127) / 128;
    size_t off_vw, off_smax, total;
    wide_offsets(rows, a.M, w.cb, a.C, &off_vw, &off_smax, &total);
    unsigned char *base = (unsigned char *)ws;
    w.vexp = base; w.vw = (float *)(base + off_vw); w.smax = (unsigned int *)(base + off_smax);
    if (shape < 0) shape = choose_shape(rows, a.M, w.nst, a.C, bits == 16);       // of plan_rows: the pre-pass is laid out for it
    qless_status rc;
    if (bits == 16) rc = launch_wide_bits<16>(a, w, shape, prepare, st);
    else rc = launch_wide_bits<8>(a, w, shape, prepare, st);
    if (rc != QLESS_OK) return rc;
    if (a.score) launch_score_finish(w.smax, a.N, a.score, st);
    return launch_status();
}

template <class Sh, bool EDGE>
static int64_t wide_reach_edge(int64_t N, int cb) {
    constexpr int MT = Sh::MT;
    const int nst = (cb + 127) / 128, over = nst * 128 - cb;
    const int64_t ttiles = (N + MT - 1) / MT;
    int64_t most = 0;
    for (int64_t tt = ttiles > 3 ? ttiles - 3 : 0; tt < ttiles; ++tt) {
        const int64_t row0 = EDGE || tt * MT + MT <= N ? tt * MT : N - MT;
        const unsigned last_row = (unsigned)((N - 1 - row0 < MT ? N - 1 - row0 : MT) * cb);
        for (int s = 0; s < nst; ++s)
            for (int q = 0; q < Sh::TCP; ++q)
                for (unsigned lane = 0; lane < 64; ++lane) {
                    const int64_t end = row0 * cb + (int64_t)s * 128 + 16 + wide_offset<EDGE>(lane, q, cb, last_row, (unsigned)(112 - (s == nst - 1 ? over : 0)));
                    most = end > most ? end : most;
                }
    }
    return most;
}
template <class Sh>
static int64_t wide_reach(int64_t N, int cb) {
    return N >= Sh::MT && cb % 128 == 0 ? wide_reach_edge<Sh, false>(N, cb) : wide_reach_edge<Sh, true>(N, cb);
}

}  // namespace qless

// For the tests, host only: the end of the last byte of the train rows that any copy of tile shape `shape` reads (at most
// N * row_bytes), from the kernel's own address arithmetic.
extern "C" int64_t qless_internal_wide_reach(int64_t N, int row_bytes, int shape) {
    using namespace qless;
    switch (shape) {
        case 0: return wide_reach<Wide<8>::T192x256>(N, row_bytes);
        case 1: return wide_reach<Wide<8>::T256x192>(N, row_bytes);
        case 2: return wide_reach<Wide<8>::T256x128>(N, row_bytes);
        default: return wide_reach<Wide<8>::T512x96>(N, row_bytes);
    }
}

// For the tests, host only: the tile shape that a call takes (rows of row_bytes: 8-bit codes or, bf16 != 0, bfloat16), and the price of a round of a shape.
extern "C" int qless_internal_wide_shape(int64_t N, int32_t M, int64_t row_bytes, int C, int bf16) {
    return qless::choose_shape(N, M, (int)((row_bytes + 127) / 128), C, bf16 != 0);
}
extern "C" double qless_internal_wide_round(int shape, int64_t row_bytes, int C, int bf16) {
    const auto &p = qless::kWidePrice[shape].us[bf16 != 0];
    return C * ((double)((row_bytes + 127) / 128) * p.line + p.checkpoint) + p.round;
}
