// qless_score against more than 64 validation vectors: the tile kernel of the 4-bit codes, as FP6 products.
//
// The integers -16 .. 16 are FP6 (E2M3) numbers in units of 1/8, and v_mfma_scale_f32_32x32x64_f8f6f4 takes FP6 operands at the rate
// of FP4 ones, twice the products of the int8 instruction per cycle (probe, random operands: 64 products per lane pair in 23.5 ns
// against 38.8).  Products and sums of these integers are exact in fp32 as long as they stay below 2^24 units, so the
// result is the integer that the int8 form gave.
//   * A train nibble q is taken as u = q + 8 = nibble ^ 8, whose four bits are the low bits of the FP6 number u / 8 as they stand.
//     Sixteen codes (two dwords a, b) become three dwords with seven vector-ALU operations: the eight nibbles of a go
//     where they lie, those of b two bits higher, three masks each and one rotation; the flip of the sign bits rides along
//     in a three-input operation (fp6_train).  The int8 form took six for eight codes and two instructions for their products.
//   * The pre-pass writes the validation codes as FP6 numbers in that order, and the sum of a row: sum (q + 8) v - 8 sum v starts
//     from an accumulator of -8 sum v.  Units of 1/64: |15 * 8 + 8 * 8| * 65536 < 2^24.
//   * Tiles of 256 x 192, 256 x 128, 512 x 96 or 192 x 256, eight wavefronts of 64 x 96, 64 x 64 or 96 x 64: an unpacked train fragment feeds three (two)
//     matrix instructions.
//   * Two rings: a line (128 bytes, 256 codes) of every train row of the tile in a ring of three (512 rows: two), half as many codes of
//     every validation row in a ring of three, both filled asynchronously.  Train rows come from HBM and may take two lines' time,
//     validation rows come out of the caches.  (One ring of two stages of both: every copy starts behind one barrier and is waited for at
//     the next, so latency and transfer add up: M = 1024 6.20 ms against 5.78, M = 285 2.20 against 1.96.)
//   * The pre-pass lays the validation rows out as the lanes read them, [half line][K step][half][row], so that neither copies nor reads
//     need an address per K step.
//   * One barrier per half line, behind the second matrix instruction of its last K step; operands of a K step are requested
//     during the one before.
// Measured, same card, N = 270 000, k = 8192, C = 4 (int8 form -> now): M = 1024 6.92 -> 5.78 ms, M = 285 2.53 -> 1.96 ms;
// 65536 x 512 0.95 -> 0.80 ms.  Without the copies (what the rings hold, any numbers) M = 1024 takes 4.8 ms.
#include "score_tile.h"

namespace qless {

typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(2))) int i32x2;
typedef __attribute__((ext_vector_type(8))) int i32x8;

struct CodesPrep {                             // workspace views (device pointers)
    unsigned char *vexp;                       // [C][val tile][half line][VBYTES]
    float *vw, *vbias;                         // [C][Mp] eta * rnorm', -sum v / 8
    unsigned int *smax;                        // [N] order-preserving keys of the row maxima
    int32_t Mp, cb, nst;                       // padded validation rows, bytes and lines per train row
};

// A wavefront owns WR x WC accumulators of 32 x 32, WY x WX wavefronts make a tile; NT lines of train rows in their ring.
template <int WR_, int WC_, int WY_, int WX_, int NT_>
struct CodesShape {
    static constexpr int WR = WR_, WC = WC_, WY = WY_, WX = WX_, NT = NT_, NV = 3, NW = WY * WX;
    static constexpr int MT = 32 * WR * WY, VT = 32 * WC * WX;
    static constexpr int TBYTES = MT * 128, V16 = 4 * VT * 16, VBYTES = 4 * VT * 24;      // a line of train rows, half a line's validation rows
    static constexpr int TCP = TBYTES / 1024, VCP = VBYTES / 1024;              // 1 KB copies
    static constexpr int TU = TCP / NW, VU = (VCP + NW - 1) / NW;               // per wavefront
    static constexpr int LDS = NT * TBYTES + NV * VBYTES;
    static_assert(TBYTES % (1024 * NW) == 0 && VBYTES % 1024 == 0, "whole copies");
    static_assert((NT == 2 || NT == 3) && LDS + 4 * MT <= (int)kLdsPerCU, "the rings and the row maxima fit in LDS");
    static_assert(2 * VU + TU < 64, "vmcnt is a 6-bit counter");
};
// 16-byte chunk c of row r lies at position c ^ ((r / 2) % 8): 16 consecutive rows read together use all 64 banks
__host__ __device__ inline unsigned codes_swizzle(unsigned r) { return (r >> 1) & 7; }

// 16 codes (dwords a, b) as 16 FP6 numbers (nibble ^ 8) / 8: number i at bits 6 i of three dwords, in the order a0 b1 a3 b4 a6 b7 |
// a1 b2 a4 b5 a7 | b0 a2 b3 a5 b6 of the nibbles.
__device__ inline void fp6_train(uint32_t a, uint32_t b, uint32_t flip0, uint32_t flip1, uint32_t flip2, int *out) {
    const uint32_t r = __builtin_amdgcn_alignbit(b, b, 30);                     // b rotated left by two
    // (x & y) ^ z: 0x6A
    out[0] = (int)__builtin_amdgcn_bitop3_b32(r, 0xC03C03C0u, __builtin_amdgcn_bitop3_b32(a, 0x0F00F00Fu, flip0, 0x6A), 0x6A);
    out[1] = (int)__builtin_amdgcn_bitop3_b32(r, 0x03C03C03u, __builtin_amdgcn_bitop3_b32(a, 0xF00F00F0u, flip1, 0x6A), 0x6A);
    out[2] = (int)__builtin_amdgcn_bitop3_b32(r, 0x3C03C03Cu, __builtin_amdgcn_bitop3_b32(a, 0x00F00F00u, flip2, 0x6A), 0x6A);
}
// The same order for the validation side, as signed numbers q / 8: the magnitudes (0 .. 8) in four bits, the signs in the sixth
__device__ inline void fp6_val(uint32_t a, uint32_t b, uint32_t *out) {
    auto magnitude = [](uint32_t w, uint32_t s) { return (w ^ ((s - (s >> 3)) | s)) + (s >> 3); };
    auto rotl = [](uint32_t x, int n) { return (x << n) | (x >> (32 - n)); };
    const uint32_t sa = a & 0x88888888u, sb = b & 0x88888888u, ma = magnitude(a, sa), mb = rotl(magnitude(b, sb), 2);
    const uint32_t ra = rotl(sa, 2), rb = rotl(sb, 4);
    out[0] = (ma & 0x0F00F00Fu) | (mb & 0xC03C03C0u) | (ra & 0x20020020u) | (rb & 0x00800800u);
    out[1] = (ma & 0xF00F00F0u) | (mb & 0x03C03C03u) | (ra & 0x00200200u) | (rb & 0x08008008u);
    out[2] = (ma & 0x00F00F00u) | (mb & 0x3C03C03Cu) | (ra & 0x02002002u) | (rb & 0x80080080u);
}

// grid (32 padded validation rows, checkpoint, part of the row): a thread takes one row's 16-byte chunks j, j + 8, .. of the part, so that
// a wavefront writes two runs of 512 bytes.  The first part also sums its rows' codes, the first checkpoint's workgroups clear the
// row-maximum keys.  (M = 1024, k = 8192, C = 4: a workgroup per row, its threads side by side on one row, 42 us, now 24.)
__global__ void __launch_bounds__(256)
score_codes_prepare_kernel(ScoreArgs a, CodesPrep w, int VT) {
    __shared__ int part_sum[8][32];
    const int ci = blockIdx.y, rl = threadIdx.x & 31, j = threadIdx.x >> 5, row = (int)blockIdx.x * 32 + rl, r = row % VT;
    // chunk t: half line t / 4; 2 * (K step) + half = t % 4
    unsigned char *dst = w.vexp + ((size_t)ci * w.Mp + row - r) * (size_t)w.nst * 192;
    const unsigned char *src = a.vc[ci] + (int64_t)(row < a.M ? row : 0) * w.cb;
    const int chunks = w.cb / 16;
    const int per = (w.nst + (int)gridDim.z - 1) / (int)gridDim.z * 8, t0 = (int)blockIdx.z * per;
    for (int t = t0 + j; t < t0 + per && t < w.nst * 8; t += 8) {
        uint4 v = make_uint4(0, 0, 0, 0);
        if (row < a.M && t < chunks) v = *(const uint4 *)(src + t * 16);
        uint32_t o[6];
        fp6_val(v.x, v.y, o);
        fp6_val(v.z, v.w, o + 3);
        unsigned char *p = dst + (size_t)(t / 4) * (4 * VT * 24);
        *(uint4 *)(p + (t % 4 * VT + r) * 16) = make_uint4(o[0], o[1], o[2], o[3]);
        *(uint2 *)(p + 4 * VT * 16 + (t % 4 * VT + r) * 8) = make_uint2(o[4], o[5]);
    }
    if (blockIdx.z == 0) {                                                      // uniform
        int sum = 0;
        if (row < a.M)
            for (int t = j; t < chunks; t += 8) {
                const uint4 v = *(const uint4 *)(src + t * 16);
                sum = __builtin_amdgcn_sdot8((int)v.x, 0x11111111, sum, false);
                sum = __builtin_amdgcn_sdot8((int)v.y, 0x11111111, sum, false);
                sum = __builtin_amdgcn_sdot8((int)v.z, 0x11111111, sum, false);
                sum = __builtin_amdgcn_sdot8((int)v.w, 0x11111111, sum, false);
            }
        part_sum[j][rl] = sum;
        __syncthreads();
        if (j == 0) {
#pragma unroll
            for (int q = 1; q < 8; ++q) sum += part_sum[q][rl];
            w.vw[ci * w.Mp + row] = row < a.M ? __fmul_rn(a.eta[ci], a.vr[ci][row]) : 0.0f;
            w.vbias[ci * w.Mp + row] = -0.125f * (float)sum;
        }
    }
    if (ci == 0) {
        const int64_t groups = (int64_t)gridDim.x * gridDim.z, g = (int64_t)blockIdx.z * gridDim.x + blockIdx.x;
        const int64_t share = (a.N + groups - 1) / groups, lo = g * share;
        for (int64_t i = lo + threadIdx.x; i < lo + share && i < a.N; i += 256) w.smax[i] = 0u;
    }
}

// Where the copies of train rows read, in bytes from the tile's first row (and the line's 128 bytes into it): copy q takes rows
// 8 q + lane / 8, of each the chunk that lies at position lane % 8.  Rows past `last_row` re-read that one (masked later),
// chunks past `last_chunk` bytes re-read that one (the validation numbers there are zero); without EDGE neither happens.
__host__ __device__ inline unsigned codes_lane_row(unsigned lane, int cb) { return lane / 8 * (unsigned)cb; }
__host__ __device__ inline unsigned codes_lane_chunk(unsigned lane, int q) {          // depends on q's parity only
    return ((lane % 8) ^ codes_swizzle(8 * (unsigned)q + lane / 8)) << 4;
}
template <bool EDGE>
__host__ __device__ inline unsigned codes_offset(unsigned lane_row, unsigned lane_chunk, int q, int cb, unsigned last_row, unsigned last_chunk) {
    unsigned row = lane_row + 8 * (unsigned)q * (unsigned)cb, at = lane_chunk;
    if (EDGE) { row = row < last_row ? row : last_row; at = at < last_chunk ? at : last_chunk; }
    return row + at;
}

// EDGE = false: every tile has MT rows that exist (the last one starts at N - MT and repeats rows of the tile before it, with the same
// results) and rows are whole lines.  EDGE = true: fewer train rows than a tile, or rows that end inside a line.
// A line is one block without a branch: the compiler moves matrix instructions past a branch to where their results are used, behind
// all the requests (and spills what it has to keep).  So the copies go on behind the last line (they repeat it, into slots that are not
// read any more), and the step to the next checkpoint is made of selections.
template <class Sh, bool EDGE>
__global__ void __launch_bounds__(64 * Sh::NW, Sh::NW / 4)
score_codes_kernel(ScoreArgs a, CodesPrep w, int64_t ttiles, int vtiles) {
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
    const int trow = wave / WX * 32 * WR, vcol = wave % WX * 32 * WC;                // this wavefront's corner inside the tile
    const int64_t row0 = EDGE || tt * MT + MT <= a.N ? tt * MT : a.N - MT;
    for (int i = tid; i < MT; i += 64 * NW) s_rowmax[i] = 0u;
    const unsigned lds0 = (unsigned)(uintptr_t)((__attribute__((address_space(3))) unsigned char *)smem);

    // ---- copies: TU of a line of train rows, VU of half a line's validation rows (linear) per wavefront; past the end of the
    // validation side a wavefront repeats its last copy, so that all count the same number
    const int nst = w.nst, T = a.C * nst;                 // lines per row, and of all checkpoints
    const int over = nst * 128 - w.cb;                    // bytes of the last line past the end of a train row
    const unsigned last_row = EDGE ? (unsigned)((a.N - 1 - row0 < MT ? a.N - 1 - row0 : MT) * w.cb) : 0u;
    const int q0 = wave * TU, v0 = wave * VU < VCP ? wave * VU : VCP - 1;
    const unsigned lane_row = codes_lane_row((unsigned)lane, w.cb);
    unsigned lane_chunk[2];                               // of copies of even and odd distance from q0
#pragma unroll
    for (int e = 0; e < 2; ++e) lane_chunk[e] = codes_lane_chunk((unsigned)lane, q0 + e) + (EDGE ? 0u : lane_row);
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
            const unsigned last_chunk = t_s == nst - 1 ? (unsigned)(112 - over) : 112u;
            global_to_lds16(tb, codes_offset<true>(lane_row, lane_chunk[u & 1], q, w.cb, last_row, last_chunk), lds);
        } else {
            global_to_lds16(tb + (unsigned)(q * 8 * w.cb), lane_chunk[u & 1], lds);
        }
    };
    auto copy_val = [&](int u) {
        const int q = v0 + u < VCP ? v0 + u : VCP - 1;
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

    // ---- operands.  Train: the lane (row l32, half) takes chunk 2 * (K step of the line) + half; validation: 16 + 8 bytes at
    // [K step of the half line][half][row].
    const unsigned a_lane = (unsigned)(l32 * 128) + ((half ^ codes_swizzle((unsigned)l32)) << 4), a_base = (unsigned)(trow * 128);
    const unsigned b_lane = (unsigned)((half * VT + vcol + l32) * 8);
    i32x4 fa[WR];
    i32x8 ua[WR], fb[WC];
    auto load_a = [&](int b, int slot, int ks) {
        fa[b] = *(const i32x4 *)(smem + (a_lane ^ (unsigned)(ks << 5)) + (unsigned)(slot * TBYTES) + a_base + b * 4096);
    };
    auto load_b = [&](int c, int slot, int ks) {
        const unsigned char *p = smem + NT * TBYTES + (unsigned)(slot * VBYTES);
        const i32x4 x = *(const i32x4 *)(p + b_lane * 2 + (2 * ks * VT + 32 * c) * 16);
        const i32x2 y = *(const i32x2 *)(p + b_lane + Sh::V16 + (2 * ks * VT + 32 * c) * 8);
        fb[c] = __builtin_shufflevector(x, __builtin_shufflevector(y, y, 0, 1, -1, -1), 0, 1, 2, 3, 4, 5, -1, -1);
    };
    uint32_t flip0 = 0x08208208u, flip1 = 0x82082082u, flip2 = 0x20820820u;     // bit 3 of every number; kept in vector registers
    asm volatile("" : "+v"(flip0), "+v"(flip1), "+v"(flip2));
    int low[3];
    auto unpack = [&](int b, int h) {                     // a train fragment in two steps (the second puts it together)
        int o[3];
        fp6_train((uint32_t)fa[b][2 * h], (uint32_t)fa[b][2 * h + 1], flip0, flip1, flip2, h == 0 ? low : o);
        if (h == 1) {
            const i32x4 x = {low[0], low[1], low[2], o[0]};
            const i32x2 y = {o[1], o[2]};
            ua[b] = __builtin_shufflevector(x, __builtin_shufflevector(y, y, 0, 1, -1, -1), 0, 1, 2, 3, 4, 5, -1, -1);
        }
    };
    auto pin = []() { __builtin_amdgcn_sched_barrier(0); };   // keeps the order below

    float facc[WR][WC][16];
#pragma unroll
    for (int b = 0; b < WR; ++b)
#pragma unroll
        for (int c = 0; c < WC; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) facc[b][c][v] = 0.0f;

    // The first requests, in the order in which the loop goes on: at the barrier of half line h validation rows h + 3, behind them
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
    wait_vmcnt<2 * VU + TU>();                            // the first line and half line
    __syncthreads();
#pragma unroll
    for (int c = 0; c < WC; ++c) load_b(c, 0, 0);
#pragma unroll
    for (int b = 0; b < WR; ++b) load_a(b, 0, 0);
    unpack(0, 0); unpack(0, 1);
    int tslot = 0, vslot = 0;
    for (int ci = 0; ci < a.C; ++ci) {
        f32x16 acc[WR][WC];
#pragma unroll
        for (int c = 0; c < WC; ++c) {
            const float start = w.vbias[ci * w.Mp + vt * VT + vcol + 32 * c + l32];
#pragma unroll
            for (int b = 0; b < WR; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[b][c][v] = start;
        }
        for (int s = 0; s < nst; ++s) {
            const int tnext = tslot + 1 == NT ? 0 : tslot + 1;
            // Column block by column block, all row blocks: a validation fragment is requested again (for the next K step) as soon
            // as its last instruction is issued, several instructions before its next use; block 0 of the train rows is unpacked
            // between its last instruction and the next K step's first, the others each behind the one before.  (Behind the very last line:
            // whatever the rings hold, not used.)
#pragma unroll
            for (int k4 = 0; k4 < 4; ++k4) {                                    // K steps of the line: h = k4 / 2 the half line
                const int h = k4 >> 1;
                const bool last = k4 & 1;                                       // of its half line
                const int vnext = vslot + 1 == NV ? 0 : vslot + 1;
                const int rt = k4 == 3 ? tnext : tslot, rv = last ? vnext : vslot, ra = (k4 + 1) & 3, rb = last ? 0 : 1;   // the next K step's
                constexpr int I = WR * WC, K0 = 1;                               // instructions of a K step; the last one's before the barrier
#pragma unroll
                for (int i = 0; i < I; ++i) {
                    const int c = i / WR, b = i % WR;
                    pin();
                    acc[b][c] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(ua[b], fb[c], acc[b][c], 2, 2, 0, 127, 0, 127);
                    asm volatile("" : "+v"(acc[b][c]) :: "memory");              // stays here, between the reads before and behind it
                    pin();
                    if (i + 1 < WR) { unpack(i + 1, 0); unpack(i + 1, 1); }
                    if (last && i == K0) {
                        // this wavefront's reads of the half line (and line) have returned and its share of the next one has
                        // landed; the barrier says so of all wavefronts.  Younger: validation rows of the half line after it and,
                        // with three lines in the ring or none needed now, a line of train rows.
                        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                        if (h == 0 || NT == 3) wait_vmcnt<VU + TU>(); else wait_vmcnt<VU>();
                        __builtin_amdgcn_s_barrier();
                        asm volatile("" ::: "memory");
                        pin();
                        load_a(0, rt, ra);
                    }
                    if (i < WR && !(last && i < K0)) load_a(i, rt, ra);          // (unpacked by now)
                    if (b == WR - 1) load_b(c, rv, rb);
                    if (i >= I - 2) { pin(); unpack(0, i - (I - 2)); }
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
        tile_add_checkpoint<WR, WC>(acc, 64.0f, a.tr[ci], row0 + trow, a.N, w.vw + ci * w.Mp + vt * VT + vcol, facc);      // acc = D / 64
    }
    wait_vmcnt<0>();                                      // no copy is under way when the workgroup gives its LDS back
    tile_finish<WR, WC>(a, facc, row0, trow, vt * VT + vcol, s_rowmax);
    if (a.score) {
        __syncthreads();
        for (int i = tid; i < MT; i += 64 * NW)
            if (row0 + i < a.N && s_rowmax[i] != 0u) atomicMax(&w.smax[row0 + i], s_rowmax[i]);
    }
}

// Padded validation rows: at most M + 191 (a shape that pads more does not serve the call).
constexpr int kCodesPad = 191;
static void codes_offsets(int64_t N, int32_t M, int64_t cb, int C, size_t *off_vw, size_t *off_bias, size_t *off_smax, size_t *total) {
    auto up = [](size_t o) { return (o + 255) & ~(size_t)255; };
    const size_t rows = (size_t)(M + kCodesPad);
    *off_vw = up((size_t)C * rows * (size_t)((cb + 127) / 128 * 192));
    *off_bias = up(*off_vw + (size_t)C * rows * 4);
    *off_smax = up(*off_bias + (size_t)C * rows * 4);
    *total = *off_smax + (size_t)(N > 0 ? N : 1) * 4;
}
size_t codes_workspace(int64_t N, int32_t M, int64_t row_bytes, int C) {
    size_t v, b, s, t;
    codes_offsets(N, M, row_bytes, C, &v, &b, &s, &t);
    return t;
}

typedef CodesShape<2, 3, 4, 2, 3> Codes256x192;
typedef CodesShape<2, 2, 4, 2, 3> Codes256x128;
typedef CodesShape<2, 3, 8, 1, 2> Codes512x96;
typedef CodesShape<3, 2, 2, 4, 3> Codes192x256;

template <class Sh>
static qless_status launch_codes_shape(const ScoreArgs &a, CodesPrep w, hipStream_t st) {
    QLESS_LDS_KERNEL((score_codes_kernel<Sh, false>), Sh::LDS);
    QLESS_LDS_KERNEL((score_codes_kernel<Sh, true>), Sh::LDS);
    w.Mp = (a.M + Sh::VT - 1) / Sh::VT * Sh::VT;
    if (w.Mp > a.M + kCodesPad) return QLESS_ERR_UNSUPPORTED;
    const int vtiles = w.Mp / Sh::VT;
    const int64_t ttiles = (a.N + Sh::MT - 1) / Sh::MT, grid = 8 * (int64_t)vtiles * ((ttiles + 7) / 8);
    if (grid > 0x7FFFFFFF) return QLESS_ERR_UNSUPPORTED;
    const unsigned rows32 = (unsigned)(w.Mp / 32);
    unsigned parts = (512 + rows32 * (unsigned)a.C - 1) / (rows32 * (unsigned)a.C);      // two workgroups per compute unit
    if (parts > (unsigned)w.nst) parts = (unsigned)w.nst;
    hipLaunchKernelGGL(score_codes_prepare_kernel, dim3(rows32, (unsigned)a.C, parts), dim3(256), 0, st, a, w, Sh::VT);
    if (a.N >= Sh::MT && w.cb % 128 == 0)
        hipLaunchKernelGGL((score_codes_kernel<Sh, false>), dim3((unsigned)grid), dim3(64 * Sh::NW), Sh::LDS, st, a, w, ttiles, vtiles);
    else
        hipLaunchKernelGGL((score_codes_kernel<Sh, true>), dim3((unsigned)grid), dim3(64 * Sh::NW), Sh::LDS, st, a, w, ttiles, vtiles);
    return QLESS_OK;
}

// The shape with the fastest rounds, those of the XCD that gets the most train tiles (all validation tiles of a train tile run on
// one).  A round takes so many microseconds per line of the rows, per checkpoint (its epilogue) and whatever its length, fitted to 389 random calls (N = 1500 ..
// 270 000, M = 65 .. 1024, k = 64 .. 16384, C = 1 .. 6), each run with every shape: the chosen one is 0.3 % behind the fastest (without the 192 x 256 tiles and with one price per padded
// pair 1.2 %, 32 % at most: 11 979 x 985 x 5, k = 5952 in tiles of 256 rows is 36 workgroups on most XCDs, a second round, 349 us; in 192 x 256 tiles 32, 254 us).
struct CodesPrice { int mt, vt; double line, checkpoint, round; };
constexpr int kCodesShapes = 4;
constexpr CodesPrice kCodesPrice[kCodesShapes] = {{256, 192, 1.55, 2.2, 8.3}, {256, 128, 1.34, 1.4, 5.7}, {512, 96, 1.76, 2.1, 8.4}, {192, 256, 1.65, 3.1, 8.3}};
static double codes_round(int shape, int lines, int C) { return C * (lines * kCodesPrice[shape].line + kCodesPrice[shape].checkpoint) + kCodesPrice[shape].round; }
static int choose_codes_shape(int64_t N, int32_t M, int lines, int C) {
    const int64_t cus = (compute_units() + 7) / 8;                   // per XCD
    int best = 0;
    double least = 0;
    for (int i = 0; i < kCodesShapes; ++i) {
        const CodesPrice &s = kCodesPrice[i];
        if ((M + s.vt - 1) / s.vt * s.vt > M + kCodesPad) continue;      // (the first shape never pads more)
        const int64_t tiles = ((N + s.mt - 1) / s.mt + 7) / 8 * ((M + s.vt - 1) / s.vt);
        const double us = (double)((tiles + cus - 1) / cus) * codes_round(i, lines, C);
        if (i == 0 || us < least) { best = i; least = us; }
    }
    return best;
}

qless_status launch_codes(const ScoreArgs &a, void *ws, hipStream_t st, int shape) {
    CodesPrep w{};
    w.cb = a.k / 2;
    w.nst = (w.cb + 127) / 128;
    size_t off_vw, off_bias, off_smax, total;
    codes_offsets(a.N, a.M, w.cb, a.C, &off_vw, &off_bias, &off_smax, &total);
    unsigned char *base = (unsigned char *)ws;
    w.vexp = base; w.vw = (float *)(base + off_vw); w.vbias = (float *)(base + off_bias); w.smax = (unsigned int *)(base + off_smax);
    qless_status rc;
    switch (shape < 0 ? choose_codes_shape(a.N, a.M, w.nst, a.C) : shape) {
        case 0: rc = launch_codes_shape<Codes256x192>(a, w, st); break;
        case 1: rc = launch_codes_shape<Codes256x128>(a, w, st); break;
        case 2: rc = launch_codes_shape<Codes512x96>(a, w, st); break;
        default: rc = launch_codes_shape<Codes192x256>(a, w, st); break;
    }
    if (rc != QLESS_OK) return rc;
    if (a.score) launch_score_finish(w.smax, a.N, a.score, st);
    return launch_status();
}

template <class Sh, bool EDGE>
static int64_t codes_reach_edge(int64_t N, int cb) {
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
                    const int64_t end = row0 * cb + (int64_t)s * 128 + 16 +
                        codes_offset<EDGE>(codes_lane_row(lane, cb), codes_lane_chunk(lane, q), q, cb, last_row, (unsigned)(112 - (s == nst - 1 ? over : 0)));
                    most = end > most ? end : most;
                }
    }
    return most;
}
template <class Sh>
static int64_t codes_reach(int64_t N, int cb) {
    return N >= Sh::MT && cb % 128 == 0 ? codes_reach_edge<Sh, false>(N, cb) : codes_reach_edge<Sh, true>(N, cb);
}

}  // namespace qless

// For the tests, host only: the end of the last byte of the train rows that any copy of tile shape `shape` (of the table above) reads (at most
// N * row_bytes), from the kernel's own address arithmetic; the shape that a call takes, and the price of a round of a shape.
extern "C" int64_t qless_internal_codes_reach(int64_t N, int row_bytes, int shape) {
    using namespace qless;
    switch (shape) {
        case 0: return codes_reach<Codes256x192>(N, row_bytes);
        case 1: return codes_reach<Codes256x128>(N, row_bytes);
        case 2: return codes_reach<Codes512x96>(N, row_bytes);
        default: return codes_reach<Codes192x256>(N, row_bytes);
    }
}
extern "C" int qless_internal_codes_shape(int64_t N, int32_t M, int64_t row_bytes, int C) { return qless::choose_codes_shape(N, M, (int)((row_bytes + 127) / 128), C); }
extern "C" double qless_internal_codes_round(int shape, int64_t row_bytes, int C) { return qless::codes_round(shape, (int)((row_bytes + 127) / 128), C); }
