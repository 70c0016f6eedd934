// qless_score against more than 64 validation vectors: the tile kernel of the 1- and 2-bit codes, as FP4 products.
//
// The codes {-1, 0, +1} are FP4 (E2M1) numbers and v_mfma_scale_f32_32x32x64_f8f6f4 multiplies 64 of them per lane pair; products and sums
// are integers (or halves that the operands' weights make integers) far below 2^24, hence exact in fp32.
//   1 bit   the train side takes its sign bits s where they are: dword j of a word's 32 codes is (w & 0x88888888) | 0x22222222 (+-1)
//           for j = 0 and w & (0x88888888 >> j) = 2 s, s, s / 2 for j = 1, 2, 3; the pre-pass stores the validation code b of those
//           positions as -b, -2 b, -4 b, so that every such product is -2 s b = a b - b, and the accumulator starts from the sum of b over
//           them.  Four vector-ALU operations per 32 codes.
//   2 bits  the train side leaves its "non-zero" bit of dwords 1, 2, 3 in place (2, 1, 1 / 2) and moves the sign: twelve operations; the
//           validation magnitudes are 1 / 2, 1, 2 there.
// Nibble n of dword j is code 4 n + 3 - j of the word on both sides.  Bound: the matrix instructions alone (random operands) take 2.75 of the
// 3.2 ms at N = 270 000, M = 1024, k = 8192, C = 4, 1 bit, at the clock that the card's power limit leaves them; the kernel before (256 x 128
// tiles, one ring, a barrier before a stage's reads) kept them busy 47 % of the cycles.
//   * A wavefront owns 2 x 3 or 3 x 2 accumulators (2 x 2 where that pads less): with the fp32 checkpoint sums next to them 192 of its 256
//     registers.  An unpacked train fragment feeds two or three matrix instructions, a validation fragment three or two.
//   * Two rings, filled asynchronously, as in score_codes.hip: 64 bytes (512 codes) of every train row (and bit plane) of the tile in a
//     ring of two or three, 256 codes of every validation row, expanded by the pre-pass to FP4 in the order [K step][half][row], in a
//     ring of three.  Every stage of 256 codes requests the same number of copies: half a piece of train rows and one stage of
//     validation rows.
//   * One barrier per stage, behind the second matrix instruction of its last K step; a validation fragment is requested again as soon as its
//     last instruction is issued, a train fragment is unpacked for the next K step as soon as its last instruction is.
//   * SPLIT: a workgroup forms the dot products of one checkpoint (or a part of its K) only and writes them to the workspace, where
//     score_split_finish_kernel joins them: a small datastore's few tiles then fill the chip (8192 x 256, k = 16384, 2 bits: 32 tiles of
//     256 x 128 for four checkpoints each).
// Measured, same card, k = 8192, C = 4 (256 x 128 and 512 x 96 tiles, 128 x 64 for small stores -> now): N = 270 000, M = 1024 1 bit 3.91 -> 3.20 ms,
// 2 bits 4.84 -> 3.60; M = 285 1.34 -> 0.97 and 1.92 -> 1.34; 65536 x 192, 2 bits 313 -> 181 us; 8192 x 256, k = 16384, 2 bits 158 -> 86 us.
#include "score_tile.h"

namespace qless {

typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(8))) int i32x8;

struct Fp4Prep {                               // workspace views (device pointers)
    unsigned char *vexp;                       // [C][val tile][stage][4 K steps][2 halves][VT rows][16 bytes]
    float *vw, *vbias;                         // [C][Mp] eta * rnorm', 1 bit: start of the accumulators
    unsigned int *smax;                        // [N] order-preserving keys of the row maxima
    int32_t Mp, cb, nst;                       // padded validation rows, bytes and 512-code pieces per train row
};
// SPLIT: pieces [part * per, (part + 1) * per) of a checkpoint per workgroup, planes [C * parts][N][M]
struct Fp4Parts { int parts, per; uint32_t *planes; };

template <int BITS_, int WR_, int WC_, int WY_, int WX_, int NT_>
struct Fp4Shape {
    static constexpr int BITS = BITS_, WR = WR_, WC = WC_, WY = WY_, WX = WX_, NT = NT_, NV = 3, NW = WY * WX;
    static constexpr int MT = 32 * WR * WY, VT = 32 * WC * WX;
    static constexpr int PBYTES = MT * 64, TBYTES = PBYTES * BITS, VBYTES = VT * 128;     // a piece of train rows, a stage of validation rows
    static constexpr int TCP = TBYTES / 1024, VCP = VBYTES / 1024;                          // 1 KB copies
    static constexpr int TP = (TCP / 2 + NW - 1) / NW, VU = (VCP + NW - 1) / NW;           // per wavefront and stage
    static constexpr int LDS = NT * TBYTES + NV * VBYTES;
    static_assert(TCP % 2 == 0 && VBYTES % 1024 == 0 && PBYTES % 1024 == 0, "whole copies");
    static_assert(WR >= 2 && (NT == 2 || NT == 3) && LDS + 4 * MT <= (int)kLdsPerCU, "the rings and the row maxima fit in LDS");
    static_assert(2 * VU + TP < 64, "vmcnt is a 6-bit counter");
};

// grid (32 padded validation rows, checkpoint, part of the row): a thread takes one row's words j, j + 8, .. of the part.  The first part also
// sums its rows' codes, the first checkpoint's workgroups clear the row-maximum keys.
template <int BITS>
__global__ void __launch_bounds__(256)
score_fp4_prepare_kernel(ScoreArgs a, Fp4Prep w, int VT) {
    __shared__ int part_sum[8][32];
    const int ci = blockIdx.y, rl = threadIdx.x & 31, j = threadIdx.x >> 5, row = (int)blockIdx.x * 32 + rl, r = row % VT;
    unsigned char *dst = w.vexp + ((size_t)ci * w.Mp + row - r) * (size_t)w.nst * 256;
    const unsigned char *src = a.vc[ci] + (int64_t)(row < a.M ? row : 0) * w.cb;
    const int words = a.k / 32, per = (2 * w.nst + (int)gridDim.z - 1) / (int)gridDim.z * 8, t0 = (int)blockIdx.z * per;
    for (int t = t0 + j; t < t0 + per && t < w.nst * 16; t += 8) {                  // word t: stage t / 8, half t % 8 / 4, K step t % 4
        uint32_t d[4] = {0, 0, 0, 0};
        if (row < a.M && t < words) {
            const uint32_t sg = ((const uint32_t *)(src + (BITS == 2 ? a.k / 8 : 0)))[t];
            const uint32_t nz = BITS == 2 ? ((const uint32_t *)src)[t] : 0u;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t s = (sg >> (3 - q)) & 0x11111111u;
                if (BITS == 2) {
                    const uint32_t x = (nz >> (3 - q)) & 0x11111111u;
                    d[q] = x * (q == 1 ? 1u : (q == 3 ? 4u : 2u)) | ((x & s) << 3);
                } else {
                    d[q] = (q == 3 ? 0x66666666u : (q == 2 ? 0x44444444u : 0x22222222u)) | ((q == 0 ? s : s ^ 0x11111111u) << 3);
                }
            }
        }
        *(uint4 *)(dst + (size_t)(t >> 3) * VT * 128 + ((2 * (t & 3) + ((t >> 2) & 1)) * VT + r) * 16) = make_uint4(d[0], d[1], d[2], d[3]);
    }
    if (blockIdx.z == 0) {                                                      // uniform
        int sum = 0;
        if (BITS == 1 && row < a.M)
            for (int t = j; t < words; t += 8) sum += 24 - 2 * (int)__popc(((const uint32_t *)src)[t] & 0x77777777u);
        part_sum[j][rl] = sum;
        __syncthreads();
        if (j == 0) {
#pragma unroll
            for (int q = 1; q < 8; ++q) sum += part_sum[q][rl];
            w.vw[ci * w.Mp + row] = row < a.M ? __fmul_rn(a.eta[ci], a.vr[ci][row]) : 0.0f;
            w.vbias[ci * w.Mp + row] = (float)sum;
        }
    }
    if (ci == 0 && w.smax) {
        const int64_t groups = (int64_t)gridDim.x * gridDim.z, g = (int64_t)blockIdx.z * gridDim.x + blockIdx.x;
        const int64_t share = (a.N + groups - 1) / groups, lo = g * share;
        for (int64_t i = lo + threadIdx.x; i < lo + share && i < a.N; i += 256) w.smax[i] = 0u;
    }
}

// Where the copies of train rows read, in bytes from the tile's first row (and the piece's 64 bytes into it): copy q takes rows
// 16 (q % (MT / 16)) + lane / 4 of plane q / (MT / 16), of each the 16-byte chunk (lane % 4) ^ ((row / 4) % 4): 16 consecutive rows read together
// use all 64 banks.  EDGE: rows past `last_row` re-read that one (masked later), chunks past `last_chunk` bytes re-read that one
// (the validation numbers there are zero).
template <int MT, bool EDGE>
__host__ __device__ inline unsigned fp4_offset(unsigned lane, int q, int cb, int plane_bytes, unsigned last_row, unsigned last_chunk) {
    unsigned row = (lane >> 2) * (unsigned)cb + 16u * (unsigned)(q % (MT / 16)) * (unsigned)cb, at = ((lane & 3) ^ ((lane >> 4) & 3)) << 4;
    if (EDGE) { row = row < last_row ? row : last_row; at = at < last_chunk ? at : last_chunk; }
    return row + (unsigned)(q / (MT / 16) * plane_bytes) + at;
}

// EDGE and the straight-line stage: see score_codes_kernel.
template <class Sh, bool EDGE, bool SPLIT>
__global__ void __launch_bounds__(64 * Sh::NW, Sh::NW / 4)
score_fp4_kernel(ScoreArgs a, Fp4Prep w, int64_t ttiles, int vtiles, Fp4Parts sp) {
    constexpr int BITS = Sh::BITS, WR = Sh::WR, WC = Sh::WC, WX = Sh::WX, NT = Sh::NT, NV = Sh::NV, NW = Sh::NW, MT = Sh::MT, VT = Sh::VT;
    constexpr int PBYTES = Sh::PBYTES, TBYTES = Sh::TBYTES, VBYTES = Sh::VBYTES, TCP = Sh::TCP, VCP = Sh::VCP, TP = Sh::TP, VU = Sh::VU;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];        // [NT][planes][MT][64], [NV][VBYTES]
    __shared__ unsigned int s_rowmax[SPLIT ? 1 : MT];
    // XCD-aware decode: the vtiles (SPLIT: and checkpoints and parts, validation tiles first) of one train tile get ids 8 apart
    const int64_t id = blockIdx.x, jj = id >> 3;
    const int per_tile = SPLIT ? vtiles * a.C * sp.parts : vtiles;
    const int sub = (int)(jj % per_tile), vt = sub % vtiles;
    const int64_t tt = (jj / per_tile) * 8 + (id & 7);
    if (tt >= ttiles) return;
    const int plane = SPLIT ? sub / vtiles : 0;                                 // ci * parts + part
    const int c_first = SPLIT ? plane / sp.parts : 0, c_count = SPLIT ? 1 : a.C;
    const int s_first = SPLIT ? plane % sp.parts * sp.per : 0, s_end = SPLIT && s_first + sp.per < w.nst ? s_first + sp.per : w.nst;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int trow = wave / WX * 32 * WR, vcol = wave % WX * 32 * WC;           // this wavefront's corner inside the tile
    const int64_t row0 = EDGE || tt * MT + MT <= a.N ? tt * MT : a.N - MT;
    if (!SPLIT)
        for (int i = tid; i < MT; i += 64 * NW) s_rowmax[i] = 0u;
    const unsigned lds0 = (unsigned)(uintptr_t)((__attribute__((address_space(3))) unsigned char *)smem);

    // ---- copies per stage and wavefront: TP of train rows (the first or second half of a piece) and VU of validation rows (linear); past
    // the end a wavefront repeats the last one, so that all count the same number
    const int nst = s_end - s_first, T = c_count * nst;   // pieces per row, and of all checkpoints
    const int plane_bytes = w.cb / BITS;
    const unsigned last_row = EDGE ? (unsigned)((a.N - 1 - row0 < MT ? a.N - 1 - row0 : MT) * w.cb) : 0u;
    const unsigned val_lane = (unsigned)(lane * 16), train_lane = fp4_offset<MT, false>((unsigned)lane, 0, w.cb, plane_bytes, 0, 0);
    // the checkpoints' train rows: lane i holds the first byte of the tile's first row of checkpoint i
    const uint64_t tile_row = (uint64_t)(a.tc[lane < a.C ? lane : 0] + row0 * w.cb + s_first * 64);
    auto train_of = [&](int ci) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)tile_row, ci);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(tile_row >> 32), ci);
        return (const unsigned char *)(((uint64_t)hi << 32) | lo);
    };
    int t_it = 0, t_ci = c_first, t_s = 0, t_slot = 0;    // the piece of train rows that is being requested
    int v_it = 0, v_s = 0, v_slot = 0;                    // and the next stage of validation rows
    const unsigned char *tb = train_of(c_first);
    const unsigned char *vb = w.vexp + ((size_t)(c_first * vtiles + vt) * (2 * w.nst) + 2 * s_first) * VBYTES;
    const size_t v_wrap = (size_t)(vtiles - 1) * (2 * w.nst) * VBYTES;
    auto copy_train = [&](int part, int u) {
        const int at = wave * TP + u, q = part * (TCP / 2) + (TCP / 2 % (NW * TP) == 0 || at < TCP / 2 ? at : TCP / 2 - 1);
        const unsigned lds = lds0 + (unsigned)(t_slot * TBYTES + q * 1024);
        if (EDGE) {
            const int left = plane_bytes - (s_first + t_s) * 64;                // bytes of the plane from this piece on
            const unsigned last_chunk = left < 64 ? (unsigned)(left - 16) : 48u;
            unsigned l = (unsigned)lane;                  // opaque: formed here, not kept in a register per copy
            asm volatile("" : "+v"(l));
            global_to_lds16(tb, fp4_offset<MT, true>(l, q, w.cb, plane_bytes, last_row, last_chunk), lds);
        } else {
            global_to_lds16(tb + (unsigned)(16 * (q % (MT / 16)) * w.cb + q / (MT / 16) * plane_bytes), train_lane, lds);
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
        tb = wrap ? first : tb + (end ? 0 : 64);
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

    // ---- operands.  Train: the lane (row l32, half) takes chunk 2 * (stage of the piece) + half of its row and plane, word ks in K step ks;
    // validation: 16 bytes at [K step][half][row].
    const unsigned a_lane = (unsigned)(l32 * 64) + ((half ^ ((l32 >> 2) & 3)) << 4), a_base = (unsigned)(trow * 64);
    const unsigned b_lane = (unsigned)((half * VT + vcol + l32) * 16);
    i32x4 fa[WR][BITS], fb[WC];
    i32x8 ua[WR];
    auto load_a = [&](int b, int slot, int h) {
#pragma unroll
        for (int p = 0; p < BITS; ++p)
            fa[b][p] = *(const i32x4 *)(smem + (a_lane ^ (unsigned)(h << 5)) + (unsigned)(slot * TBYTES) + a_base + b * 2048 + p * PBYTES);
    };
    auto load_b = [&](int c, int slot, int ks) {
        fb[c] = *(const i32x4 *)(smem + NT * TBYTES + (unsigned)(slot * VBYTES) + b_lane + (2 * ks * VT + 32 * c) * 16);
    };
    uint32_t one = 0x22222222u;                           // eight FP4 codes of +1.0, kept in a vector register
    asm volatile("" : "+v"(one));
    auto unpack = [&](int b, int ks) {
        const uint32_t sg = (uint32_t)fa[b][BITS - 1][ks], nz = (uint32_t)fa[b][0][ks];
        i32x4 d;
        if (BITS == 1)
            d = i32x4{(int)((sg & 0x88888888u) | one), (int)(sg & 0x44444444u), (int)(sg & 0x22222222u), (int)(sg & 0x11111111u)};
        else
            d = i32x4{(int)((sg & 0x88888888u) | ((nz >> 2) & 0x22222222u)), (int)(((sg << 1) & 0x88888888u) | (nz & 0x44444444u)),
                      (int)(((sg << 2) & 0x88888888u) | (nz & 0x22222222u)), (int)(((sg << 3) & 0x88888888u) | (nz & 0x11111111u))};
        ua[b] = __builtin_shufflevector(d, d, 0, 1, 2, 3, -1, -1, -1, -1);
    };
    auto pin = []() { __builtin_amdgcn_sched_barrier(0); };   // keeps the order below

    float facc[WR][WC][16];
#pragma unroll
    for (int b = 0; b < WR; ++b)
#pragma unroll
        for (int c = 0; c < WC; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) facc[b][c][v] = 0.0f;

    // The first requests, in the order in which the loop goes on: at the barrier of stage g half a piece of train rows, behind it the
    // validation rows of stage g + 3.
    for (int i = 0; i < NT - 1; ++i) {
#pragma unroll
        for (int part = 0; part < 2; ++part)
#pragma unroll
            for (int u = 0; u < TP; ++u) copy_train(part, u);
        next_train();
    }
    for (int i = 0; i < NV; ++i) {
        if (i == NV - 1) {
#pragma unroll
            for (int u = 0; u < TP; ++u) copy_train(0, u);
        }
#pragma unroll
        for (int u = 0; u < VU; ++u) copy_val(u);
        next_val();
    }
    wait_vmcnt<2 * VU + TP>();                            // the first piece and stage
    __syncthreads();
#pragma unroll
    for (int c = 0; c < WC; ++c) load_b(c, 0, 0);
#pragma unroll
    for (int b = 0; b < WR; ++b) load_a(b, 0, 0);
#pragma unroll
    for (int b = 0; b < WR; ++b) unpack(b, 0);
    int tslot = 0, vslot = 0;
    for (int ci = c_first; ci < c_first + c_count; ++ci) {
        f32x16 acc[WR][WC];
#pragma unroll
        for (int c = 0; c < WC; ++c) {
            const float start = BITS == 1 && s_first == 0 ? w.vbias[ci * w.Mp + vt * VT + vcol + 32 * c + l32] : 0.0f;
#pragma unroll
            for (int b = 0; b < WR; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[b][c][v] = start;
        }
        for (int s = 0; s < nst; ++s) {
            const int tnext = tslot + 1 == NT ? 0 : tslot + 1;
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) {                                    // K steps of the piece: stage h, K step ks
                const int h = kk >> 2, ks = kk & 3, vnext = vslot + 1 == NV ? 0 : vslot + 1;
                const bool last = ks == 3;
                constexpr int I = WR * WC, K0 = 1;                              // instructions of a K step; the last one's before the barrier
#pragma unroll
                for (int i = 0; i < I; ++i) {
                    const int c = i / WR, b = i % WR;
                    pin();
                    const i32x8 vf = __builtin_shufflevector(fb[c], fb[c], 0, 1, 2, 3, -1, -1, -1, -1);
                    acc[b][c] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(ua[b], vf, acc[b][c], 4, 4, 0, 127, 0, 127);
                    asm volatile("" : "+v"(acc[b][c]) :: "memory");              // stays here, between the reads before and behind it
                    pin();
                    if (last && i == K0) {
                        // this wavefront's reads of the stage have returned and its share of the next one has landed; the barrier says
                        // so of all wavefronts.  Younger: what the barrier before requested (a ring of two pieces: its validation rows).
                        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                        if (h == 0 || NT == 3) wait_vmcnt<VU + TP>(); else wait_vmcnt<VU>();
                        __builtin_amdgcn_s_barrier();
                        asm volatile("" ::: "memory");
                        pin();
#pragma unroll
                        for (int q = 0; q < WR; ++q) load_a(q, h == 1 ? tnext : tslot, h ^ 1);
                    }
                    if (b == WR - 1) load_b(c, last ? vnext : vslot, (ks + 1) & 3);
                    if (c == WC - 1) { pin(); unpack(b, (ks + 1) & 3); }
                    if (last && i >= K0) {
#pragma unroll
                        for (int u = 0; u < TP + VU; ++u)                       // spread over the instructions behind the barrier
                            if (u * (I - K0) / (TP + VU) == i - K0) { if (u < TP) copy_train(h ^ 1, u); else copy_val(u - TP); }
                    }
                }
                if (last) { next_val(); vslot = vnext; if (h == 0) next_train(); }
            }
            tslot = tnext;
        }
        if constexpr (SPLIT) {
            uint32_t *out = sp.planes + (size_t)plane * (size_t)a.N * (size_t)a.M;
#pragma unroll
            for (int b = 0; b < WR; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int64_t r = row0 + trow + 32 * b + 8 * (v >> 2) + 4 * half + (v & 3);
#pragma unroll
                    for (int c = 0; c < WC; ++c) {
                        const int col = vt * VT + vcol + 32 * c + l32;
                        if (r < a.N && col < a.M) out[(size_t)r * a.M + col] = (uint32_t)(int)acc[b][c][v];
                    }
                }
        } else {
            tile_add_checkpoint<WR, WC>(acc, 1.0f, a.tr[ci], row0 + trow, a.N, w.vw + ci * w.Mp + vt * VT + vcol, facc);
        }
    }
    wait_vmcnt<0>();                                      // no copy is under way when the workgroup gives its LDS back
    if constexpr (!SPLIT) {
        tile_finish<WR, WC>(a, facc, row0, trow, vt * VT + vcol, s_rowmax);
        if (a.score) {
            __syncthreads();
            for (int i = tid; i < MT; i += 64 * NW)
                if (row0 + i < a.N && s_rowmax[i] != 0u) atomicMax(&w.smax[row0 + i], s_rowmax[i]);
        }
    }
}

// ---- shapes.  Microseconds of a round with a tile on every compute unit: per piece (512 codes), per checkpoint (its epilogue) and whatever its length.  These and
// the other figures of fp4_plan and use_fp4 are fitted to 760 random calls (N = 256 .. 270 000, M = 65 .. 1024, k = 128 .. 16384, C = 1 .. 6), each run with every shape and
// number of parts and, where the store is small, with the 128 x 64 tiles: the chosen kernel is 0.4 % (1 bit) and 0.9 % (2 bits) behind the fastest on small stores, the
// chosen shape and parts 0.5 and 0.4 % in all; on another 118 small stores 1.4 %, and none of these more than 3 % slower than before this kernel (with prices from one k and C and
// none for an epilogue 32 and 9 %, 2.1 and 2.9 %, and a tenth of the small stores slower).
struct Fp4Cost { int bits, mt, vt; double piece_us, checkpoint_us, round_us; };
constexpr int kFp4Shapes = 7;
constexpr Fp4Cost kFp4Cost[kFp4Shapes] = {{1, 384, 128, 1.85, 2.35, 6.5}, {1, 512, 96, 1.85, 1.55, 6.5}, {1, 256, 192, 1.80, 1.60, 6.5}, {1, 256, 128, 1.38, 1.25, 5.3},
                                          {2, 256, 192, 2.08, 2.00, 6.8}, {2, 256, 128, 1.76, 1.30, 5.6}, {2, 384, 128, 2.34, 3.00, 7.4}};
template <class Sh> constexpr bool fp4_is(const Fp4Cost &c) { return Sh::BITS == c.bits && Sh::MT == c.mt && Sh::VT == c.vt; }
typedef Fp4Shape<1, 3, 2, 4, 2, 3> Fp4Signs384x128;
typedef Fp4Shape<1, 2, 3, 8, 1, 3> Fp4Signs512x96;
typedef Fp4Shape<1, 2, 3, 4, 2, 3> Fp4Signs256x192;
typedef Fp4Shape<1, 2, 2, 4, 2, 3> Fp4Signs256x128;
typedef Fp4Shape<2, 2, 3, 4, 2, 2> Fp4Ternary256x192;
typedef Fp4Shape<2, 2, 2, 4, 2, 3> Fp4Ternary256x128;
typedef Fp4Shape<2, 3, 2, 4, 2, 2> Fp4Ternary384x128;
static_assert(fp4_is<Fp4Signs384x128>(kFp4Cost[0]) && fp4_is<Fp4Signs512x96>(kFp4Cost[1]) && fp4_is<Fp4Signs256x192>(kFp4Cost[2]) &&
              fp4_is<Fp4Signs256x128>(kFp4Cost[3]) && fp4_is<Fp4Ternary256x192>(kFp4Cost[4]) && fp4_is<Fp4Ternary256x128>(kFp4Cost[5]) &&
              fp4_is<Fp4Ternary384x128>(kFp4Cost[6]), "the table's order is launch_fp4's");

// The shape and, where the call leaves compute units idle, the number of workgroups that share a tile's checkpoints and K (parts per
// checkpoint; 0: one workgroup walks all of them).  A round is the tiles of the XCD that gets the most (all validation tiles of a train tile run
// on one); sharing costs the planes' way through memory and a kernel that joins them.
struct Fp4Plan { int shape, parts, per; double us; };
static Fp4Plan fp4_plan(int64_t N, int32_t M, int32_t k, int bits, int C, bool share) {
    const int64_t cus = (compute_units() + 7) / 8;                   // per XCD
    const int nst = (k + 511) / 512;
    Fp4Plan best{-1, 0, nst, 0};
    for (int i = 0; i < kFp4Shapes; ++i) {
        const Fp4Cost &c = kFp4Cost[i];
        if (c.bits != bits) continue;
        const int64_t tiles = ((N + c.mt - 1) / c.mt + 7) / 8 * ((M + c.vt - 1) / c.vt);
        int last = -1;
        for (int want = 0; want <= (share ? 8 : 0); ++want) {
            const int per = want ? (nst + want - 1) / want : nst, parts = want ? (nst + per - 1) / per : 0;
            if (parts == last) continue;
            last = parts;
            const int64_t wgs = tiles * (parts ? (int64_t)parts * C : 1);
            const double round = parts ? per * c.piece_us * 1.08 + c.round_us - 1.0 : C * (per * c.piece_us + c.checkpoint_us) + c.round_us;
            const double bytes = (double)C * parts * (double)N * (double)M * 4;
            double us = (double)((wgs + cus - 1) / cus) * round;
            if (parts) us += 3.5 + 0.5e-6 * (bytes < 20e6 ? bytes : 10e6 + 0.5 * bytes) + (double)N * 0.2e-3;
            if (bytes > (double)((size_t)256 << 20)) continue;
            if (best.shape < 0 || us < best.us) best = Fp4Plan{i, parts, per, us};
        }
    }
    return best;
}

// Padded validation rows: at most M + 191.
static void fp4_offsets(int64_t N, int32_t M, int32_t k, int C, int parts, size_t *off_vw, size_t *off_bias, size_t *off_smax, size_t *off_planes, size_t *total) {
    auto up = [](size_t o) { return (o + 255) & ~(size_t)255; };
    const size_t rows = (size_t)(M + 191);
    *off_vw = up((size_t)C * rows * (size_t)((k + 511) / 512 * 256));
    *off_bias = up(*off_vw + (size_t)C * rows * 4);
    *off_smax = up(*off_bias + (size_t)C * rows * 4);
    *off_planes = up(*off_smax + (size_t)(N > 0 ? N : 1) * 4);
    *total = *off_planes + (size_t)C * parts * (size_t)N * (size_t)M * 4;
}
size_t fp4_workspace(int64_t N, int32_t M, int32_t k, int bits, int C, bool share) {
    size_t v, b, s, p, t;
    fp4_offsets(N, M, k, C, share ? fp4_plan(N, M, k, bits, C, true).parts : 0, &v, &b, &s, &p, &t);
    return t;
}

template <class Sh>
static qless_status launch_fp4_shape(const ScoreArgs &a, Fp4Prep w, const Fp4Parts &sp, hipStream_t st) {
    QLESS_LDS_KERNEL((score_fp4_kernel<Sh, false, false>), Sh::LDS);
    QLESS_LDS_KERNEL((score_fp4_kernel<Sh, true, false>), Sh::LDS);
    QLESS_LDS_KERNEL((score_fp4_kernel<Sh, false, true>), Sh::LDS);
    QLESS_LDS_KERNEL((score_fp4_kernel<Sh, true, true>), Sh::LDS);
    w.Mp = (a.M + Sh::VT - 1) / Sh::VT * Sh::VT;
    const int vtiles = w.Mp / Sh::VT;
    const int64_t ttiles = (a.N + Sh::MT - 1) / Sh::MT, grid = 8 * (int64_t)vtiles * ((ttiles + 7) / 8) * (sp.parts ? a.C * sp.parts : 1);
    if (grid > 0x7FFFFFFF) return QLESS_ERR_UNSUPPORTED;
    const unsigned rows32 = (unsigned)(w.Mp / 32);
    unsigned parts = (512 + rows32 * (unsigned)a.C - 1) / (rows32 * (unsigned)a.C);      // two workgroups per compute unit
    if (parts > 2 * (unsigned)w.nst) parts = 2 * (unsigned)w.nst;
    hipLaunchKernelGGL((score_fp4_prepare_kernel<Sh::BITS>), dim3(rows32, (unsigned)a.C, parts), dim3(256), 0, st, a, w, Sh::VT);
    const bool edge = !(a.N >= Sh::MT && a.k % 512 == 0);
    const dim3 g((unsigned)grid), t(64 * Sh::NW);
    if (sp.parts) {
        if (edge) hipLaunchKernelGGL((score_fp4_kernel<Sh, true, true>), g, t, Sh::LDS, st, a, w, ttiles, vtiles, sp);
        else hipLaunchKernelGGL((score_fp4_kernel<Sh, false, true>), g, t, Sh::LDS, st, a, w, ttiles, vtiles, sp);
    } else {
        if (edge) hipLaunchKernelGGL((score_fp4_kernel<Sh, true, false>), g, t, Sh::LDS, st, a, w, ttiles, vtiles, sp);
        else hipLaunchKernelGGL((score_fp4_kernel<Sh, false, false>), g, t, Sh::LDS, st, a, w, ttiles, vtiles, sp);
    }
    return QLESS_OK;
}

// The 128 x 64 tiles of a small datastore (few enough for the chip to hold all of them) take 9.2 us, 1.2 per piece of a workgroup with one of them on every
// compute unit, 1.4 to 1.6 with two on some or all, and an epilogue per checkpoint; this path 7.8 us and what its plan says (843 x 1024 x 6, k = 256, 1 bit 18.7 against
// 29.8 us, 3931 x 320 x 1, k = 4096 20.4 and 25.4; 2 bits 8192 x 256 x 4, k = 16384 158 and 86).
bool use_fp4(int64_t N, int32_t M, int32_t k, int bits, int C) {
    const int64_t cus = compute_units();
    if (((N + 255) / 256) * ((M + 127) / 128) * 2 > cus) return true;
    const int64_t tiles = ((N + 127) / 128) * ((M + 63) / 64);
    const double piece = tiles <= cus ? 1.2 : 1.4 + 0.2 * (tiles >= 2 * cus ? 1.0 : (double)(tiles - cus) / (double)cus);
    return fp4_plan(N, M, k, bits, C, true).us + 7.8 < 9.2 + C * ((k + 511) / 512 * piece + (bits == 1 ? 0.5 : 2.1));
}

static qless_status launch_fp4_plan(const ScoreArgs &a, int bits, const Fp4Plan &p, void *ws, hipStream_t st) {
    Fp4Prep w{};
    w.cb = a.k / 8 * bits;
    w.nst = (a.k + 511) / 512;
    size_t off_vw, off_bias, off_smax, off_planes, total;
    fp4_offsets(a.N, a.M, a.k, a.C, p.parts, &off_vw, &off_bias, &off_smax, &off_planes, &total);
    unsigned char *base = (unsigned char *)ws;
    w.vexp = base; w.vw = (float *)(base + off_vw); w.vbias = (float *)(base + off_bias); w.smax = p.parts ? nullptr : (unsigned int *)(base + off_smax);
    const Fp4Parts sp{p.parts, p.per, (uint32_t *)(base + off_planes)};
    qless_status rc;
    switch (p.shape) {
        case 0: rc = launch_fp4_shape<Fp4Signs384x128>(a, w, sp, st); break;
        case 1: rc = launch_fp4_shape<Fp4Signs512x96>(a, w, sp, st); break;
        case 2: rc = launch_fp4_shape<Fp4Signs256x192>(a, w, sp, st); break;
        case 3: rc = launch_fp4_shape<Fp4Signs256x128>(a, w, sp, st); break;
        case 4: rc = launch_fp4_shape<Fp4Ternary256x192>(a, w, sp, st); break;
        case 5: rc = launch_fp4_shape<Fp4Ternary256x128>(a, w, sp, st); break;
        default: rc = launch_fp4_shape<Fp4Ternary384x128>(a, w, sp, st); break;
    }
    if (rc != QLESS_OK) return rc;
    if (p.parts) return launch_split_finish(a, p.parts, sp.planes, false, nan_below_all(), st);
    if (a.score) launch_score_finish(w.smax, a.N, a.score, st);
    return launch_status();
}

qless_status launch_fp4(const ScoreArgs &a, int bits, void *ws, size_t ws_bytes, hipStream_t st) {
    // (a workspace laid out for a larger call may be too small for the planes: one workgroup walks all checkpoints then)
    return launch_fp4_plan(a, bits, fp4_plan(a.N, a.M, a.k, bits, a.C, ws_bytes >= fp4_workspace(a.N, a.M, a.k, bits, a.C, true)), ws, st);
}

size_t fp4_workspace_as(int64_t N, int32_t M, int32_t k, int C, int parts) {
    size_t v, b, s, p, t;
    fp4_offsets(N, M, k, C, parts, &v, &b, &s, &p, &t);
    return t;
}
qless_status launch_fp4_as(const ScoreArgs &a, int bits, int shape, int parts, void *ws, hipStream_t st) {
    const int nst = (a.k + 511) / 512, per = parts ? (nst + parts - 1) / parts : nst;
    if (shape < 0 || shape >= kFp4Shapes || kFp4Cost[shape].bits != bits || a.k % 128 != 0 || parts < 0 || (parts && (nst + per - 1) / per != parts)) return QLESS_ERR_UNSUPPORTED;
    return launch_fp4_plan(a, bits, Fp4Plan{shape, parts, per, 0}, ws, st);
}

}  // namespace qless

namespace qless {
template <class Sh, bool EDGE>
static int64_t fp4_reach_edge(int64_t N, int32_t k) {
    constexpr int MT = Sh::MT, BITS = Sh::BITS;
    const int plane_bytes = k / 8, cb = plane_bytes * BITS, nst = (k + 511) / 512;
    const int64_t ttiles = (N + MT - 1) / MT;
    int64_t most = 0;
    for (int64_t tt = ttiles > 3 ? ttiles - 3 : 0; tt < ttiles; ++tt) {
        const int64_t row0 = EDGE || tt * MT + MT <= N ? tt * MT : N - MT;
        const unsigned last_row = (unsigned)((N - 1 - row0 < MT ? N - 1 - row0 : MT) * cb);
        for (int s = 0; s < nst; ++s) {
            const int left = plane_bytes - s * 64;
            for (int q = 0; q < Sh::TCP; ++q)
                for (unsigned lane = 0; lane < 64; ++lane) {
                    const int64_t end = row0 * cb + (int64_t)s * 64 + 16 +
                        fp4_offset<MT, EDGE>(lane, q, cb, plane_bytes, last_row, left < 64 ? (unsigned)(left - 16) : 48u);
                    most = end > most ? end : most;
                }
        }
    }
    return most;
}
template <class Sh> static int64_t fp4_reach(int64_t N, int32_t k) {
    return N >= Sh::MT && k % 512 == 0 ? fp4_reach_edge<Sh, false>(N, k) : fp4_reach_edge<Sh, true>(N, k);
}
}  // namespace qless

// For the tests, host only: the end of the last byte of the train rows that any copy of the shape reads (at most N rows of k codes), from the
// kernel's own address arithmetic; and a call's plan: {train rows, validation rows of a tile, parts per checkpoint, pieces per part, use_fp4}.
extern "C" int64_t qless_internal_fp4_reach(int64_t N, int32_t k, int shape) {
    using namespace qless;
    switch (shape) {
        case 0: return fp4_reach<Fp4Signs384x128>(N, k);
        case 1: return fp4_reach<Fp4Signs512x96>(N, k);
        case 2: return fp4_reach<Fp4Signs256x192>(N, k);
        case 3: return fp4_reach<Fp4Signs256x128>(N, k);
        case 4: return fp4_reach<Fp4Ternary256x192>(N, k);
        case 5: return fp4_reach<Fp4Ternary256x128>(N, k);
        default: return fp4_reach<Fp4Ternary384x128>(N, k);
    }
}
extern "C" void qless_internal_fp4_plan(int64_t N, int32_t M, int32_t k, int bits, int C, int share, int *out) {
    const qless::Fp4Plan p = qless::fp4_plan(N, M, k, bits, C, share != 0);
    out[0] = qless::kFp4Cost[p.shape].mt; out[1] = qless::kFp4Cost[p.shape].vt; out[2] = p.parts; out[3] = p.per;
    out[4] = qless::use_fp4(N, M, k, bits, C) && !qless::use_split(N, M, (int64_t)k / 8 * bits, bits, C);
}
