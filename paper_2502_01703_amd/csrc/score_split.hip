// qless_score / qless_score16 on few pairs: the rows a batch just added, small datastores.
//
// There the other kernels are bound by latency: a handful of workgroups walk all checkpoints and all of K one stage after
// the other (64 rows x 512 validation vectors x 4 checkpoints, k = 8192, 1 bit: 8 workgroups, 86 us).  Here K and the
// checkpoints are shared out as well: a workgroup forms the dot products of a 64 x 64 tile of pairs over a part of one
// checkpoint's K, its four wavefronts a quarter of that part each (operands straight from memory into registers, four
// chunks in flight, no barrier), joins them in LDS and writes them to the workspace; a second kernel adds
// the parts and applies the fp32 epilogue in checkpoint order.  Integer parts add exactly (sign and ternary codes as FP4
// products: integers below 2^24 in fp32); bfloat16 rows' fp32 parts are added in a fixed order.
#include <type_traits>
#include "score.h"

namespace qless {

typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(8))) int i32x8;
typedef __attribute__((ext_vector_type(16))) int i32x16;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;

constexpr int kSplitWaves = 4, kSplitTile = 64;

template <int BITS> struct SplitAcc { typedef i32x16 type; };
template <> struct SplitAcc<1> { typedef f32x16 type; };
template <> struct SplitAcc<2> { typedef f32x16 type; };
template <> struct SplitAcc<16> { typedef f32x16 type; };

// 32 bytes of every row (16 of each bit plane for the ternary codes): the lane (row, half) holds 16-byte chunk 2 t + half
template <int BITS> struct SplitChunk { uint4 w[BITS == 2 ? 2 : 1]; };

// 32 codes of a chunk word as four dwords of FP4 codes (nibble n of dword j: code 4 n + 3 - j); zero where `live` is 0
__device__ inline i32x8 split_fp4(uint32_t sg, uint32_t nz, bool ternary, int live) {
    i32x8 r = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t mag = ternary ? ((j >= 2 ? nz << (j - 2) : nz >> (2 - j)) & 0x22222222u) : 0x22222222u;
        r[j] = (int)((((sg << j) & 0x88888888u) | mag) & (uint32_t)live);
    }
    return r;
}
__device__ inline uint32_t word_of(const uint4 &v, int j) { return j == 0 ? v.x : j == 1 ? v.y : j == 2 ? v.z : v.w; }

// live_lo, live_hi: -1 or 0 for the chunk's first and second eight bytes
template <int BITS>
__device__ inline void split_products(const SplitChunk<BITS> (&t)[2], const SplitChunk<BITS> (&v)[2], int live_lo, int live_hi,
                                      typename SplitAcc<BITS>::type (&acc)[2][2]) {
    if constexpr (BITS <= 2) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            i32x8 a[2], b[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                a[e] = split_fp4(word_of(t[e].w[BITS - 1], j), word_of(t[e].w[0], j), BITS == 2, -1);
                b[e] = split_fp4(word_of(v[e].w[BITS - 1], j), word_of(v[e].w[0], j), BITS == 2, j < 2 ? live_lo : live_hi);
            }
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int y = 0; y < 2; ++y)
                    acc[x][y] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a[x], b[y], acc[x][y], 4, 4, 0, 127, 0, 127);
        }
    } else {
        constexpr int SUB = BITS == 4 ? 2 : 1;
        auto part = [](const uint4 &w, int sub, int keep) {
            if (BITS != 4) return i32x4{(int)w.x & keep, (int)w.y & keep, (int)w.z & keep, (int)w.w & keep};
            const uint32_t px = sub ? w.z : w.x, py = sub ? w.w : w.y;                  // 16 q of 16 codes
            return i32x4{(int)((px << 4) & 0xF0F0F0F0u) & keep, (int)(px & 0xF0F0F0F0u) & keep,
                         (int)((py << 4) & 0xF0F0F0F0u) & keep, (int)(py & 0xF0F0F0F0u) & keep};
        };
#pragma unroll
        for (int sub = 0; sub < SUB; ++sub) {
            i32x4 a[2], b[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) { a[e] = part(t[e].w[0], sub, live_lo); b[e] = part(v[e].w[0], sub, live_lo); }
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int y = 0; y < 2; ++y) {
                    if constexpr (BITS == 16)
                        acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[x]), __builtin_bit_cast(bf16x8, b[y]), acc[x][y], 0, 0, 0);
                    else
                        acc[x][y] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[x], b[y], acc[x][y], 0, 0, 0);
                }
        }
    }
}

// grid (train tiles, val tiles, C * parts); part p of a checkpoint takes chunk steps [p * per, (p + 1) * per).  Two wavefronts
// per SIMD, so that two workgroups share a compute unit as split_plan counts them (left free, the compiler took 198 + 64 registers for
// the ternary codes, one workgroup: 256 x 256 x 4, k = 16384 26.9 us, now 23.8).
template <int BITS>
__global__ void __launch_bounds__(64 * kSplitWaves, 2)
score_split_kernel(ScoreArgs a, int cb, int parts, int per, uint32_t *planes) {
    constexpr int DEPTH = BITS == 2 ? 2 : 4, NPL = BITS == 2 ? 2 : 1;
    extern __shared__ __attribute__((aligned(16))) uint32_t join[];             // [wavefront][64 rows][64 columns]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int64_t row0 = (int64_t)blockIdx.x * kSplitTile;
    const int v0 = (int)blockIdx.y * kSplitTile, ci = (int)blockIdx.z / parts, part = (int)blockIdx.z % parts;
    const int plane = cb / NPL, nchunks = (plane + 15) / 16, steps = (nchunks + 1) / 2;  // 16-byte chunks per row (and plane)
    // this wavefront's quarter of the part's steps
    const int p0 = part * per, p1 = p0 + per < steps ? p0 + per : steps;
    const int q = (p1 - p0 + kSplitWaves - 1) / kSplitWaves;
    const int t0 = p0 + wave * q, t1 = t0 + q < p1 ? t0 + q : p1;
    const unsigned char *tp[2], *vp[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int64_t r = row0 + 32 * e + l32;
        const int c = v0 + 32 * e + l32;
        tp[e] = a.tc[ci] + (r < a.N ? r : a.N - 1) * cb;                        // rows past the end: masked by the second kernel
        vp[e] = a.vc[ci] + (int64_t)(c < a.M ? c : a.M - 1) * cb;
    }
    typename SplitAcc<BITS>::type acc[2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[x][y][v] = 0;
    SplitChunk<BITS> ts[DEPTH][2], vs[DEPTH][2];
    auto fetch = [&](int t, int slot) {
        // chunks that reach past the row (or plane) end re-read its last 16 bytes; what is not theirs is multiplied by 0.  Rows
        // are multiples of 8 bytes: the last chunk may own the second half of those 16 bytes only.
        const int at = 16 * (2 * t + half), off = at + 16 <= plane ? at : plane - 16;
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int p = 0; p < NPL; ++p) {
                ts[slot][e].w[p] = *(const uint4 *)(tp[e] + p * plane + off);
                vs[slot][e].w[p] = *(const uint4 *)(vp[e] + p * plane + off);
            }
    };
#pragma unroll
    for (int u = 0; u < DEPTH; ++u)
        if (t0 + u < t1) fetch(t0 + u, u);
    for (int t = t0; t < t1; t += DEPTH) {                                      // wave-uniform
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
            if (t + u >= t1) break;
            const int at = 16 * (2 * (t + u) + half), live_lo = at + 16 <= plane ? -1 : 0, live_hi = at < plane ? -1 : 0;
            SplitChunk<BITS> x[2] = {ts[u][0], ts[u][1]}, y[2] = {vs[u][0], vs[u][1]};
            if (t + u + DEPTH < t1) fetch(t + u + DEPTH, u);
            split_products<BITS>(x, y, live_lo, live_hi, acc);
        }
    }
    // acc[x][y][v]: train row 32 x + 8 (v / 4) + 4 half + v % 4, val column 32 y + l32
    uint32_t *mine = join + wave * (kSplitTile * kSplitTile);
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = 32 * x + 8 * (v >> 2) + 4 * half + (v & 3);
                uint32_t d;
                if constexpr (BITS == 16) d = __float_as_uint(acc[x][y][v]);
                else if constexpr (BITS == 4) d = (uint32_t)((int)acc[x][y][v] >> 8);
                else d = (uint32_t)(int)acc[x][y][v];
                mine[r * kSplitTile + 32 * y + l32] = d;
            }
    __syncthreads();
    uint32_t *out = planes + (size_t)blockIdx.z * (size_t)a.N * (size_t)a.M;
    for (int i = tid; i < kSplitTile * kSplitTile; i += 64 * kSplitWaves) {
        const int64_t r = row0 + i / kSplitTile;
        const int c = v0 + i % kSplitTile;
        if (r >= a.N || c >= a.M) continue;
        uint32_t d = join[i];
#pragma unroll
        for (int w = 1; w < kSplitWaves; ++w) {
            const uint32_t o = join[w * (kSplitTile * kSplitTile) + i];
            d = BITS == 16 ? __float_as_uint(__uint_as_float(d) + __uint_as_float(o)) : d + o;
        }
        out[(size_t)r * a.M + c] = d;
    }
}

// U checkpoints of one pair's influence: the parts of their sums go out together (two at a time, four of one or two checkpoints), all requested before
// the first is used; the additions stay in the order of the parts and of the checkpoints.
template <int U>
__device__ inline float split_group(const ScoreArgs &a, int c0, int parts, const uint32_t *p, size_t plane, int bf16, int64_t z, int c, float acc) {
    constexpr int V = U > 2 ? 2 : 4;
    float rt[U], wv[U], D[U];
    uint32_t d[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        rt[u] = a.tr[c0 + u] ? a.tr[c0 + u][z] : 1.0f;
        wv[u] = bf16 ? a.eta[c0 + u] : __fmul_rn(a.eta[c0 + u], a.vr[c0 + u][c]);
        d[u] = p[(size_t)u * parts * plane];
        D[u] = __uint_as_float(d[u]);
    }
    auto add = [&](int s, auto n) {
        constexpr int W = decltype(n)::value;
        uint32_t t[U][W];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int v = 0; v < W; ++v) t[u][v] = p[((size_t)u * parts + s + v) * plane];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int v = 0; v < W; ++v) {
                D[u] = __fadd_rn(D[u], __uint_as_float(t[u][v]));
                d[u] += t[u][v];
            }
    };
    int s = 1;
    for (; s + V <= parts; s += V) add(s, std::integral_constant<int, V>());
    for (; s < parts; ++s) add(s, std::integral_constant<int, 1>());
#pragma unroll
    for (int u = 0; u < U; ++u) acc = __fadd_rn(acc, __fmul_rn(__fmul_rn(bf16 ? D[u] : (float)(int)d[u], rt[u]), wv[u]));
    return acc;
}
// One pair's influence: four checkpoints at a time, the rest together (four loads each whatever is left took 2179 x 737, one
// checkpoint, k = 3264, 1 bit from 24 to 34 us)
template <bool ONE>
__device__ inline float split_pair(const ScoreArgs &a, int parts, const uint32_t *planes, size_t plane, int bf16, int64_t z, int c) {
    const uint32_t *p = planes + (size_t)z * a.M + c;
    if (ONE) return split_group<1>(a, 0, parts, p, plane, bf16, z, c, 0.0f);
    const size_t step = (size_t)parts * plane;
    float acc = 0.0f;
    int c0 = 0;
    for (; c0 + 4 <= a.C; c0 += 4) acc = split_group<4>(a, c0, parts, p + c0 * step, plane, bf16, z, c, acc);
    const int rest = a.C - c0;
    p += c0 * step;
    if (rest == 3) return split_group<3>(a, c0, parts, p, plane, bf16, z, c, acc);
    if (rest == 2) return split_group<2>(a, c0, parts, p, plane, bf16, z, c, acc);
    return rest ? split_group<1>(a, c0, parts, p, plane, bf16, z, c, acc) : acc;
}

// The parts of every pair added, the epilogue of Eq.(6),(7) in checkpoint order, row maximum.  Few rows: what it takes is the time of its loads
// one behind the other, so they go out together and every thread has one column (up to 1024): with a walk of 256 threads over the
// columns and one load at a time 64 x 512 x 4 took 13.5 us at 1 bit, so 5.9 (with the sums 8 bits 47 -> 21 us, bfloat16 51 -> 26).  Many rows
// keep the chip full by themselves, and 256 threads to a row start and end faster (8503 x 764 x 2, k = 960, 1 bit 72 us with 768 threads, 52 with 256;
// 200 x 800 x 5, k = 4096, 8 bits 37 and 44): the line is the wavefronts that the chip holds.  Eight wavefronts per SIMD either way (16453 x 453 x 2,
// k = 2368 111 us with four, 99 with eight).  ROWS train rows per workgroup of four wavefronts: one each (up to 64 columns), or
// all wavefronts on one row (with a row per wavefront 1800 x 145 x 4 took 27 us instead of 22).  ONE: a single checkpoint, whose calls that makes 5 % faster.
template <int ROWS, bool ONE>
__global__ void __launch_bounds__(ROWS == 1 ? 1024 : 256, 8)
score_split_finish_kernel(ScoreArgs a, int parts, const uint32_t *planes, int bf16, float none) {
    __shared__ float wave_best[16];
    const int wave = threadIdx.x >> 6;
    const int64_t z = ROWS == 1 ? blockIdx.x : (int64_t)blockIdx.x * 4 + wave;
    const size_t plane = (size_t)a.N * (size_t)a.M;
    if (ROWS > 1 && z >= a.N) return;                // (no barrier below then)
    float best = neg_inf();
    for (int c = ROWS == 1 ? threadIdx.x : threadIdx.x & 63; c < a.M; c += ROWS == 1 ? blockDim.x : 64) {
        const float acc = split_pair<ONE>(a, parts, planes, plane, bf16, z, c);
        if (a.full) a.full[z * a.M + c] = acc;
        best = fmaxf(best, acc);
    }
    if (!a.score) return;                            // uniform
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) best = fmaxf(best, __shfl_xor(best, o, 64));
    if (ROWS == 1) {
        if ((threadIdx.x & 63) == 0) wave_best[wave] = best;
        __syncthreads();
        if (threadIdx.x) return;
        for (int w = 1; w < (int)(blockDim.x >> 6); ++w) best = fmaxf(best, wave_best[w]);
    }
    if ((threadIdx.x & 63) == 0) a.score[z] = best > neg_inf() ? best : none;
}
template <bool ONE>
static void launch_split_finish_of(const ScoreArgs &a, int parts, const uint32_t *planes, bool bf16, float none, hipStream_t st) {
    if (a.M <= 64 && a.N >= 1024) {
        hipLaunchKernelGGL((score_split_finish_kernel<4, ONE>), dim3((unsigned)((a.N + 3) / 4)), dim3(256), 0, st, a, parts, planes, bf16, none);
        return;
    }
    const int64_t waves = (a.M + 63) / 64;
    const int64_t most = a.N * waves <= 32 * (int64_t)compute_units() ? 16 : 4;
    hipLaunchKernelGGL((score_split_finish_kernel<1, ONE>), dim3((unsigned)a.N), dim3((unsigned)(64 * (waves < most ? waves : most))), 0, st, a, parts, planes, bf16, none);
}
qless_status launch_split_finish(const ScoreArgs &a, int parts, const uint32_t *planes, bool bf16, float none, hipStream_t st) {
    if (a.C == 1) launch_split_finish_of<true>(a, parts, planes, bf16, none, st);
    else launch_split_finish_of<false>(a, parts, planes, bf16, none, st);
    return launch_status();
}

struct SplitPlan { int parts, per; size_t bytes; };
static SplitPlan split_plan(int64_t N, int32_t M, int64_t cb, int bits, int C) {
    SplitPlan p{};
    const int64_t tiles = ((N + kSplitTile - 1) / kSplitTile) * ((M + kSplitTile - 1) / kSplitTile) * C;
    const int64_t chunks = ((bits == 2 ? cb / 2 : cb) + 15) / 16, steps = (chunks + 1) / 2;
    int64_t want = (512 + tiles - 1) / tiles;                      // two workgroups per compute unit
    const int64_t most = (steps + 2 * kSplitWaves - 1) / (2 * kSplitWaves);     // at least two steps per wavefront
    if (want > most) want = most;
    if (want < 1) want = 1;
    p.per = (int)((steps + want - 1) / want);
    p.parts = (int)((steps + p.per - 1) / p.per);
    p.bytes = (size_t)C * p.parts * (size_t)N * (size_t)M * 4;
    return p;
}
size_t split_workspace(int64_t N, int32_t M, int64_t row_bytes, int bits, int C) { return split_plan(N, M, row_bytes, bits, C).bytes; }

template <int BITS>
static void launch_split_bits(const ScoreArgs &a, int cb, const SplitPlan &p, uint32_t *ws, hipStream_t st) {
    constexpr int lds = kSplitWaves * kSplitTile * kSplitTile * 4;
    QLESS_LDS_KERNEL((score_split_kernel<BITS>), lds);
    const dim3 grid((unsigned)((a.N + kSplitTile - 1) / kSplitTile), (unsigned)((a.M + kSplitTile - 1) / kSplitTile), (unsigned)(a.C * p.parts));
    hipLaunchKernelGGL((score_split_kernel<BITS>), grid, dim3(64 * kSplitWaves), lds, st, a, cb, p.parts, p.per, ws);
}
qless_status launch_split(const ScoreArgs &a, int bits, float none, void *ws, hipStream_t st) {
    const int cb = bits == 16 ? a.k : a.k * bits / 8;
    const SplitPlan p = split_plan(a.N, a.M, cb, bits, a.C);
    uint32_t *w = (uint32_t *)ws;
    switch (bits) {
        case 16: launch_split_bits<16>(a, cb, p, w, st); break;
        case 8: launch_split_bits<8>(a, cb, p, w, st); break;
        case 4: launch_split_bits<4>(a, cb, p, w, st); break;
        case 2: launch_split_bits<2>(a, cb, p, w, st); break;
        default: launch_split_bits<1>(a, cb, p, w, st); break;
    }
    return launch_split_finish(a, p.parts, w, bits == 16, none, st);
}

// The other paths walk their stages one after the other whatever the number of pairs (measured with few pairs: about a
// microsecond per stage of a tile or slice of a stream); here the operands of every tile are read again, at about 6 TB/s
// out of the L2 caches, and the parts are written and read once.  Both in microseconds; the line is drawn where this path is
// estimated a tenth faster (8192 x 256 x 4, k = 16384: 1 bit 121 against 166 us, 2 bits 200 against 177, 8 bits 619 against 522).
bool use_split(int64_t N, int32_t M, int64_t row_bytes, int bits, int C) {
    double stages;
    if (bits <= 2 && row_bytes / bits % 16 != 0) stages = (M <= 8 ? 0.3 : (double)((M + 63) / 64)) * (double)((row_bytes / bits + 63) / 64) * 3.2;   // popcounts
    else if (bits <= 2 && M <= 16) stages = (double)((row_bytes / bits + 127) / 128) * 1.2;              // one wavefront's slices
    else if (bits == 1 && M <= 192 && row_bytes % 64 == 0) stages = (double)((M + 63) / 64) * (double)(row_bytes / 64) * 1.2;
    else if ((bits == 4 && M <= 96) || (bits == 8 && M <= 32)) stages = (double)(row_bytes / 64) * (bits == 4 ? 0.8 : 0.62);
    else if (bits == 1) stages = (double)((row_bytes + 63) / 64) * 1.4;
    else if (bits == 16) stages = (double)((row_bytes + 127) / 128) * 0.9;
    else stages = (double)((row_bytes + 127) / 128) * (bits == 2 ? 1.5 : (bits == 4 ? 1.3 : 0.75));
    const double there = 0.9 * (5 + stages * C);
    const double tiles = (double)((N + kSplitTile - 1) / kSplitTile) * (double)((M + kSplitTile - 1) / kSplitTile);
    // (the second kernel takes a workgroup per row: 1.2 ns each)
    double here = 12 + tiles * kSplitTile * kSplitTile * (double)row_bytes / 32 / 6e6 * C + (double)N * 1.2e-3;
    if (here >= there || tiles > 65535) return false;       // (a grid takes 65535 val tiles)
    const SplitPlan p = split_plan(N, M, row_bytes, bits, C);
    here += (double)p.bytes * 2 / 4e6;
    return here < there && p.bytes <= ((size_t)256 << 20) && C * p.parts <= 65535;
}

}  // namespace qless
