// qless_project: P = R G^T-style random projection (paper Eq.(1); matrix families of Sec. 2.4)
// as a bf16 MFMA GEMM whose B operand (the random matrix) is generated in registers.
//
// Shape of the problem: M-dimension = batch rows n (small), N-dimension = k projected
// coordinates, contraction over the gradient dimension d (huge).  One workgroup of 8 waves
// owns a 64 (rows) x 1024 (coordinates) output tile for one slice of d; each wave owns
// 64 x 128 of it as 2 x 4 MFMA 32x32 accumulators.  Gaussian projections of batches that
// fill 128-row tiles take 128 x 512 tiles (4 x 2 accumulators per wave): every
// generated fragment of the random operand then feeds four matrix instructions instead of two.
// Other batches take tiles of 16, 32 or 48 rows on 16 x 16 matrix instructions (project_narrow_kernel);
// make_plans() chooses the shape and the number of d-slices by what they cost.  The gradient tile is
// staged through LDS; partial tiles of the d-slices go to the workspace and are summed in a fixed
// order by a second kernel, so results are run-to-run identical.
// Measured, before (64-row tiles for every batch) -> now: 16 x 2^19 bf16 -> 8192 326 -> 166 us, 32 x 2^20 637 -> 432 us,
// 1 x 2^20 623 -> 317 us; 37 x 1 000 017 at odd row offsets -> 4096 439 -> 293 us; 1024 x 16384 fp32 -> 512 42.6 -> 33.7 us.
//
// Random operand: lanes 0..31 of a wave take one 32-column word of R for their row m, lanes
// 32..63 the next word; the 32 sign bits of a word feed four MFMA K-steps of 8 columns each.
// Column c of a word reads hash bit 4*(c%8) + 3 - c/8, which is exactly what
// ((h << s) & 0x88888888) | 0x22222222 places in the sign position of eight FP4 (E2M1) codes
// of +-1.0 for K-step s; V_CVT_SCALEF32_PK_BF16_FP4 expands them to packed bf16 +-1.0, two
// elements per instruction.
#include <type_traits>
#include "common.h"

namespace qless {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kWaves = 8;
constexpr int kStageD = 128;                   // gradient columns per LDS stage
constexpr int kLdsStride = kStageD * 2 + 16;   // bytes per staged row (+16: conflict-free b128 reads)
// NB = 32-row blocks per workgroup tile (2 or 4); a wave owns NB x (8 / NB) accumulators
template <int NB> struct ProjShape {
    static_assert(NB == 2 || NB == 4, "64- or 128-row tiles");
    static constexpr int KB = 8 / NB;                   // 32-coordinate blocks per wave
    static constexpr int kTileRows = 32 * NB;           // batch rows per workgroup
    static constexpr int kWaveCols = 32 * KB;           // projected coordinates per wave
    static constexpr int kTileCols = kWaves * kWaveCols;   // 1024 or 512 per workgroup
    static constexpr int kStageBytes = kTileRows * kLdsStride;
    static constexpr int kDirectStageBytes = kTileRows * kStageD * 2;
};
// Tile shapes (rows x projected coordinates of a workgroup), how many workgroups a compute unit holds, microseconds a round costs
// whatever its length (the narrow 512-wide tiles join two groups' sums in LDS), and microseconds per 128 gradient columns with a
// workgroup on every slot of the chip for each kind of input: bf16, fp32 (converted while it is staged), Gaussian bf16 (bound by the
// table look-ups, which a fragment costs whatever it feeds), Gaussian fp32.  Fitted, with the two figures for a d-slice in
// make_plans, to 1950 random calls (n = 1 .. 1024, d = 512 .. 2^25, k = 64 .. 16384) that were each run with every shape, by the kernels before
// staged rows were requested without a branch and Gaussian look-ups pipelined: the chosen plan was 1.2 % behind the fastest one on average.  With the
// present kernels it is 2.6, 3.5, 2.9 and 3.3 % behind the best shape (150 random calls each).
enum ProjectTile { kTile128, kTile64, kTile48, kTile48x512, kTile32x512, kTile16x512, kTiles };
constexpr int kPlanKinds = 4;
struct TileCost { int rows, cols, per_cu; double fixed, stage[kPlanKinds]; };
constexpr TileCost kTileCost[kTiles] = {
    {128, 512, 1, 4.5, {2.45, 4.10, 4.50, 4.30}}, {64, 1024, 1, 4.5, {2.35, 3.25, 6.20, 5.00}},
    {48, 1024, 1, 5.5, {2.08, 2.78, 5.70, 5.10}}, {48, 512, 1, 8.0, {1.05, 1.76, 2.80, 2.70}},
    {32, 512, 1, 4.0, {0.93, 1.45, 2.48, 2.35}}, {16, 512, 2, 6.0, {1.13, 2.10, 3.90, 4.20}}};

struct ProjectPlan {
    int shape;
    int64_t ntiles, ktiles, nsplit, stages_per_split, slices, grid;
    size_t ws_bytes;
};

// The plans of the four kinds of input (bf16, fp32, Gaussian bf16, Gaussian fp32), in one pass: it runs on every call.
static int plan_kind(bool gauss, bool fp32) { return 2 * gauss + fp32; }
static void make_plans(int64_t n, int64_t d_len, int32_t k, ProjectPlan (&p)[kPlanKinds]) {
    for (ProjectPlan &q : p) q = ProjectPlan{};
    if (n <= 0 || d_len <= 0) return;
    const int64_t stages = (d_len + kStageD - 1) / kStageD;
    // Over the shapes and the numbers of d-slices: rounds of workgroups times a workgroup's columns, plus the round's fixed
    // share, plus the partial sums of the slices: their way through memory (written and read once, mostly in the caches) and a
    // share each of the kernel that adds them one after the other (without it 1 x 169 856 fp32 -> 320 took 443 slices: 45 us, 30 with
    // 222).  A (row tile, d-slice) runs on one XCD with all its column tiles, so the rounds are those of the XCD with the most
    // of them (416 x 2 020 480 -> 8256: 28 slices x 9 column tiles are 252 workgroups, but 36 of them on four of the XCDs: 19.3
    // against 15.6 ms).
    double least[kPlanKinds] = {0, 0, 0, 0};
    const double plane = (double)n * k * 8 / 6.2e6 + 0.07;
    for (int t = 0; t < kTiles; ++t) {
        const TileCost &c = kTileCost[t];
        const int64_t nt = (n + c.rows - 1) / c.rows, kt = (k + c.cols - 1) / c.cols, slots = 32 * c.per_cu;     // per XCD
        for (int rounds = 1; rounds <= 2; ++rounds) {
            int64_t w = rounds * slots / kt * 8 / nt;         // the most d-slices that fit these rounds
            if (w < 1) w = 1;
            if (w > stages) w = stages;
            const int64_t per = (stages + w - 1) / w, splits = (stages + per - 1) / per;
            const int64_t r = ((nt * splits + 7) / 8 * kt + slots - 1) / slots;
            const int64_t cols = t >= kTile48x512 ? (per + 1) / 2 * 2 : per;                  // two groups of wavefronts, alternate columns
            for (int v = 0; v < kPlanKinds; ++v) {
                const double us = (double)r * ((double)cols * c.stage[v] + c.fixed) + (double)splits * plane;
                if (least[v] == 0 || us < least[v]) { least[v] = us; p[v].shape = t; p[v].stages_per_split = per; p[v].nsplit = splits; }
            }
        }
    }
    for (ProjectPlan &q : p) {
        const TileCost &c = kTileCost[q.shape];
        q.ntiles = (n + c.rows - 1) / c.rows;
        q.ktiles = (k + c.cols - 1) / c.cols;
        q.slices = q.ntiles * q.nsplit;
        q.grid = q.ktiles * 8 * ((q.slices + 7) / 8);
        q.ws_bytes = (size_t)q.nsplit * (size_t)n * (size_t)k * sizeof(float);
    }
}

struct ProjectArgs {
    const void *G;
    float *ws;
    int64_t n, d_len, ldG;
    uint32_t wbase;          // d_offset / 32
    int32_t k;
    SeedKeys sk;
    int32_t ktiles, nsplit;
    int64_t slices, stages_per_split;
};

struct GaussTable { uint16_t v[256]; };

// How gradient tiles reach LDS: asynchronous copies (bf16, 16-byte aligned rows, a length of whole stages), or through
// registers (fp32, any alignment, any length).
enum ProjectInput { kDirectBf16, kStagedBf16, kStagedF32 };

// 16 bytes from any element boundary (a wide load has no alignment of its own to keep: rows at odd element offsets take as
// many load instructions as aligned ones; eight 2-byte loads instead made 37 x 1 000 017 bf16 -> 4096 30 % slower)
__device__ inline uint4 load_any(const void *p) {
    struct __attribute__((packed, aligned(2))) Bytes { uint4 v; };
    return ((const Bytes *)p)->v;
}
__device__ inline uint32_t pack2_bf16(float a, float b) {          // round to nearest even (v_cvt_pk_bf16_f32)
    bf16x2 r;
    r[0] = (__bf16)a; r[1] = (__bf16)b;
    return __builtin_bit_cast(uint32_t, r);
}

// Loads 8 consecutive gradient elements (row, col..col+7) as packed bf16; elements outside
// [0, n) x [0, c_end) read as zero.
template <ProjectInput IN>
__device__ inline uint4 load_chunk(const ProjectArgs &a, int64_t row, int64_t col, int64_t c_end) {
    uint4 v = make_uint4(0, 0, 0, 0);
    if (row >= a.n || col >= c_end) return v;
    if (IN == kStagedF32) {
        const float *p = (const float *)a.G + row * a.ldG + col;
        if (col + 8 <= c_end) {
            const uint4 lo = load_any(p), hi = load_any(p + 4);
            v.x = pack2_bf16(__uint_as_float(lo.x), __uint_as_float(lo.y)); v.y = pack2_bf16(__uint_as_float(lo.z), __uint_as_float(lo.w));
            v.z = pack2_bf16(__uint_as_float(hi.x), __uint_as_float(hi.y)); v.w = pack2_bf16(__uint_as_float(hi.z), __uint_as_float(hi.w));
        } else {
            float f[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) f[e] = col + e < c_end ? p[e] : 0.0f;
            v.x = pack2_bf16(f[0], f[1]); v.y = pack2_bf16(f[2], f[3]); v.z = pack2_bf16(f[4], f[5]); v.w = pack2_bf16(f[6], f[7]);
        }
    } else {
        const uint16_t *p = (const uint16_t *)a.G + row * a.ldG + col;
        if (col + 8 <= c_end) {
            v = load_any(p);
        } else {
            uint32_t h[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) h[e] = col + e < c_end ? p[e] : 0u;
            v.x = h[0] | (h[1] << 16); v.y = h[2] | (h[3] << 16); v.z = h[4] | (h[5] << 16); v.w = h[6] | (h[7] << 16);
        }
    }
    return v;
}

// The same eight elements as they are in memory, of a row and columns that exist (no branch), and packed where they are written to LDS
template <ProjectInput IN>
struct RawChunk {
    static constexpr int kElem = IN == kStagedF32 ? 4 : 2, kRegs = kElem / 2;
    uint4 v[kRegs];
    __device__ inline void load(const ProjectArgs &a, int64_t row, int64_t col) {
        const unsigned char *p = (const unsigned char *)a.G + (row * a.ldG + col) * kElem;
#pragma unroll
        for (int e = 0; e < kRegs; ++e) v[e] = load_any(p + 16 * e);
    }
    __device__ inline uint4 packed() const {
        if constexpr (kElem == 2) return v[0];
        else {
            auto two = [](uint32_t x, uint32_t y) { return pack2_bf16(__uint_as_float(x), __uint_as_float(y)); };
            return make_uint4(two(v[0].x, v[0].y), two(v[0].z, v[0].w), two(v[1].x, v[1].y), two(v[1].z, v[1].w));
        }
    }
};

union Frag { bf16x8 v; bf16x2 p[4]; uint4 u; uint32_t w[4]; uint16_t h[8]; };

// DIRECT: gradient tiles go global -> LDS asynchronously (no VGPR staging) into a ring of kRing
// unpadded, XOR-swizzled stage buffers, three stages ahead of the MFMAs; the other inputs are staged
// through registers into two padded buffers.
constexpr int kRing = 4;
constexpr int kProjectMaxLds = 160 * 1024;      // largest request of any shape (Gaussian, 128-row tiles)

// Gaussian table in LDS, at offset 0: entry i for lane l is the dword at byte 256 i + 4 l, holding the bfloat16 value in its
// upper half.  Every lane looks up in a column of its own, so no lookup conflicts with another, and the address
// is one byte permute of the hash (its byte above the lane's constant); the lower element of a pair is read as the
// dword's upper 16 bits and the two halves are joined by an OR.  Twelve vector-ALU operations per fragment beside the two
// hashes; 32 copies of 2 bytes, whose addresses took a shift, a mask and an addition, took more than twice that
// (128 x 2^18 -> 8192: 570 -> 516 us, 64 x 2^19 801 -> 675, 1 x 2^19 796 -> 457 with the 16-row tiles).
constexpr int kGaussBytes = 256 * 256;
__device__ inline void gauss_fill(unsigned char *tab, const GaussTable &gt) {       // (16 bytes a store: 128 x 896 -> 128 17.1 us with 4, now 14.3)
#pragma unroll
    for (int u = 0; u < kGaussBytes / 16 / (kWaves * 64); ++u) {
        const int i = (int)threadIdx.x + u * kWaves * 64;
        const uint32_t e = (uint32_t)gt.v[i >> 4] << 16;
        ((uint4 *)tab)[i] = make_uint4(e, e, e, e);
    }
}
// A fragment's eight entries come from two hash words, in three steps that are spread over three fragments: the words of fragment
// f + 2 are hashed and the entries of fragment f + 1 requested while the matrix instructions of fragment f run, and joined
// behind them.  The LDS addresses are formed as such: the table is
// the first thing in a kernel's dynamic LDS, which starts at 0 (no static LDS: checked at run time, QLESS_LDS_KERNEL), and a
// pointer into the array would cost an addition of that 0 per lookup.
struct GaussWords { uint32_t h[2]; };
struct GaussRaw { uint32_t lo[4], hi[4]; };
__device__ inline GaussWords gauss_words(RowKey key, uint32_t counter) {
    GaussWords w;
    w.h[0] = key_word(key, counter);
    w.h[1] = key_word(key, counter + kGold);
    return w;
}
__device__ inline void gauss_request(const GaussWords &w, uint32_t lane4, GaussRaw &r) {
    typedef __attribute__((address_space(3))) const uint16_t *lds16;
    typedef __attribute__((address_space(3))) const uint32_t *lds32;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const uint32_t h = w.h[e];
        r.lo[2 * e] = ((lds16)(uintptr_t)__builtin_amdgcn_perm(h, lane4, 0x0C0C0400u))[1];
        r.hi[2 * e] = *(lds32)(uintptr_t)__builtin_amdgcn_perm(h, lane4, 0x0C0C0500u);
        r.lo[2 * e + 1] = ((lds16)(uintptr_t)__builtin_amdgcn_perm(h, lane4, 0x0C0C0600u))[1];
        r.hi[2 * e + 1] = *(lds32)(uintptr_t)__builtin_amdgcn_perm(h, lane4, 0x0C0C0700u);
    }
}
__device__ inline Frag gauss_join(const GaussRaw &r) {
    Frag f;
#pragma unroll
    for (int i = 0; i < 4; ++i) f.w[i] = r.lo[i] | r.hi[i];
    return f;
}

template <ProjectInput IN, bool GAUSS, int NB>
__global__ void __launch_bounds__(kWaves * 64, 2)
project_kernel(ProjectArgs a, GaussTable gt) {
    constexpr bool DIRECT = IN == kDirectBf16;
    constexpr int RING = GAUSS && NB == 4 ? 3 : kRing;         // next to the table three stages of 128 rows fit
    using Sh = ProjShape<NB>;
    constexpr int KB = Sh::KB, kTileRows = Sh::kTileRows, kWaveCols = Sh::kWaveCols, kTileCols = Sh::kTileCols;
    constexpr int kStageBytes = Sh::kStageBytes, kDirectStageBytes = Sh::kDirectStageBytes;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    // XCD-aware decode: consecutive workgroup ids land on different XCDs, so the ktiles
    // workgroups that share one gradient slice are given ids 8 apart (same XCD, same L2).
    const int64_t id = blockIdx.x;
    const int xcd = (int)(id & 7);
    const int64_t t = id >> 3;
    const int kt = (int)(t % a.ktiles);
    const int64_t slice = (t / a.ktiles) * 8 + xcd;
    if (slice >= a.slices) return;
    const int64_t ntile = slice / a.nsplit;
    const int split = (int)(slice % a.nsplit);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int half = lane >> 5, l32 = lane & 31;
    const int64_t row0 = ntile * kTileRows;
    const int64_t c_begin = (int64_t)split * a.stages_per_split * kStageD;
    int64_t c_end = c_begin + a.stages_per_split * kStageD;
    if (c_end > a.d_len) c_end = a.d_len;
    const int nstages = (int)((c_end - c_begin + kStageD - 1) / kStageD);

    unsigned char *smem = lds + (GAUSS ? kGaussBytes : 0);          // the stage ring
    const uint32_t lane4 = (uint32_t)lane * 4u;
    if (GAUSS) gauss_fill(lds, gt);

    // row keys of this lane's KB 32-row blocks of the random matrix
    const int mbase = kt * kTileCols + wave * kWaveCols;
    RowKey key[KB];
    bool live[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        int m = mbase + 32 * kb + l32;
        live[kb] = (mbase + 32 * kb) < a.k;            // wave-uniform (k is a multiple of 64)
        key[kb] = row_key(a.sk, (uint32_t)m);
        key[kb].a += (uint32_t)half * (GAUSS ? 8u * kGold : kGold);   // upper half-wave reads the next word (eight words)
    }

    f32x16 acc[NB][KB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[nb][kb][v] = 0.0f;

    // staging (register path): kTileRows rows x 16 chunks of 8 columns; thread handles chunks tid + kThreads*i, one stage ahead, requested
    // without a branch (fp32 with a branch and a conversion behind every load: 128 x 131072 -> 8192 210 us, now 192, Gaussian 306, now 276;
    // 500 x 100000 -> 2048 178, now 152).  The Rademacher tiles of 128 rows have no registers for that (8 and, fp32, 30 spilled: 128 x 4 044 256 -> 1088 fp32
    // 1793 -> 1871 us, 349 x 1 118 053 -> 512 521 -> 581, bf16 337 -> 351) and keep packed chunks.
    constexpr bool RAW = GAUSS || NB == 2;
    constexpr int kThreads = kWaves * 64;
    constexpr int kChunksPerThread = kTileRows * (kStageD / 8) / kThreads;
    const int nfull = __builtin_amdgcn_readfirstlane((int)((c_end - c_begin) / kStageD));      // stages that are whole
    std::conditional_t<RAW, RawChunk<IN>, uint4> stage_regs[DIRECT ? 1 : kChunksPerThread];
    auto staged_row = [&](int i) { const int64_t row = row0 + ((tid + kThreads * i) >> 4); return row < a.n ? row : a.n - 1; };   // (never stored)
    auto fetch = [&](int s) {                      // (RAW: nfull > 0)
        const int64_t cs = c_begin + (int64_t)(!RAW || s < nfull ? s : nfull - 1) * kStageD;
#pragma unroll
        for (int i = 0; i < kChunksPerThread; ++i) {
            if constexpr (RAW) stage_regs[DIRECT ? 0 : i].load(a, staged_row(i), cs + (tid & 15) * 8);
            else stage_regs[DIRECT ? 0 : i] = load_chunk<IN>(a, row0 + ((tid + kThreads * i) >> 4), cs + (tid & 15) * 8, c_end);
        }
    };
    auto commit = [&](int buf, int s) {
#pragma unroll
        for (int i = 0; i < kChunksPerThread; ++i) {
            int c = tid + kThreads * i;
            int r = c >> 4, cc = c & 15;
            uint4 o;
            if constexpr (!RAW) o = stage_regs[DIRECT ? 0 : i];
            else if (s < nfull) o = stage_regs[DIRECT ? 0 : i].packed();
            else o = load_chunk<IN>(a, staged_row(i), c_begin + (int64_t)s * kStageD + cc * 8, c_end);
            *(uint4 *)(smem + buf * kStageBytes + r * kLdsStride + cc * 16) = o;
        }
    };

    // staging (direct path): a stage is kTileRows rows x 256 bytes = 16 or 32 wavefront copies of 1 KB,
    // two or four per wave.  Copy q fills LDS chunks 64 q .. 64 q + 63 (rows 4 q .. 4 q + 3); chunk `pos` of row r
    // holds gradient chunk pos ^ (r & 15), so 16 consecutive rows read the same gradient chunk
    // from 16 different bank groups.  Rows past n re-read row n-1 (never stored).
    constexpr int kCopies = kDirectStageBytes / 1024 / kWaves;
    const unsigned char *cptr[kCopies];
    unsigned cdst[kCopies];
    const unsigned lds0 = (unsigned)(uintptr_t)((__attribute__((address_space(3))) unsigned char *)smem);
    const int uwave = __builtin_amdgcn_readfirstlane(wave);
    if (DIRECT) {
#pragma unroll
        for (int u = 0; u < kCopies; ++u) {
            const int q = uwave * kCopies + u;
            const int r = 4 * q + (lane >> 4), pos = lane & 15;
            int64_t grow = row0 + r;
            if (grow > a.n - 1) grow = a.n - 1;
            cptr[u] = (const unsigned char *)a.G + (grow * a.ldG + c_begin) * 2 + ((pos ^ (r & 15)) << 4);
            cdst[u] = (unsigned)q * 1024u;
        }
    }
    auto issue = [&](int slot) {                   // start the copies of the next stage into a slot of the ring
        const unsigned buf = lds0 + (unsigned)slot * kDirectStageBytes;
#pragma unroll
        for (int u = 0; u < kCopies; ++u) {
            global_to_lds16(cptr[u], buf + cdst[u]);
            cptr[u] += kStageD * 2;
        }
    };
    // A fragment (rows 32 nb + l32, columns 64 bp + 32 half + 8 ks .. +7) of the stage in `slot`
    const unsigned a_sw = (unsigned)(((4 * half) ^ (l32 & 15)) << 4);
    auto read_a = [&](int slot, int nb, int bp, int ks) -> uint4 {
        if (DIRECT)
            return *(const uint4 *)(smem + slot * kDirectStageBytes + (32 * nb + l32) * (kStageD * 2) +
                                    (a_sw ^ (unsigned)((8 * bp + ks) << 4)));
        return *(const uint4 *)(smem + slot * kStageBytes + (32 * nb + l32) * kLdsStride +
                                (64 * bp + 32 * half + 8 * ks) * 2);
    };

    if constexpr (GAUSS) {
        // Fragment f of a stage (K step f / KB, coordinate block f % KB): its NB matrix instructions, behind the first of them the
        // look-ups of the next fragment and then the hashes of the one after that, the join last, so that neither the
        // look-ups' latency nor the chain of a hash is waited for.  The gradient fragments of a K step are read during the
        // first block of the one before, those of the next stage too: the stage's only barrier stands behind the first matrix
        // instruction of its last fragment, where every read of its slot has returned, and the slot is filled again
        // at once.  (128 x 2^18 -> 8192 609 -> 531 us, 64 x 2^20 1460 -> 1317, 128 x 2^22 -> 16384 16.5 -> 15.3 ms; entries requested
        // two fragments ahead instead of one are no faster.)
        constexpr int F = 8 * KB;
        auto word = [&](int s, int f) -> uint32_t {              // counter of fragment f of stage s (f may reach into the next)
            const int ks = f / KB % 8;
            const uint32_t w = a.wbase + (uint32_t)((c_begin + ((int64_t)s + f / F) * kStageD) >> 5);
            return (w * 8u + 16u * (uint32_t)(ks >> 2) + 2u * (uint32_t)(ks & 3)) * kGold + kSaltStride;
        };
        if (DIRECT) {
#pragma unroll
            for (int s = 0; s < RING; ++s)
                if (s < nstages) issue(s);
            if (nstages >= RING) wait_vmcnt<(RING - 1) * kCopies>(); else wait_vmcnt<0>();
        } else {
            if (nfull > 0) fetch(0);
            commit(0, 0);
        }
        __syncthreads();                           // stage 0 and the table visible to all waves
        Frag ag[2][NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) ag[0][nb].u = read_a(0, nb, 0, 0);
        GaussRaw raw;
        GaussWords next = gauss_words(key[0], word(0, 0));
        gauss_request(next, lane4, raw);
        next = gauss_words(key[1], word(0, 1));
        Frag bf = gauss_join(raw);
        for (int s = 0, buf = 0; s < nstages; ++s) {
            const int nbuf = buf + 1 < (DIRECT ? RING : 2) ? buf + 1 : 0;
            if (!DIRECT && s + 1 < nstages) fetch(s + 1);
#pragma unroll
            for (int f = 0; f < F; ++f) {
                const int ks = f / KB, kb = f % KB, kn = ks + 1;
                __builtin_amdgcn_sched_barrier(0);
                acc[0][kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ag[ks & 1][0].v, bf.v, acc[0][kb], 0, 0, 0);
                if (f == F - 1) {
                    __builtin_amdgcn_sched_barrier(0);
                    if (DIRECT) {
                        // stage s + 1 is the oldest copy group in flight; RING - 2 younger ones may stay outstanding
                        if (s + RING - 1 < nstages) wait_vmcnt<(RING - 2) * kCopies>(); else wait_vmcnt<0>();
                    } else if (s + 1 < nstages) {
                        commit(nbuf, s + 1);
                    }
                    __syncthreads();
                    if (DIRECT && s + RING < nstages) issue(buf);
                    // (after the last stage: in bounds, not used)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) ag[0][nb].u = read_a(nbuf, nb, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
                gauss_request(next, lane4, raw);
                if (kb == 0 && kn < 8) {
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) ag[kn & 1][nb].u = read_a(buf, nb, kn >> 2, kn & 3);
                }
                next = gauss_words(key[(f + 2) % KB], word(s, f + 2));
#pragma unroll
                for (int nb = 1; nb < NB; ++nb)
                    acc[nb][kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ag[ks & 1][nb].v, bf.v, acc[nb][kb], 0, 0, 0);
                bf = gauss_join(raw);
                // order: look-ups right behind the first matrix instruction, the hashes between the others
                if (f != F - 1) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
#pragma unroll
                for (int nb = 1; nb < NB; ++nb) {
                    __builtin_amdgcn_sched_group_barrier(0x002, NB == 2 ? 16 : 4, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                }
            }
            buf = nbuf;
        }
    } else {
    if (DIRECT) {
#pragma unroll
        for (int s = 0; s < RING - 1; ++s)
            if (s < nstages) issue(s);
    } else {
        if (!RAW || nfull > 0) fetch(0);
        commit(0, 0);
        __syncthreads();
    }

    uint32_t fp4_one = 0x22222222u;                // eight FP4 codes of +1.0
    asm volatile("" : "+v"(fp4_one));              // keep it in a vector register
    for (int s = 0; s < nstages; ++s) {
        const int buf = DIRECT ? s % RING : (s & 1);
        if (DIRECT) {
            // stage s is the oldest copy group in flight; two younger ones may stay outstanding
            if (s + RING - 2 < nstages) wait_vmcnt<(RING - 2) * kCopies>(); else wait_vmcnt<0>();
            __syncthreads();                       // stage s visible to all waves; slot of stage s-1 free
            if (s + RING - 1 < nstages) issue((s + RING - 1) % RING);
        } else {
            if (s + 1 < nstages) fetch(s + 1);
        }
        const int64_t cs = c_begin + (int64_t)s * kStageD;       // multiple of 128
        const uint32_t wstage = a.wbase + (uint32_t)(cs >> 5);
#pragma unroll
        for (int bp = 0; bp < 2; ++bp) {
            // A fragments: rows 32*nb + l32, columns 64*bp + 32*half + 8*ks .. +7
            Frag af[NB][4];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
                    af[nb][ks].u = read_a(buf, nb, bp, ks);
            const uint32_t wpair = wstage + 2u * bp;             // word index of lanes 0..31
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                // row blocks past k (last k-tile only) are computed and dropped in the epilogue
                {
                    const uint32_t h = key_word(key[kb], wpair * kGold);
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) {
                        // (h << ks) & 0x88888888 | 0x22222222 in two instructions: the fused and-or takes one
                        // literal only, so the second constant is held in a register
                        uint32_t x;
                        asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(x) : "v"(h << ks), "s"(0x88888888u), "v"(fp4_one));
                        Frag bf;
                        bf.p[0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(x, 1.0f, 0);
                        bf.p[1] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(x, 1.0f, 1);
                        bf.p[2] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(x, 1.0f, 2);
                        bf.p[3] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(x, 1.0f, 3);
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb)
                            acc[nb][kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[nb][ks].v, bf.v, acc[nb][kb], 0, 0, 0);
                    }
                }
            }
        }
        if (!DIRECT) {
            if (s + 1 < nstages) commit(buf ^ 1, s + 1);
            __syncthreads();
        }
    }
    }

    // partial tile -> workspace [split][n][k];  D[i][j]: j = lane%32, i = 8*(v/4) + 4*(lane/32) + v%4
    float *wsp = a.ws + (size_t)split * (size_t)a.n * (size_t)a.k;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            if (!live[kb]) continue;
            const int m = mbase + 32 * kb + l32;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int64_t row = row0 + 32 * nb + 8 * (v >> 2) + 4 * half + (v & 3);
                if (row < a.n) wsp[(size_t)row * a.k + m] = acc[nb][kb][v];
            }
        }
}

// ------------------------------------------------------------------------------------------
// Batches that do not fill 64-row tiles, and few projected coordinates: tiles of 16 NR rows (NR = 1 .. 4).
//
// The same product with v_mfma_f32_16x16x32_bf16: a fragment of the random operand is 16 coordinates x 32 columns and
// feeds NR matrix instructions of 16 cycles, so a batch of 16 pays for 16 rows and not for 64.  Bound there: vector
// ALU, 8.4 operations per fragment (33 cycles beside 16 NR of the matrix cores; 16 rows: 67 % and 32 % of all cycles).  A lane (coordinate
// lane % 16, group lane / 16) takes word 4 s + lane / 16 of its row for sub-stage s of 128 columns; the word's four
// bytes-of-columns are the lane's 8 columns of the four K steps, on both operands.
//   NX wavefronts side by side cover 128 NX coordinates; NK = 8 / NX groups of them take alternate sub-stages of the
//   workgroup's d-slice (k <= 512: all eight wavefronts have work although the tile is 512 wide) and join their
//   sums in LDS at the end.
// ------------------------------------------------------------------------------------------
constexpr int kNarrowCols = 128;                // coordinates per wavefront
template <int NR, int NX> struct NarrowShape {
    static constexpr int NK = kWaves / NX, kRows = 16 * NR, kCols = kNarrowCols * NX;
    static constexpr int kSubBytes = kRows * kStageD * 2;         // a sub-stage: kRows x 256 bytes, chunk c of row r at c ^ (r % 16)
    static constexpr int kStage = NK * kSubBytes;
    // stages in the ring (asynchronous copies; 2 when staged); Gaussian: two, so that two workgroups of 16-row tiles fit
    static constexpr int ring(bool gauss) { return gauss ? 2 : 4; }
    static constexpr int kJoin = (NK - 1) * kRows * kCols * 4;     // sums of the other groups, after the last stage: over everything else
    static constexpr int lds(bool direct, bool gauss) {
        const int r = (direct ? ring(gauss) : 2) * kStage + (gauss ? kGaussBytes : 0);
        return r > kJoin ? r : kJoin;
    }
    static_assert(lds(true, false) <= kProjectMaxLds && lds(true, true) <= kProjectMaxLds, "LDS of one compute unit");
    // as many workgroups on a compute unit as the plan counts: two of 16-row tiles, 81 920 bytes each when Gaussian (with the
    // sums beside the table 98 304, one workgroup: 1 x 2^19 -> 8192 553 us, now 463; 4 x 194 560 fp32 280, now 202)
    static constexpr int kPerCU = NX == 8 ? kTileCost[kTile48].per_cu
        : kTileCost[NR == 3 ? kTile48x512 : (NR == 2 ? kTile32x512 : kTile16x512)].per_cu;
    static_assert(kPerCU * lds(true, false) <= kProjectMaxLds && kPerCU * lds(true, true) <= kProjectMaxLds, "the plan's workgroups fit");
};

template <ProjectInput IN, bool GAUSS, int NR, int NX>
__global__ void __launch_bounds__(kWaves * 64, NR == 1 ? 4 : 2)      // (wavefronts per SIMD: two workgroups of 16-row tiles)
project_narrow_kernel(ProjectArgs a, GaussTable gt) {
    using Sh = NarrowShape<NR, NX>;
    constexpr int NK = Sh::NK, KB = kNarrowCols / 16, kSubBytes = Sh::kSubBytes, kStage = Sh::kStage;
    constexpr bool DIRECT = IN == kDirectBf16;
    constexpr int RING = DIRECT ? Sh::ring(GAUSS) : 2;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    // XCD-aware decode as in project_kernel
    const int64_t id = blockIdx.x, t = id >> 3;
    const int kt = (int)(t % a.ktiles);
    const int64_t slice = (t / a.ktiles) * 8 + (id & 7);
    if (slice >= a.slices) return;
    const int64_t ntile = slice / a.nsplit;
    const int split = (int)(slice % a.nsplit);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lg = lane >> 4;
    const int wx = wave % NX, wk = wave / NX;
    const int64_t row0 = ntile * Sh::kRows;
    const int64_t c_begin = (int64_t)split * a.stages_per_split * kStageD;
    int64_t c_end = c_begin + a.stages_per_split * kStageD;
    if (c_end > a.d_len) c_end = a.d_len;
    const int nsub = __builtin_amdgcn_readfirstlane((int)((c_end - c_begin + kStageD - 1) / kStageD)), nstages = (nsub + NK - 1) / NK;
    const int nfull = __builtin_amdgcn_readfirstlane((int)((c_end - c_begin) / kStageD));      // sub-stages that are whole

    unsigned char *smem = lds + (GAUSS ? kGaussBytes : 0);
    const uint32_t lane4 = (uint32_t)lane * 4u;
    if (GAUSS) gauss_fill(lds, gt);

    const int mbase = kt * Sh::kCols + wx * kNarrowCols;
    RowKey key[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        key[kb] = row_key(a.sk, (uint32_t)(mbase + 16 * kb + l16));
        key[kb].a += (uint32_t)lg * (GAUSS ? 8u * kGold : kGold);
    }
    f32x4 acc[NR][KB];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) acc[r][kb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    // ---- staging through registers, two stages ahead (but see below): chunks of eight elements of the stage, [sub-stage][row][chunk], as they are in
    // memory.  Every stage requests the same loads without a branch (one would make the wait for a stage a wait for all of them): rows past
    // the last one re-read it (never stored), sub-stages that are not whole the last whole one; what is left of a row there is read element
    // by element where the stage is written to LDS.  (One stage ahead, with the end of the rows told apart by every load: fp32, 32 x 262144 -> 4096
    // 90 us, now 72, 16 x 300000 -> 8192 114, now 103, 1024 x 16384 -> 512 35.6, now 32.4; bf16 at odd offsets 1 x 400000 -> 8192 131, now 125.)
    constexpr int kThreads = kWaves * 64, kChunks = kStage / 16, kPer = (kChunks + kThreads - 1) / kThreads;
    // Gaussian bf16 tiles of 16 rows stay one stage ahead: their stages take longer than a load (two ahead, in twice the code, 1 x 100000 -> 8192 96 -> 98 us).
    constexpr bool TWO = !(GAUSS && IN == kStagedBf16 && NR == 1);
    RawChunk<IN> regs[TWO ? 2 : 1][DIRECT ? 1 : kPer];
    struct Chunk { int at, sub; int64_t row, cc; };
    auto chunk = [&](int i) {                      // thread's chunk i of a stage (past the last one: its first again, not written)
        const int c = kChunks % kThreads == 0 || tid + kThreads * i < kChunks ? tid + kThreads * i : tid;
        const int64_t row = row0 + c / 16 % Sh::kRows;
        return Chunk{c, __builtin_amdgcn_readfirstlane(c / (kSubBytes / 16)), row < a.n ? row : a.n - 1, (int64_t)(c & 15) * 8};
    };
    auto fetch = [&](int set, int s) {             // (nfull > 0)
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const Chunk c = chunk(i);
            const int q = s * NK + c.sub < nfull ? s * NK + c.sub : nfull - 1;
            regs[set][DIRECT ? 0 : i].load(a, c.row, c_begin + (int64_t)q * kStageD + c.cc);
        }
    };
    auto commit = [&](int set, int buf, int s) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const Chunk c = chunk(i);
            const int r = c.at >> 4, cc = c.at & 15;                            // r counts rows over all sub-stages: r % 16 is the row's
            uint4 o;
            if (s * NK + c.sub < nfull) o = regs[set][DIRECT ? 0 : i].packed();                 // wave-uniform
            else o = load_chunk<IN>(a, c.row, c_begin + ((int64_t)s * NK + c.sub) * kStageD + c.cc, c_end);
            if (tid + kThreads * i < kChunks) *(uint4 *)(smem + buf * kStage + r * 256 + ((cc ^ (r & 15)) << 4)) = o;
        }
    };
    // ---- asynchronous copies of 1 KB (4 rows); past the end of a stage a wavefront repeats its last copy, past the end
    // of the slice (an odd number of sub-stages) a group that has no sub-stage left re-reads the last one
    constexpr int kCp = kStage / 1024, kCopies = (kCp + kWaves - 1) / kWaves;
    const unsigned lds0 = (unsigned)(uintptr_t)((__attribute__((address_space(3))) unsigned char *)smem);
    const unsigned char *cptr[kCopies];
    unsigned cdst[kCopies];
    int csub[kCopies];
    if (DIRECT) {
#pragma unroll
        for (int u = 0; u < kCopies; ++u) {
            const int q = wave * kCopies + u < kCp ? wave * kCopies + u : kCp - 1;
            csub[u] = q / (kSubBytes / 1024);
            const int r = 4 * (q % (kSubBytes / 1024)) + (lane >> 4);
            int64_t grow = row0 + r;
            if (grow > a.n - 1) grow = a.n - 1;                                 // never stored
            cptr[u] = (const unsigned char *)a.G + (grow * a.ldG + c_begin) * 2 + (((lane & 15) ^ (r & 15)) << 4);
            cdst[u] = (unsigned)q * 1024u;
        }
    }
    auto issue = [&](int s) {
        const unsigned buf = lds0 + (unsigned)(s % RING) * kStage;
#pragma unroll
        for (int u = 0; u < kCopies; ++u) {
            const int sub = s * NK + csub[u] < nsub ? s * NK + csub[u] : nsub - 1;   // wave-uniform
            global_to_lds16(cptr[u] + (int64_t)sub * (kStageD * 2), buf + cdst[u]);
        }
    };
    if (DIRECT) {
#pragma unroll
        for (int s = 0; s < RING - 1; ++s)
            if (s < nstages) issue(s);
    } else {
        if (nfull > 0) { fetch(0, 0); if (TWO) fetch(TWO ? 1 : 0, 1); }
        commit(0, 0, 0);
        __syncthreads();
    }

    uint32_t fp4_one = 0x22222222u;                // eight FP4 codes of +1.0
    asm volatile("" : "+v"(fp4_one));
    GaussRaw raw;
    GaussWords next;
    auto stage = [&](int s, auto odd, auto only) { // odd: s % 2 where staged; only: there is no other one
        const int buf = DIRECT ? s % RING : (int)odd;
        if (DIRECT) {
            if (s + RING - 2 < nstages) wait_vmcnt<(RING - 2) * kCopies>(); else wait_vmcnt<0>();
            __syncthreads();
            if (s + RING - 1 < nstages) issue(s + RING - 1);
        } else if (!only) {
            if constexpr (TWO) fetch(odd, s + 2); else fetch(0, s + 1);
        }
        const int sub = s * NK + wk;
        if (sub < nsub) {                                                       // wave-uniform
            const unsigned char *sb = smem + buf * kStage + wk * kSubBytes + l16 * 256;
            Frag af[NR][4];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                for (int r = 0; r < NR; ++r) af[r][ks].u = *(const uint4 *)(sb + r * 4096 + (((4 * lg + ks) ^ l16) << 4));
            const uint32_t wstage = a.wbase + (uint32_t)((c_begin + (int64_t)sub * kStageD) >> 5);
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                uint32_t h = 0;
                if (!GAUSS) h = key_word(key[kb], wstage * kGold);
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    Frag bf;
                    if (!GAUSS) {
                        uint32_t x;
                        asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(x) : "v"(h << ks), "s"(0x88888888u), "v"(fp4_one));
                        bf.p[0] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(x, 1.0f, 0);
                        bf.p[1] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(x, 1.0f, 1);
                        bf.p[2] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(x, 1.0f, 2);
                        bf.p[3] = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(x, 1.0f, 3);
                    } else {
                        // hashed two fragments ahead, requested one ahead, in the order of use
                        auto words = [&](int f) { return gauss_words(key[f >> 2], (wstage * 8u + 2u * (uint32_t)(f & 3)) * kGold + kSaltStride); };
                        const int f = 4 * kb + ks;
                        if (f == 0) {
                            next = words(0);
                            gauss_request(next, lane4, raw);
                            next = words(1);
                        }
                        bf = gauss_join(raw);
                        if (f + 1 < 4 * KB) gauss_request(next, lane4, raw);
                        if (f + 2 < 4 * KB) next = words(f + 2);
                    }
#pragma unroll
                    for (int r = 0; r < NR; ++r)
                        acc[r][kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[r][ks].v, bf.v, acc[r][kb], 0, 0, 0);
                }
            }
        }
        if (!DIRECT) {
            if (!only && s + 1 < nstages) commit(TWO ? odd ^ 1 : 0, odd ^ 1, s + 1);
            __syncthreads();
        }
    };
    typedef std::integral_constant<int, 0> Even;
    typedef std::integral_constant<int, 1> Odd;
    if (DIRECT) {
        for (int s = 0; s < nstages; ++s) stage(s, Even(), std::false_type());
    } else if (nfull == 0) {
        stage(0, Even(), std::true_type());
    } else if (!TWO) {
        for (int s = 0; s < nstages; ++s) stage(s, s & 1, std::false_type());
    } else {
        for (int s = 0;;) {                        // the register sets by name
            stage(s, Even(), std::false_type());
            if (++s >= nstages) break;
            stage(s, Odd(), std::false_type());
            if (++s >= nstages) break;
        }
    }
    if (NK > 1) {
        // the other groups' sums pass through LDS ([group][row][column], over the ring and the table: every copy has landed and
        // every look-up returned before the barrier), added in group order
        float *join = (float *)lds;
        __syncthreads();
        if (wk > 0) {
#pragma unroll
            for (int r = 0; r < NR; ++r)
#pragma unroll
                for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        join[((wk - 1) * Sh::kRows + 16 * r + 4 * lg + v) * Sh::kCols + wx * kNarrowCols + 16 * kb + l16] = acc[r][kb][v];
        }
        __syncthreads();
        if (wk > 0) return;
#pragma unroll
        for (int z = 1; z < NK; ++z)
#pragma unroll
            for (int r = 0; r < NR; ++r)
#pragma unroll
                for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        acc[r][kb][v] += join[((z - 1) * Sh::kRows + 16 * r + 4 * lg + v) * Sh::kCols + wx * kNarrowCols + 16 * kb + l16];
    }
    // partial tile -> workspace [split][n][k];  D[i][j]: j = lane % 16, i = 4 (lane / 16) + v
    float *wsp = a.ws + (size_t)split * (size_t)a.n * (size_t)a.k;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        const int m = mbase + 16 * kb + l16;
        if (mbase + 16 * kb >= a.k) continue;                                   // wave-uniform (k is a multiple of 64)
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int64_t row = row0 + 16 * r + 4 * lg + v;
                if (row < a.n) wsp[(size_t)row * a.k + m] = acc[r][kb][v];
            }
    }
}

// P = (accumulate ? P : 0) + ((p_0 + p_1) + p_2) + ...   fixed order over the d-slices; four elements of a row per thread,
// eight planes in flight (bound: memory; 16 x 8192 with 32 planes 9.8 us with one 4-byte load at a time)
__global__ void __launch_bounds__(256)
project_reduce_kernel(const float *ws, int nsplit, int64_t n, int32_t k, int accumulate,
                      float *P, int64_t ldP, int vec) {
    const int64_t total = n * (int64_t)k;
    const size_t plane = (size_t)total / 4;                   // k is a multiple of 64
    for (int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4; i < total; i += (int64_t)gridDim.x * 1024) {
        const float4 *src = (const float4 *)(ws + i);
        float4 s = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        int sp = 0;
        for (; sp + 8 <= nsplit; sp += 8) {
            float4 t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = src[(size_t)(sp + u) * plane];
#pragma unroll
            for (int u = 0; u < 8; ++u) { s.x += t[u].x; s.y += t[u].y; s.z += t[u].z; s.w += t[u].w; }
        }
        for (; sp < nsplit; ++sp) {
            const float4 t = src[(size_t)sp * plane];
            s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
        }
        const int64_t row = i / k, m = i - row * k;
        float *dst = P + row * ldP + m;
        if (vec) {
            if (accumulate) {
                const float4 o = *(const float4 *)dst;
                s.x = o.x + s.x; s.y = o.y + s.y; s.z = o.z + s.z; s.w = o.w + s.w;
            }
            *(float4 *)dst = s;
        } else {
            const float v[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) dst[e] = accumulate ? dst[e] + v[e] : v[e];
        }
    }
}
static void launch_reduce(const float *ws, int nsplit, int64_t n, int32_t k, int accumulate, float *P, int64_t ldP, hipStream_t st) {
    int64_t blocks = (n * (int64_t)k / 4 + 255) / 256;
    if (blocks > 1 << 20) blocks = 1 << 20;                   // a launch takes fewer than 2^32 threads (n k of 2^34 and more)
    const int vec = (uintptr_t)P % 16 == 0 && ldP % 4 == 0;
    hipLaunchKernelGGL(project_reduce_kernel, dim3((unsigned)blocks), dim3(256), 0, st, ws, nsplit, n, k, accumulate, P, ldP, vec);
}

__global__ void generator_words_kernel(SeedKeys sk, uint32_t m0, int32_t nrows, uint32_t w0,
                                       int32_t nwords, uint32_t salt, uint32_t *out) {
    const int64_t total = (int64_t)nrows * nwords;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t r = (uint32_t)(i / nwords), t = (uint32_t)(i % nwords);
        out[i] = key_word(row_key(sk, m0 + r), (w0 + t) * kGold + salt * kSaltStride);
    }
}

}  // namespace qless

using namespace qless;

// Enough for every kind of input and for every smaller batch or gradient length (the plans of those may cut d into more
// slices, and a program that lays its workspace out for its largest batch uses it for the last one too): a batch
// of n rows in tiles of r takes at most the slices of two rounds, shared by its row tiles.
extern "C" size_t qless_project_workspace(int64_t n, int64_t d_len, int32_t k) {
    if (n <= 0 || d_len <= 0 || k <= 0) return 0;
    int64_t rows = 0;                                              // n times d-slices, at most
    for (const TileCost &c : kTileCost) {
        const int64_t kt = (k + c.cols - 1) / c.cols, w = 2 * (32 * c.per_cu) / kt * 8, r = (n < c.rows ? n : c.rows) * w;
        rows = r > rows ? r : rows;
    }
    const int64_t stages = (d_len + kStageD - 1) / kStageD;
    if (stages < rows && n * stages < rows) rows = n * stages;
    return (size_t)(rows > n ? rows : n) * (size_t)k * sizeof(float);
}

template <ProjectInput IN, bool GAUSS, int NR, int NX>
static void launch_narrow_shape(dim3 grid, hipStream_t st, const ProjectArgs &a, const GaussTable &gt) {
    using Sh = NarrowShape<NR, NX>;
    constexpr int lds = Sh::lds(IN == kDirectBf16, GAUSS);
    QLESS_LDS_KERNEL((project_narrow_kernel<IN, GAUSS, NR, NX>), lds, GAUSS);
    hipLaunchKernelGGL((project_narrow_kernel<IN, GAUSS, NR, NX>), grid, dim3(kWaves * 64), lds, st, a, gt);
}
template <ProjectInput IN, bool GAUSS, int NB>
static void launch_project_shape(dim3 grid, hipStream_t st, const ProjectArgs &a, const GaussTable &gt) {
    QLESS_LDS_KERNEL((project_kernel<IN, GAUSS, NB>), kProjectMaxLds, GAUSS);
    constexpr size_t ring = GAUSS && NB == 4 ? 3 : kRing;
    constexpr size_t lds = (IN == kDirectBf16 ? ring * (32 * NB) * kStageD * 2 : (size_t)2 * (32 * NB) * kLdsStride) + (GAUSS ? kGaussBytes : 0);
    static_assert(lds <= (size_t)kProjectMaxLds, "LDS of one compute unit");
    hipLaunchKernelGGL((project_kernel<IN, GAUSS, NB>), grid, dim3(kWaves * 64), lds, st, a, gt);
}
template <ProjectInput IN, bool GAUSS>
static void launch_project(const ProjectPlan &p, dim3 grid, hipStream_t st, const ProjectArgs &a, const GaussTable &gt) {
    switch (p.shape) {
        case kTile128: launch_project_shape<IN, GAUSS, 4>(grid, st, a, gt); break;
        case kTile64: launch_project_shape<IN, GAUSS, 2>(grid, st, a, gt); break;
        case kTile48: launch_narrow_shape<IN, GAUSS, 3, 8>(grid, st, a, gt); break;
        case kTile48x512: launch_narrow_shape<IN, GAUSS, 3, 4>(grid, st, a, gt); break;
        case kTile32x512: launch_narrow_shape<IN, GAUSS, 2, 4>(grid, st, a, gt); break;
        default: launch_narrow_shape<IN, GAUSS, 1, 4>(grid, st, a, gt); break;
    }
}

// Validates the projection arguments shared by both entry points and launches the split-d
// partial sums into ws ([nsplit][n][k]).  *nsplit_out = 0 when there is nothing to launch.
static qless_status project_partials(const void *G, qless_dtype dt, int64_t n, int64_t d_len, int64_t ldG,
                                     int64_t d_offset, int32_t k, qless_proj kind, uint64_t seed,
                                     void *ws, size_t ws_bytes, hipStream_t st, int *nsplit_out) {
    *nsplit_out = 0;
    if (n < 0 || d_len < 0 || d_offset < 0 || k <= 0 || ldG < d_len) return QLESS_ERR_INVALID_ARG;
    if (n > 0 && d_len > 0 && !G) return QLESS_ERR_INVALID_ARG;
    if (dt != QLESS_F32 && dt != QLESS_BF16) return QLESS_ERR_UNSUPPORTED;
    if (kind != QLESS_RADEMACHER && kind != QLESS_GAUSSIAN) return QLESS_ERR_UNSUPPORTED;
    if (k % 64 != 0 || d_offset % 32 != 0) return QLESS_ERR_UNSUPPORTED;
    if (d_offset + d_len > ((int64_t)1 << 36)) return QLESS_ERR_UNSUPPORTED;
    // the Gaussian stream numbers its words with 32 bits, four columns to a word
    if (kind == QLESS_GAUSSIAN && d_offset + d_len > ((int64_t)1 << 34)) return QLESS_ERR_UNSUPPORTED;
    if (n > ((int64_t)1 << 31)) return QLESS_ERR_UNSUPPORTED;
    if (n == 0) return QLESS_OK;
    ProjectPlan plans[kPlanKinds];
    make_plans(n, d_len, k, plans);
    const ProjectPlan &plan = plans[plan_kind(kind == QLESS_GAUSSIAN, dt == QLESS_F32)];
    if (plan.ws_bytes > 0 && (!ws || ws_bytes < plan.ws_bytes || (uintptr_t)ws % 16 != 0)) return QLESS_ERR_WORKSPACE;
    if (plan.grid > 0x7FFFFFFF) return QLESS_ERR_UNSUPPORTED;
    if (plan.nsplit == 0) return QLESS_OK;

    ProjectArgs a{};
    a.G = G; a.ws = (float *)ws; a.n = n; a.d_len = d_len; a.ldG = ldG;
    a.wbase = (uint32_t)(d_offset >> 5); a.k = k; a.sk = seed_keys(seed);
    a.ktiles = (int32_t)plan.ktiles; a.nsplit = (int32_t)plan.nsplit;
    a.slices = plan.slices; a.stages_per_split = plan.stages_per_split;
    GaussTable gt{};
    const bool gauss = kind == QLESS_GAUSSIAN;
    if (gauss) { const uint16_t *t = gaussian_table_bf16(); for (int i = 0; i < 256; ++i) gt.v[i] = t[i]; }
    const bool direct = dt == QLESS_BF16 && (uintptr_t)G % 16 == 0 && (ldG * 2) % 16 == 0 && d_len % kStageD == 0;
    const ProjectInput in = direct ? kDirectBf16 : (dt == QLESS_F32 ? kStagedF32 : kStagedBf16);
    const qless_status ready = device_ready();     // more than 64 KB of dynamic LDS has to be allowed per kernel
    if (ready != QLESS_OK) return ready;
    const dim3 grid((unsigned)plan.grid);
    switch (in) {
        case kDirectBf16: gauss ? launch_project<kDirectBf16, true>(plan, grid, st, a, gt) : launch_project<kDirectBf16, false>(plan, grid, st, a, gt); break;
        case kStagedBf16: gauss ? launch_project<kStagedBf16, true>(plan, grid, st, a, gt) : launch_project<kStagedBf16, false>(plan, grid, st, a, gt); break;
        default: gauss ? launch_project<kStagedF32, true>(plan, grid, st, a, gt) : launch_project<kStagedF32, false>(plan, grid, st, a, gt); break;
    }
    if (launch_status() != QLESS_OK) return QLESS_ERR_DEVICE;
    *nsplit_out = (int)plan.nsplit;
    return QLESS_OK;
}

extern "C" qless_status qless_project(const void *G, qless_dtype dt, int64_t n, int64_t d_len,
                                      int64_t ldG, int64_t d_offset, int32_t k, qless_proj kind,
                                      uint64_t seed, int accumulate, float *P, int64_t ldP,
                                      void *ws, size_t ws_bytes, void *stream) {
    if (ldP < k || (n > 0 && !P)) return QLESS_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    int nsplit = 0;
    const qless_status rc = project_partials(G, dt, n, d_len, ldG, d_offset, k, kind, seed, ws, ws_bytes,
                                             st, &nsplit);
    if (rc != QLESS_OK || n == 0) return rc;
    if (nsplit == 0 && accumulate) return QLESS_OK;       // nothing to add
    launch_reduce((const float *)ws, nsplit, n, k, accumulate, P, ldP, st);
    return launch_status();
}

extern "C" qless_status qless_project_quantize(const void *G, qless_dtype dt, int64_t n, int64_t d_len,
                                               int64_t ldG, int64_t d_offset, int32_t k, qless_proj kind,
                                               uint64_t seed, int bits, void *codes, float *S, float *rnorm,
                                               float *P, int64_t ldP, void *ws, size_t ws_bytes,
                                               void *stream) {
    if (d_len <= 0 || (P && ldP < k)) return QLESS_ERR_INVALID_ARG;
    if (n > 0 && (!codes || !S || !rnorm)) return QLESS_ERR_INVALID_ARG;
    if ((uintptr_t)codes % 4) return QLESS_ERR_INVALID_ARG;
    if (!valid_bits(bits)) return QLESS_ERR_UNSUPPORTED;
    if (ws && (uintptr_t)ws % 16 != 0) return QLESS_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    int nsplit = 0;
    const qless_status rc = project_partials(G, dt, n, d_len, ldG, d_offset, k, kind, seed, ws, ws_bytes,
                                             st, &nsplit);
    if (rc != QLESS_OK || n == 0) return rc;
    return quantize_rows((const float *)ws, k, nsplit, (size_t)n * (size_t)k, P, ldP, n, k, bits, codes, S,
                         rnorm, st);
}

// P = (accumulate ? P : 0) + other, element by element (joins two accumulators when the last slice is
// too long-rowed for the fused path)
__global__ void __launch_bounds__(256)
add_rows_kernel(float *P, int64_t ldP, const float *other, int64_t ldO, int64_t n, int32_t k) {
    const int64_t total = n * (int64_t)k;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t row = i / k, m = i - row * k;
        P[row * ldP + m] = P[row * ldP + m] + other[row * ldO + m];
    }
}

extern "C" qless_status qless_project_quantize_slice(const void *G, qless_dtype dt, int64_t n, int64_t d_len,
                                                     int64_t ldG, int64_t d_offset, int32_t k, qless_proj kind,
                                                     uint64_t seed, int first, int last, float *P, int64_t ldP,
                                                     const float *P_other, int64_t ldO, int bits, void *codes,
                                                     float *S, float *rnorm, void *ws, size_t ws_bytes,
                                                     void *stream) {
    if (ldP < k || (n > 0 && !P) || (P_other && ldO < k)) return QLESS_ERR_INVALID_ARG;
    if (P_other && !last) return QLESS_ERR_INVALID_ARG;
    if (last) {
        if (n > 0 && (!codes || !S || !rnorm)) return QLESS_ERR_INVALID_ARG;
        if ((uintptr_t)codes % 4) return QLESS_ERR_INVALID_ARG;
        if (!valid_bits(bits)) return QLESS_ERR_UNSUPPORTED;
    }
    hipStream_t st = (hipStream_t)stream;
    int nsplit = 0;
    const qless_status rc = project_partials(G, dt, n, d_len, ldG, d_offset, k, kind, seed, ws, ws_bytes,
                                             st, &nsplit);
    if (rc != QLESS_OK || n == 0) return rc;
    const int64_t total = n * (int64_t)k;
    int64_t blocks = (total + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    // the last slice of rows that fit in registers: its partial sums, the accumulator and the second
    // accumulator are added by the quantiser itself, in the order of the separate kernels
    const bool fused = last && nsplit > 0 && k <= 16384;
    if (!fused) {
        if (nsplit > 0 || first)
            launch_reduce((const float *)ws, nsplit, n, k, first ? 0 : 1, P, ldP, st);
        if (!last) return launch_status();
        if (P_other)
            hipLaunchKernelGGL(add_rows_kernel, dim3((unsigned)blocks), dim3(256), 0, st, P, ldP, P_other, ldO, n, k);
        return quantize_rows(P, ldP, 1, 0, nullptr, 0, n, k, bits, codes, S, rnorm, st);
    }
    return quantize_rows((const float *)ws, k, nsplit, (size_t)n * (size_t)k, P, ldP, n, k, bits, codes, S,
                         rnorm, st, first ? nullptr : P, ldP, P_other, ldO);
}

extern "C" qless_status qless_generator_words(uint64_t seed, uint32_t m0, int32_t nrows,
                                              uint32_t w0, int32_t nwords, uint32_t salt,
                                              uint32_t *out, void *stream) {
    if (nrows < 0 || nwords < 0 || (!out && nrows > 0 && nwords > 0)) return QLESS_ERR_INVALID_ARG;
    const int64_t total = (int64_t)nrows * nwords;
    if (total == 0) return QLESS_OK;
    int64_t blocks = (total + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(generator_words_kernel, dim3((unsigned)blocks), dim3(256), 0,
                       (hipStream_t)stream, seed_keys(seed), m0, nrows, w0, nwords, salt, out);
    return launch_status();
}

// For the tests, host only: {rows and coordinates of the tile, d-slices, 128-column stages per d-slice, workspace bytes} of a
// projection's plan.
extern "C" void qless_internal_project_plan(int64_t n, int64_t d_len, int32_t k, int gauss, int fp32, int64_t *out) {
    ProjectPlan plans[kPlanKinds];
    make_plans(n, d_len, k, plans);
    const ProjectPlan &p = plans[plan_kind(gauss != 0, fp32 != 0)];
    out[0] = kTileCost[p.shape].rows; out[1] = kTileCost[p.shape].cols;
    out[2] = p.nsplit; out[3] = p.stages_per_split; out[4] = (int64_t)p.ws_bytes;
}

// For the tests: bytes of scratch memory (spilled registers) per lane of the Rademacher kernel of 64- or 128-row tiles whose rows pass through
// registers; -1 if the device does not say.
extern "C" int qless_internal_project_scratch(int rows, int fp32) {
    using namespace qless;
    const void *fn = rows == 128 ? (fp32 ? (const void *)project_kernel<kStagedF32, false, 4> : (const void *)project_kernel<kStagedBf16, false, 4>)
                                 : (fp32 ? (const void *)project_kernel<kStagedF32, false, 2> : (const void *)project_kernel<kStagedBf16, false, 2>);
    hipFuncAttributes at{};
    return hipFuncGetAttributes(&at, fn) == hipSuccess ? (int)at.localSizeBytes : -1;
}
