// qless_topk: indices of the k_sel largest scores, ordered by (score descending, index ascending)
// (paper Sec. 4.1: the top 5 % of the training examples by influence score).
//
// Every example gets a 64-bit key  (order-preserving image of the fp32 score) << 32 | (2^32-1 - index);
// keys are distinct and "larger key" is exactly "selected earlier".  Steps:
//   1. find the k_sel-th largest score, to a digit that leaves few keys too many.  Up to 16384 scores one workgroup holds all of them in
//   registers and does this and the compaction in a single launch (topk_select_one_kernel); above that, one histogram launch for each of
//   the three digits (10, 11 and 11 bits) of the score, whose workgroups each first pick the digit of the pass before from its finished
//   histogram (a scan of its bins, cheaper than a launch of its own); the passes stop as soon as the keys from the bucket of
//   the k_sel-th key on are no more than the ordering takes along (it drops those behind the k_sel-th).  If the threshold score T is
//   shared by more examples than that, the r with the smallest indices are the first r in array order: a count of the examples with
//   score T per 1024 examples and the sum of the counts before them (taken where it is needed, above 4096 such groups by a scan
//   launch) give every such example its position among them, and that is its place behind all keys above T;
//   2. compact the keys above the threshold (one atomic per workgroup and 1024 examples);
//   3. order them, descending: up to 16384 selected keys by rank (every key counts the larger ones
//   among all of them, k_sel^2 comparisons spread over the whole chip, and its index and score go to the slot of
//   its rank: one launch); above that, a bitonic network (LDS spans of 4096 keys with global
//   steps in between), then  4. decode indices and gather the scores.
// Latency is all there is to save: what a launch more costs is 3 to 5 us.
#include "common.h"
#include <atomic>
#include <mutex>

namespace qless {

constexpr int kSortBlock = 4096;   // keys sorted per workgroup in LDS (32 KB)
constexpr int kSortOne = 16384;    // most (padded) selected keys that are ordered by rank instead of sorted
constexpr int kPasses = 3;         // digits of the score half of the keys (histogram launches; four digits of 8 bits were a launch more)
constexpr int kDigitBits[kPasses] = {10, 11, 11}, kDigitShift[kPasses] = {54, 43, 32}, kHistAt[kPasses] = {0, 1024, 3072};
constexpr int kHistBins = 5120;
constexpr int64_t kSelectOneMax = 16384;     // scores one workgroup selects from in a single launch (top 5 % of 32768: 26 - 49 us, by the launches 26 - 30)

struct TopkPlan {
    int64_t padded;                // power of two >= k_sel (>= kSortBlock)
    size_t off_sel, off_hist, off_state, off_ties, total;
    int64_t chunks;                // groups of 1024 examples
};

static TopkPlan topk_plan(int64_t N, int64_t k_sel) {
    TopkPlan p{};
    int64_t pad = kSortBlock;
    while (pad < k_sel) pad <<= 1;
    p.padded = pad;
    size_t o = 0;
    p.off_sel = o;   o += (size_t)pad * 8;
    p.off_hist = o;  o += 4096 + (size_t)pad * 4;   // one histogram per pass, 20 480 bytes
    p.off_state = o; o += 192;                      // state before each pass and after the last; compaction cursor
    p.chunks = (N + 1023) / 1024;
    p.off_ties = o;  o += (size_t)(p.chunks + 1) * 4;   // examples at the threshold score per 1024 examples
    p.total = o;
    return p;
}

static_assert(kHistBins * 4 <= 4096 + kSortBlock * 4, "the histograms' share of the workspace");

struct SelectState {
    unsigned long long prefix;     // high digits of the threshold found so far
    unsigned long long remaining;  // rank still to locate inside the current prefix bucket
    unsigned int count;            // compaction cursor (of the last state only)
    unsigned int done;             // the threshold is final (the keys from `prefix` on are compacted): later passes return at once
    unsigned long long take;       // keys that the ordering is given before the examples at the threshold score: 32 bytes per state
};

__device__ inline uint32_t order_key(float f) {
    if (f == 0.0f) f = 0.0f;                       // -0 and +0 compare equal
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ inline unsigned long long make_key(float sc, int64_t i) {
    return ((unsigned long long)order_key(sc) << 32) | (0xFFFFFFFFull - (unsigned long long)i);
}

// state[0] = nothing chosen yet; the histograms from bin `from` on and the compaction cursor (state[kPasses].count) cleared by a workgroup
__device__ inline void clear_states(unsigned int *hist, int from, SelectState *state, unsigned long long k_sel) {
    if (threadIdx.x == 0) {
        state[0].prefix = 0; state[0].remaining = k_sel; state[0].count = 0; state[0].done = 0; state[0].take = 0;
        state[kPasses].count = 0;
    }
    for (int i = from + threadIdx.x; i < kHistBins; i += blockDim.x) hist[i] = 0;
}
__global__ void __launch_bounds__(256) topk_init_kernel(unsigned int *hist, SelectState *state, unsigned long long k_sel) {
    clear_states(hist, 0, state, k_sel);
}

// The digit that holds the remaining rank `rem`, walking the B bins of a finished histogram from the top, in a workgroup of 256 threads.
// Of the first digit there may be `parts` histograms of 16-bit counts instead, one of each workgroup, to be added.
// The thread of that digit returns it, with the rank left inside its bin and the bin's count; the others return -1.  If no bin
// reaches the rank the digit is 0.  `part` is LDS scratch of four entries.  All threads call it.
template <int B>
__device__ inline int pick_digit(const unsigned int *bins, int parts, unsigned long long *part, unsigned long long rem, unsigned long long &left, unsigned int &count) {
    constexpr int P = B / 256;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, top = B - 1 - P * (int)threadIdx.x;      // thread 0 has the highest bins
    unsigned int c[P];
    unsigned long long sum = 0;
    if (P == 4 && parts) {                              // uniform
#pragma unroll
        for (int q = 0; q < P; ++q) c[q] = 0;
        for (int w0 = 0; w0 < parts; w0 += 8) {
            uint2 t[8];
#pragma unroll
            for (int w = 0; w < 8; ++w) t[w] = *(const uint2 *)((const unsigned short *)bins + (w0 + w < parts ? w0 + w : 0) * B + top - 3);
#pragma unroll
            for (int w = 0; w < 8; ++w)
                if (w0 + w < parts) { c[0] += t[w].y >> 16; c[1] += t[w].y & 0xFFFFu; c[2] += t[w].x >> 16; c[3] += t[w].x & 0xFFFFu; }
        }
    } else {
#pragma unroll
        for (int q = 0; q < P; ++q) c[q] = bins[top - q];
    }
#pragma unroll
    for (int q = 0; q < P; ++q) sum += c[q];
    unsigned long long upto = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long below = __shfl_up(upto, o, 64);
        if (lane >= o) upto += below;
    }
    if (lane == 63) part[wave] = upto;
    __syncthreads();
    for (int q = 0; q < wave; ++q) upto += part[q];
    unsigned long long before = upto - sum;
    const bool last = threadIdx.x == 255;
    if (before >= rem || (upto < rem && !last)) return -1;
#pragma unroll
    for (int q = 0; q < P; ++q) {
        if (before + c[q] >= rem || (last && q == P - 1)) { left = rem - before; count = c[q]; return top - q; }
        before += c[q];
    }
    return -1;
}

// Inclusive sum over the threads of a 1024-thread workgroup; `part` is LDS scratch of 16 entries.  All threads call it.
__device__ inline unsigned int block_scan(unsigned int v, unsigned int *part) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned int below = __shfl_up(v, o, 64);
        if (lane >= o) v += below;
    }
    __syncthreads();                                    // part may still be read from the call before
    if (lane == 63) part[wave] = v;
    __syncthreads();
    unsigned int base = 0;
#pragma unroll
    for (int q = 0; q < 16; ++q) base += q < wave ? part[q] : 0u;
    return v + base;
}

// Selection and compaction in one workgroup: thread t holds the keys of scores t, t + 1024, .., U of them, in registers.  The range
// of keys that holds the k_sel-th largest is cut into 2048 equal bins, counted in LDS, until a bin is taken as a whole or holds one value:
// two or three rounds for the scores of a datastore, whose keys lie close together (their leading bits, which a radix select starts
// with, are the same for nearly all of them, so its first passes count into a handful of bins).  A range over most of the 32 bits (infinities,
// NaN, both signs) puts nearly all keys into a few bins again: there the lanes that share the first one's bin are added at once.
// The bins start at the smallest key, so the last one may end past the largest: the range that is kept ends there (without that the end wrapped
// past 2^32 for NaN of bits 0x7FE00000 and above, whose keys are the last 2^21, and the rounds behind it counted nothing).
// Bound: latency (top 5 % of 16384, 8192 and 4096 scores 28.4, 21.4 and 19.1 us with up to eight radix passes and the compaction, ranks and output in
// launches of their own, now 17.5, 12.8 and 13.5; all scores equal 58 -> 27 us).
template <int U>
__global__ void __launch_bounds__(1024)
topk_select_one_kernel(const float *score, int N, unsigned int k_sel, unsigned long long *sel, int padded) {
    __shared__ unsigned int hist[2048], part[16], lohi[32], ties[16 * U];
    __shared__ unsigned int sh_bin, sh_left, sh_count;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t key[U], lo = 0xFFFFFFFFu, hi = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = u * 1024 + tid;
        const float f = score[i < N ? i : N - 1];
        key[u] = order_key(f);
        lo = key[u] < lo ? key[u] : lo;
        hi = key[u] > hi ? key[u] : hi;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t l = (uint32_t)__shfl_xor((int)lo, o, 64), h = (uint32_t)__shfl_xor((int)hi, o, 64);
        lo = l < lo ? l : lo;
        hi = h > hi ? h : hi;
    }
    if (lane == 0) { lohi[wave] = lo; lohi[16 + wave] = hi; }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        lo = lohi[q] < lo ? lohi[q] : lo;
        hi = lohi[16 + q] > hi ? lohi[16 + q] : hi;
    }
    int shift = lo == hi ? 0 : 32 - __builtin_clz(hi - lo) - 11;
    if (shift < 0) shift = 0;
    unsigned int rem = k_sel;
    bool cut;                                           // the threshold score is shared by more examples than are still to be taken
    for (;;) {                                          // uniform; every round narrows the range 2048-fold
        hist[tid] = 0; hist[tid + 1024] = 0;
        __syncthreads();
        if (shift > 16) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool in = u * 1024 + tid < N && key[u] >= lo && key[u] <= hi;
                const unsigned int bin = in ? (key[u] - lo) >> shift : 0u;
                const unsigned long long act = __ballot(in);
                if (act) {
                    const int leader = __ffsll((long long)act) - 1;
                    const unsigned int b0 = (unsigned int)__builtin_amdgcn_readlane((int)bin, leader);
                    const unsigned long long same = __ballot(in && bin == b0);
                    if (lane == leader) atomicAdd(&hist[b0], (unsigned int)__popcll(same));
                    if (in && bin != b0) atomicAdd(&hist[bin], 1u);
                }
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (u * 1024 + tid < N && key[u] >= lo && key[u] <= hi) atomicAdd(&hist[(key[u] - lo) >> shift], 1u);
        }
        __syncthreads();
        // bins from the top: thread t has 2047 - 2 t and the one below it
        const unsigned int c0 = hist[2047 - 2 * tid], c1 = hist[2046 - 2 * tid];
        const unsigned int upto = block_scan(c0 + c1, part), before = upto - c0 - c1;
        if (before < rem && rem <= upto) {
            const bool upper = rem <= before + c0;
            sh_bin = upper ? 2047 - 2 * tid : 2046 - 2 * tid;
            sh_left = rem - (upper ? before : before + c0);
            sh_count = upper ? c0 : c1;
        }
        __syncthreads();
        lo += sh_bin << shift;
        const uint32_t width = (1u << shift) - 1u;          // the bin's, which may reach past `hi` and past 2^32
        hi = hi - lo < width ? hi : lo + width;
        rem = sh_left;
        cut = sh_count != rem;
        if (!cut || shift == 0) break;
        shift = shift > 11 ? shift - 11 : 0;
    }
    // taken: keys from lo on, or, where lo is a value that not all examples with it are taken of, keys above it and the first `rem` with it
    unsigned long long take = 0;
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (u * 1024 + tid < N && (cut ? key[u] > lo : key[u] >= lo)) take |= 1ull << u;
    if (cut) {                                          // positions in array order: by u, then wavefront, then lane
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned long long m = __ballot(u * 1024 + tid < N && key[u] == lo);
            if (lane == 0) ties[u * 16 + wave] = (unsigned int)__popcll(m);
        }
        __syncthreads();
        const unsigned int mine = tid < 16 * U ? ties[tid] : 0u, upto = block_scan(mine, part);
        if (tid < 16 * U) ties[tid] = upto - mine;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool tie = u * 1024 + tid < N && key[u] == lo;
            const unsigned long long m = __ballot(tie);
            if (tie && ties[u * 16 + wave] + (unsigned int)__popcll(m & ((1ull << lane) - 1ull)) < rem) take |= 1ull << u;
        }
    }
    const unsigned int mine = (unsigned int)__popcll(take);
    unsigned int at = block_scan(mine, part) - mine;
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (take >> u & 1) {
            if (at < k_sel) sel[at] = ((unsigned long long)key[u] << 32) | (0xFFFFFFFFull - (unsigned long long)(u * 1024 + tid));
            ++at;
        }
    for (int i = (int)k_sel + tid; i < padded; i += 1024) sel[i] = 0;     // padding sorts last (real keys are > 0)
}

// The state after the digit pick of pass PASS (from the state before it and the pass's finished
// histogram), computed by every thread of a 256-thread workgroup alike; workgroup 0 also records
// it in state[PASS + 1].  `part` and `sh` are LDS scratch.
template <int PASS>
__device__ inline SelectState next_state(SelectState *state, const unsigned int *bins, int parts, unsigned int extra, unsigned long long *part, SelectState *sh) {
    const SelectState before = state[PASS];
    if (before.done) {                              // uniform
        if (blockIdx.x == 0 && threadIdx.x == 0) { state[PASS + 1].prefix = before.prefix; state[PASS + 1].remaining = before.remaining; state[PASS + 1].done = 1; state[PASS + 1].take = before.take; }
        return before;
    }
    unsigned long long left = 0;
    unsigned int count = 0;
    const int digit = pick_digit<1 << kDigitBits[PASS]>(bins, parts, part, before.remaining, left, count);
    if (digit >= 0) {
        sh->prefix = before.prefix | ((unsigned long long)digit << kDigitShift[PASS]);
        sh->remaining = left;
        // at most `extra` keys of the bucket are not wanted: all of it is taken, the prefix with zeros below is the threshold
        sh->done = count - left <= (unsigned long long)extra;
        sh->take = before.take + before.remaining - left + (sh->done ? count : 0u);
    }
    __syncthreads();
    SelectState after = *sh;
    after.count = 0;
    __syncthreads();
    if (blockIdx.x == 0 && threadIdx.x == 0) { state[PASS + 1].prefix = after.prefix; state[PASS + 1].remaining = after.remaining; state[PASS + 1].done = after.done; state[PASS + 1].take = after.take; }
    return after;
}

// Histogram of digit PASS (0 = most significant) over keys whose higher digits equal the prefix chosen so far; the pick of the pass before
// is done here first, by every workgroup for itself.  With PARTS there are few workgroups in the first pass: each stores a histogram of its
// own (16-bit counts, in the place of the selected keys, that the second pass adds), so that nothing has to be cleared by a launch before
// it, and the first one clears what the launches behind it count into.
template <int PASS, bool PARTS>
__global__ void __launch_bounds__(PASS == 0 && PARTS ? 1024 : 256)
topk_hist_kernel(const float *score, int64_t N, SelectState *state, unsigned int *hist, unsigned int *parts, int nparts, unsigned int extra,
                 unsigned long long k_sel) {
    constexpr int B = 1 << kDigitBits[PASS], shift = kDigitShift[PASS], T = PASS == 0 && PARTS ? 1024 : 256, PER = PASS == 0 && PARTS ? 4 : 8;
    __shared__ unsigned int h[B];
    __shared__ unsigned long long part[4];
    __shared__ SelectState sh;
    SelectState cur;
    if constexpr (PASS == 0) {
        if (PARTS) { cur.prefix = 0; cur.done = 0; if (blockIdx.x == 0) clear_states(hist, kHistAt[1], state, k_sel); }
        else cur = state[0];
    } else if constexpr (PASS == 1 && PARTS) cur = next_state<0>(state, parts, nparts, extra, part, &sh);
    else cur = next_state<PASS - 1>(state, hist + kHistAt[PASS - 1], 0, extra, part, &sh);
    if (cur.done) return;                           // uniform
    for (int i = threadIdx.x; i < B; i += T) h[i] = 0;
    __syncthreads();
    const unsigned long long prefix = cur.prefix;
    // bits above the current digit: pass 0 has none (mask 0), later passes compare them all
    constexpr unsigned long long himask = PASS == 0 ? 0ull : (~0ull << (shift + kDigitBits[PASS]) % 64);
    // a workgroup takes PER * T consecutive examples at a time (few workgroups: every one of them ends
    // with an atomic on every bin it has counted into), PER loads in flight per thread
    for (int64_t c0 = (int64_t)blockIdx.x * (T * PER); c0 < N; c0 += (int64_t)gridDim.x * (T * PER)) {   // uniform
        float v[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int64_t i = c0 + u * T + threadIdx.x;
            v[u] = i < N ? score[i] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int64_t i = c0 + u * T + threadIdx.x;
            const unsigned long long key = make_key(v[u], i);
            const bool match = i < N && ((key ^ prefix) & himask) == 0;
            const unsigned int d = (unsigned int)(key >> shift) & (unsigned int)(B - 1);
            // the leading digits of scores are few: the lanes that share the digit of the first matching
            // lane are added at once, the others one by one
            const unsigned long long act = __ballot(match);
            if (act) {
                const int leader = __ffsll((long long)act) - 1;
                const unsigned int d0 = (unsigned int)__builtin_amdgcn_readlane((int)d, leader);
                const unsigned long long same = __ballot(match && d == d0);
                if ((int)(threadIdx.x & 63) == leader) atomicAdd(&h[d0], (unsigned int)__popcll(same));
                if (match && d != d0) atomicAdd(&h[d], 1u);
            }
        }
    }
    __syncthreads();
    if (PASS == 0 && PARTS) {
        for (int i = threadIdx.x; i < B / 2; i += T) parts[blockIdx.x * (B / 2) + i] = h[2 * i] | h[2 * i + 1] << 16;
    } else {
        for (int i = threadIdx.x; i < B; i += T)
            if (h[i]) atomicAdd(&hist[kHistAt[PASS] + i], h[i]);
    }
}

constexpr int kCompactPer = 4;                      // examples per thread and round
constexpr int kChunk = 256 * kCompactPer;           // examples per round of a workgroup

// After the last histogram: picks its digit and gathers the keys above the threshold (or from it on, if its bucket is taken whole) in any
// order; the slots behind what is ordered are cleared up to `padded`.  A workgroup takes kChunk consecutive examples at a time
// and one atomic for all it selects among them.  If the threshold score's examples are taken by position, those of each group are counted.
__global__ void __launch_bounds__(256)
topk_finish_kernel(const float *score, int64_t N, SelectState *state, const unsigned int *hist, unsigned int extra,
                   unsigned int *ties, unsigned long long *sel, int64_t k_sel, int64_t slots, int64_t padded) {
    __shared__ unsigned long long part[4];
    __shared__ SelectState sh;
    __shared__ unsigned int offs[4 * kCompactPer + 1];
    __shared__ unsigned int cnt;
    const SelectState fin = next_state<kPasses - 1>(state, hist + kHistAt[kPasses - 1], 0, extra, part, &sh);
    const bool by_position = !fin.done;             // uniform
    const unsigned long long thr = by_position ? (fin.prefix | 0xFFFFFFFFull) + 1ull : fin.prefix;   // T + 1 in the score half
    const bool none_above = by_position && thr == 0ull;     // T is the largest score key: nothing lies above it
    const uint32_t T = (uint32_t)(fin.prefix >> 32);
    const int64_t used = by_position ? k_sel : (int64_t)fin.take;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t span = N > padded ? N : padded;
    for (int64_t c0 = (int64_t)blockIdx.x * kChunk; c0 < span; c0 += (int64_t)gridDim.x * kChunk) {   // uniform per workgroup
        unsigned long long key[kCompactPer], mask[kCompactPer];
        bool take[kCompactPer];
        unsigned int same = 0;
        if (threadIdx.x == 0) cnt = 0;
#pragma unroll
        for (int u = 0; u < kCompactPer; ++u) {
            const int64_t i = c0 + u * 256 + threadIdx.x;
            if (i >= used && i < padded) sel[i] = 0;   // padding sorts last (real keys are > 0)
            key[u] = 0; take[u] = false;
            bool tie = false;
            if (i < N) {
                key[u] = make_key(score[i], i);
                take[u] = !none_above && key[u] >= thr;
                tie = by_position && (uint32_t)(key[u] >> 32) == T;
            }
            mask[u] = __ballot(take[u]);
            same += (unsigned int)__popcll(__ballot(tie));
            if (lane == 0) offs[wave * kCompactPer + u] = (unsigned int)__popcll(mask[u]);
        }
        __syncthreads();
        if (lane == 0 && same) atomicAdd(&cnt, same);
        if (threadIdx.x == 0) {                      // exclusive prefix over the 16 counts, then one atomic
            unsigned int run = 0;
            for (int q = 0; q < 4 * kCompactPer; ++q) { const unsigned int v = offs[q]; offs[q] = run; run += v; }
            offs[4 * kCompactPer] = run ? atomicAdd(&state[kPasses].count, run) : 0u;
        }
        __syncthreads();
        if (by_position && threadIdx.x == 0 && c0 < N) ties[c0 / kChunk] = cnt;
        const unsigned int wgbase = offs[4 * kCompactPer];
#pragma unroll
        for (int u = 0; u < kCompactPer; ++u) {
            const unsigned int pos = wgbase + offs[wave * kCompactPer + u] +
                                     (unsigned int)__popcll(mask[u] & ((1ull << lane) - 1ull));
            if (take[u] && (int64_t)pos < slots) sel[pos] = key[u];
        }
        __syncthreads();                             // offs and cnt are reused by the next round
    }
}

// One workgroup: exclusive scan, in place, of the per-group counts.
__global__ void __launch_bounds__(1024)
topk_tie_scan_kernel(const SelectState *state, unsigned int *ties, int64_t chunks) {
    __shared__ unsigned int part[1024];
    __shared__ unsigned int carry;
    if (state[kPasses].done) return;                // written by the launch before
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int64_t b = 0; b < chunks; b += 1024) {
        const int64_t c = b + threadIdx.x;
        const unsigned int v = c < chunks ? ties[c] : 0u;
        part[threadIdx.x] = v;
        __syncthreads();
        for (int step = 1; step < 1024; step <<= 1) {   // Hillis-Steele, inclusive
            const unsigned int add = (int)threadIdx.x >= step ? part[threadIdx.x - step] : 0u;
            __syncthreads();
            part[threadIdx.x] += add;
            __syncthreads();
        }
        const unsigned int base = carry;
        if (c < chunks) ties[c] = base + part[threadIdx.x] - v;
        __syncthreads();
        if (threadIdx.x == 1023) carry = base + part[1023];
        __syncthreads();
    }
}

// The first `remaining` examples with the threshold score, in array order: place(position, index, score) for each, by the workgroups of 1024
// threads of a grid.  `ties` holds the counts per group of kChunk examples, summed over the groups before it (scanned) or not.
template <class F>
__device__ inline void each_tie(const SelectState &fin, const float *score, int64_t N, const unsigned int *ties, int scanned, F place) {
    __shared__ unsigned int part[16];
    __shared__ unsigned int base;
    static_assert(kChunk == 1024, "one example per thread");
    const uint32_t T = (uint32_t)(fin.prefix >> 32);
    const int64_t chunks = (N + kChunk - 1) / kChunk;
    for (int64_t c = blockIdx.x; c < chunks; c += gridDim.x) {     // uniform
        if (threadIdx.x == 0) base = scanned ? ties[c] : 0u;
        __syncthreads();
        if (!scanned) {
            unsigned int mine = 0;
            for (int64_t g = threadIdx.x; g < c; g += 1024) mine += ties[g];
            if (mine) atomicAdd(&base, mine);
        }
        __syncthreads();
        const unsigned long long first = base;
        if (first >= fin.remaining) return;          // uniform; later groups have more before them
        const int64_t i = c * kChunk + threadIdx.x;
        const float f = score[i < N ? i : N - 1];
        const bool tie = i < N && order_key(f) == T;
        const unsigned long long pos = first + block_scan(tie ? 1u : 0u, part) - 1ull;
        if (tie && pos < fin.remaining) place((int64_t)pos, i, f);
    }
}

// Where the selected keys are sorted: the examples with the threshold score behind those above it
__global__ void __launch_bounds__(1024)
topk_ties_kernel(const float *score, int64_t N, const SelectState *state, const unsigned int *ties, int scanned,
                 unsigned long long *sel, int64_t k_sel) {
    const SelectState fin = state[kPasses];
    if (fin.done) return;                           // uniform
    each_tie(fin, score, N, ties, scanned, [&](int64_t pos, int64_t i, float f) {
        if ((int64_t)fin.take + pos < k_sel) sel[fin.take + pos] = make_key(f, i);
    });
}

// Rank of every selected key = how many selected keys are larger (keys are distinct); its index and score go to the slot of that rank.
// A workgroup ranks 32 keys, one per lane of a half wavefront: its 32 halves count the larger ones in a share each of all keys, staged in LDS
// 4096 at a time and read by all lanes of a half at once (a broadcast), and the counts are joined in LDS.  k_sel^2 comparisons: for k_sel <=
// kSortOne only.  (Two launches, counts joined by global atomics, then written out: 3276 of 65536 2 us more; 64 keys to a workgroup leave
// half the chip idle there.)
// With a state (of a selection by launches) it says how many keys there are: those that a bucket held behind the k_sel-th are dropped, and
// examples with the threshold score that are taken by position go behind the others, without a rank.
// (Eight wavefronts per SIMD, two workgroups per compute unit: with one scalar register too many for that 16384 keys took 34 us instead of 27.)
__global__ void __launch_bounds__(1024, 8)
topk_rank_kernel(const unsigned long long *sel, int k_sel, int slots, const SelectState *state, const unsigned int *ties, int scanned,
                 const float *score, int64_t N, int64_t *idx, float *val) {
    __shared__ __attribute__((aligned(16))) unsigned long long tile[4096];
    __shared__ unsigned int larger[32][32];
    const int lane = threadIdx.x & 31, part = threadIdx.x >> 5, mine_at = (int)blockIdx.x * 32 + lane;
    SelectState fin;
    int keys = k_sel;
    if (state) {
        fin = state[kPasses];
        keys = fin.take < (unsigned long long)slots ? (int)fin.take : slots;
    }
    if ((int)blockIdx.x * 32 < keys) {              // uniform
        const unsigned long long mine = mine_at < keys ? sel[mine_at] : ~0ull;
        unsigned int cnt = 0;
        for (int jb = 0; jb < keys; jb += 4096) {
            const int n = keys - jb < 4096 ? keys - jb : 4096, share = (n + 63) / 64 * 2;     // keys per half, a multiple of two
            __syncthreads();
            for (int t = threadIdx.x; t < 32 * share; t += 1024) tile[t] = t < n ? sel[jb + t] : 0ull;   // 0 is below every key
            __syncthreads();
            const int t0 = part * share;
#pragma unroll 8
            for (int t = 0; t < share; t += 2) {
                const ulonglong2 pr = *(const ulonglong2 *)&tile[t0 + t];
                cnt += (pr.x > mine) + (pr.y > mine);
            }
        }
        larger[part][lane] = cnt;
        __syncthreads();
        if (part == 0 && mine_at < keys) {
#pragma unroll
            for (int q = 1; q < 32; ++q) cnt += larger[q][lane];
            const int64_t i = (int64_t)(0xFFFFFFFFull - (mine & 0xFFFFFFFFull));
            if (cnt < (unsigned int)k_sel) {
                idx[cnt] = i;
                const uint32_t s = (uint32_t)(mine >> 32);          // the score's bits, but for the sign of a zero
                if (val) val[cnt] = s == 0x80000000u ? score[i < N ? i : N - 1] : __uint_as_float(s & 0x80000000u ? s & 0x7FFFFFFFu : ~s);
            }
        }
    }
    if (!state || fin.done) return;                 // uniform
    each_tie(fin, score, N, ties, scanned, [&](int64_t pos, int64_t i, float f) {
        const int64_t at = keys + pos;
        if (at >= k_sel) return;
        idx[at] = i;
        if (val) val[at] = f;
    });
}

// Bitonic network, descending.  Stage size kk (sub-sequence length), step jj (partner distance).
__device__ inline void cmpswap_desc(unsigned long long &x, unsigned long long &y, bool desc) {
    if ((x < y) == desc) { const unsigned long long t = x; x = y; y = t; }
}

// all steps with jj < kSortBlock for stages kk_from..kk_to inside LDS.  Thread t handles the pairs t
// and t + 1024 of a step; for a partner distance jj <= 64 both pairs of every thread of a wavefront lie
// inside two 128-element segments that only this wavefront touches, so consecutive steps with
// jj <= 64 need no workgroup barrier (LDS operations of a wavefront complete in order).
__global__ void __launch_bounds__(1024)
topk_bitonic_local_kernel(unsigned long long *data, int64_t kk_from, int64_t kk_to) {
    __shared__ unsigned long long s[kSortBlock];
    const int64_t base = (int64_t)blockIdx.x * kSortBlock;
    for (int t = threadIdx.x; t < kSortBlock; t += 1024) s[t] = data[base + t];
    __syncthreads();
    bool wide_before = true;                           // the previous step crossed wavefront segments
    for (int64_t kk = kk_from; kk <= kk_to; kk <<= 1) {
        int64_t j0 = kk >> 1;
        if (j0 >= kSortBlock) j0 = kSortBlock >> 1;
        for (int lj = 63 - __builtin_clzll((unsigned long long)j0); lj >= 0; --lj) {   // partner distance 2^lj
            const int jj = 1 << lj;
            const bool wide = jj > 64;
            if (wide || wide_before) __syncthreads();
            else { __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront"); __builtin_amdgcn_wave_barrier(); }
            wide_before = wide;
            for (int t = threadIdx.x; t < kSortBlock / 2; t += 1024) {
                const int lo = ((t >> lj) << (lj + 1)) | (t & (jj - 1));
                const int hi = lo + jj;
                const bool desc = (((base + lo) & kk) == 0);
                unsigned long long x = s[lo], y = s[hi];
                cmpswap_desc(x, y, desc);
                s[lo] = x; s[hi] = y;
            }
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < kSortBlock; t += 1024) data[base + t] = s[t];
}

__global__ void topk_bitonic_global_kernel(unsigned long long *data, int64_t n, int64_t kk, int64_t jj) {
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n / 2;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t lo = (t / jj) * 2 * jj + (t % jj), hi = lo + jj;
        const bool desc = ((lo & kk) == 0);
        unsigned long long x = data[lo], y = data[hi];
        if ((x < y) == desc) { data[lo] = y; data[hi] = x; }
    }
}

__global__ void topk_emit_kernel(const unsigned long long *sel, int64_t k_sel, const float *score,
                                 int64_t N, int64_t *idx, float *val) {
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < k_sel;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = (int64_t)(0xFFFFFFFFull - (sel[t] & 0xFFFFFFFFull));
        idx[t] = i;
        if (val) val[t] = score[i < N ? i : N - 1];
    }
}

}  // namespace qless

using namespace qless;

extern "C" size_t qless_topk_workspace(int64_t N, int64_t k_sel) {
    if (N < 0 || k_sel < 0) return 0;
    return topk_plan(N, k_sel).total;
}

// Histograms of the first pass that its workgroups store one by one; 0: counted by atomics into one.  Every workgroup of the second pass reads
// all of them, so they are few whatever N is, and fit where any selection's keys go.  Top 5 % with them and without: 16385 scores 20.9 and 22.0 us, 65536
// 24.6 and 26.3, 131072 30.8 and 29.6, 270000 47.3 and 47.4, 10^6 (123 of them) 137 and 129, 10^7 (1221) 625 and 390.
constexpr int kFirstParts = kSortBlock * 8 / 2048;
static int first_pass_parts(int64_t N) { return N <= kFirstParts * (int64_t)8192 ? (int)((N + 8191) / 8192) : 0; }

// Enqueues the whole selection on `st`; `ws` holds at least topk_plan(N, k_sel).total bytes, 8-byte
// aligned; 1 <= k_sel <= N < 2^32, all pointers checked by the caller.
static qless_status topk_run(const float *score, int64_t N, int64_t k_sel, int64_t *idx, float *val,
                             void *ws, hipStream_t st) {
    const TopkPlan p = topk_plan(N, k_sel);
    unsigned char *w = (unsigned char *)ws;
    unsigned long long *sel = (unsigned long long *)(w + p.off_sel);
    unsigned int *hist = (unsigned int *)(w + p.off_hist);
    SelectState *state = (SelectState *)(w + p.off_state);
    unsigned int *ties = (unsigned int *)(w + p.off_ties);

    auto blocks_for = [](int64_t n) { int64_t b = (n + 255) / 256; if (b < 1) b = 1; if (b > 2048) b = 2048; return (unsigned)b; };
    const bool ranked = p.padded <= kSortOne, one = N <= kSelectOneMax;
    // up to 2^22 scores (4096 groups of 1024) the counts of the groups before one are summed where they are needed: a launch less
    const bool scan = p.chunks > 4096;
    // keys behind the k_sel-th that are ordered with the others, so that fewer digits tell: ranking takes the square of the keys, sorting the padded number
    int64_t extra = ranked && k_sel / 16 > 256 ? k_sel / 16 : 256;
    if (!ranked || extra > p.padded - k_sel) extra = p.padded - k_sel;
    if (one) {
        const auto select = N <= 4096 ? topk_select_one_kernel<4> : (N <= 8192 ? topk_select_one_kernel<8> : topk_select_one_kernel<16>);
        hipLaunchKernelGGL(select, dim3(1), dim3(1024), 0, st, score, (int)N, (unsigned int)k_sel, sel, (int)p.padded);
    } else {
        const unsigned long long want = (unsigned long long)k_sel;
        const unsigned ex = (unsigned)extra;
        // a histogram per workgroup of the first pass (2 KB, where the selected keys go later), of two rounds of 4096 scores at most so that its
        // counts fit 16 bits; else by atomics into one that a launch clears
        const int nparts = first_pass_parts(N);
        unsigned int *parts = (unsigned int *)sel;
        int64_t hblocks = (N + 2047) / 2048;
        if (hblocks > 2048) hblocks = 2048;
        if (nparts) {
            hipLaunchKernelGGL((topk_hist_kernel<0, true>), dim3((unsigned)nparts), dim3(1024), 0, st, score, N, state, hist, parts, 0, ex, want);
            hipLaunchKernelGGL((topk_hist_kernel<1, true>), dim3((unsigned)hblocks), dim3(256), 0, st, score, N, state, hist, parts, nparts, ex, want);
        } else {
            hipLaunchKernelGGL(topk_init_kernel, dim3(1), dim3(256), 0, st, hist, state, want);
            hipLaunchKernelGGL((topk_hist_kernel<0, false>), dim3((unsigned)hblocks), dim3(256), 0, st, score, N, state, hist, parts, 0, ex, want);
            hipLaunchKernelGGL((topk_hist_kernel<1, false>), dim3((unsigned)hblocks), dim3(256), 0, st, score, N, state, hist, parts, 0, ex, want);
        }
        hipLaunchKernelGGL((topk_hist_kernel<2, false>), dim3((unsigned)hblocks), dim3(256), 0, st, score, N, state, hist, parts, 0, ex, want);
        const int64_t clear = ranked ? 0 : p.padded, span = N > clear ? N : clear;
        int64_t cblocks = (span + kChunk - 1) / kChunk;
        if (cblocks > 2048) cblocks = 2048;
        hipLaunchKernelGGL(topk_finish_kernel, dim3((unsigned)cblocks), dim3(256), 0, st, score, N, state,
                           (const unsigned int *)hist, ex, ties, sel, k_sel, p.padded, clear);
        if (scan) hipLaunchKernelGGL(topk_tie_scan_kernel, dim3(1), dim3(1024), 0, st, (const SelectState *)state, ties, p.chunks);
        if (!ranked) hipLaunchKernelGGL(topk_ties_kernel, dim3((unsigned)(p.chunks < 512 ? p.chunks : 512)), dim3(1024), 0, st, score, N,
                                        (const SelectState *)state, (const unsigned int *)ties, scan ? 1 : 0, sel, k_sel);
    }
    if (ranked) {
        const int64_t most = one ? k_sel : k_sel + extra;
        int64_t rblocks = (most + 31) / 32;
        if (!one && rblocks < p.chunks) rblocks = p.chunks < 256 ? p.chunks : (rblocks > 256 ? rblocks : 256);     // (groups of examples with the threshold score)
        hipLaunchKernelGGL(topk_rank_kernel, dim3((unsigned)rblocks), dim3(1024), 0, st, (const unsigned long long *)sel, (int)k_sel, (int)p.padded,
                           one ? (const SelectState *)nullptr : (const SelectState *)state, (const unsigned int *)ties, scan ? 1 : 0, score, N, idx, val);
        return launch_status();
    }
    // many selected keys: sort them, descending, with a bitonic network
    const unsigned nblk = (unsigned)(p.padded / kSortBlock);
    hipLaunchKernelGGL(topk_bitonic_local_kernel, dim3(nblk), dim3(1024), 0, st, sel, (int64_t)2, (int64_t)kSortBlock);
    for (int64_t kk = 2 * kSortBlock; kk <= p.padded; kk <<= 1) {
        for (int64_t jj = kk >> 1; jj >= kSortBlock; jj >>= 1)
            hipLaunchKernelGGL(topk_bitonic_global_kernel, dim3(blocks_for(p.padded / 2)), dim3(256), 0, st, sel, p.padded, kk, jj);
        hipLaunchKernelGGL(topk_bitonic_local_kernel, dim3(nblk), dim3(1024), 0, st, sel, kk, kk);
    }
    hipLaunchKernelGGL(topk_emit_kernel, dim3(blocks_for(k_sel)), dim3(256), 0, st, sel, k_sel, score, N, idx, val);
    return launch_status();
}

static qless_status topk_check(const float *score, int64_t N, int64_t k_sel, const int64_t *idx) {
    if (N < 0 || k_sel < 0 || k_sel > N) return QLESS_ERR_INVALID_ARG;
    if (N > 0 && !score) return QLESS_ERR_INVALID_ARG;
    if (k_sel > 0 && !idx) return QLESS_ERR_INVALID_ARG;
    if (N >= ((int64_t)1 << 32)) return QLESS_ERR_UNSUPPORTED;
    return QLESS_OK;
}

extern "C" qless_status qless_topk(const float *score, int64_t N, int64_t k_sel, int64_t *idx,
                                   float *val, void *ws, size_t ws_bytes, void *stream) {
    const qless_status rc = topk_check(score, N, k_sel, idx);
    if (rc != QLESS_OK || k_sel == 0) return rc;
    if (!ws || ws_bytes < topk_plan(N, k_sel).total) return QLESS_ERR_WORKSPACE;
    if ((uintptr_t)ws % 8) return QLESS_ERR_WORKSPACE;
    return topk_run(score, N, k_sel, idx, val, ws, (hipStream_t)stream);
}

// ------------------------------------------------------------------------------------------
// The same selection for callers that cannot allocate: its workspace is a file-scope device
// array, one copy per GPU.  On the host the array's name only stands for the symbol; the
// address the kernels receive is the one hipGetSymbolAddress returns on each device.
// ------------------------------------------------------------------------------------------
constexpr int64_t kNoAllocMaxN = QLESS_TOPK_NOALLOC_MAX_N;
constexpr int64_t kNoAllocMaxSel = QLESS_TOPK_NOALLOC_MAX_SEL;
// topk_plan(kNoAllocMaxN, kNoAllocMaxSel).total, rounded up (checked at set-up)
constexpr size_t kScratchBytes = (size_t)kNoAllocMaxSel * 12 + 4096 + 256 + (size_t)(kNoAllocMaxN / 1024 + 2) * 4 + 256;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
static std::mutex scratch_mutex;
static std::atomic<void *> scratch_ptr[kMaxDevices];

// device address of this GPU's copy of `scratch` (resolved once per device, with that device current)
qless_status qless::topk_scratch_address(void **out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return QLESS_ERR_DEVICE;
    void *p = scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        std::lock_guard<std::mutex> lock(scratch_mutex);
        p = scratch_ptr[dev].load(std::memory_order_relaxed);
        if (!p) {
            if (topk_plan(kNoAllocMaxN, kNoAllocMaxSel).total > kScratchBytes) return QLESS_ERR_WORKSPACE;
            if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return QLESS_ERR_DEVICE;
            scratch_ptr[dev].store(p, std::memory_order_release);
        }
    }
    *out = p;
    return QLESS_OK;
}

extern "C" qless_status qless_topk_noalloc(const float *score, int64_t N, int64_t k_sel, int64_t *idx,
                                           float *val, void *stream) {
    const qless_status rc = topk_check(score, N, k_sel, idx);
    if (rc != QLESS_OK) return rc;
    if (N > kNoAllocMaxN || k_sel > kNoAllocMaxSel) return QLESS_ERR_UNSUPPORTED;
    if (k_sel == 0) return QLESS_OK;
    void *ws = nullptr;
    const qless_status rs = topk_scratch_address(&ws);
    if (rs != QLESS_OK) return rs;
    // every word of the workspace that a launch reads is written earlier in the same call (the first launch /
    // select kernels clear histograms, states and the cursor; the compaction clears padding;
    // the tie counts are written before they are scanned), so nothing of the call before survives
    return topk_run(score, N, k_sel, idx, val, ws, (hipStream_t)stream);
}

// For the tests, host only: the histograms that every workgroup of the second pass reads in a selection from N scores by launches.
extern "C" int qless_internal_topk_parts(int64_t N) { return first_pass_parts(N); }
