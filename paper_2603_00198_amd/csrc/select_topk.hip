// select_topk: indices of the K largest scores, ascending (paper Sec. 3.1, "Token Selection":
// keep the top K while preserving temporal order).  Ties at the K-th value go to the lowest
// index, which is what a stable sort by (score desc, index asc) gives.
//
// N is at most a few hundred thousand (<= 512 KB of scores), so the problem is latency-bound.
// Up to 32768 scores (and beyond 2^20, streaming) one 1024-lane workgroup does everything in one
// launch; between the two a chain of short launches with one workgroup per 4096 scores is
// three to four times faster than streaming (see "Wide form" below).
// The one-launch form: an MSB radix select on the order-preserving integer image of
// the floats, which yields the exact K-th value and how many of its duplicates to keep, then one
// ordered pass (packed prefix sums) writes the surviving indices.  The digits (11 bits each,
// histogram in LDS) are taken from key - min(key): the scores of a layer lie close together, so
// the leading bits of the raw keys carry no information, while the significant bits of the
// offsets usually fit two passes and spread over the bins.  Each lane owns 4 consecutive scores
// of every 4096-score tile; up to 32768 scores the keys are read from memory once and stay in
// registers for all passes, beyond that they are re-read in batches of 8 tiles with all loads of
// a batch in flight together.  Same-address LDS atomics serialise, so in the first pass every bin
// has 16 copies (fewer for up to 16384 scores), one per lane modulo 16, in adjacent LDS words (different
// banks), summed when a bin is picked; later passes only count the keys of one bin of the pass before and use 2 copies
// when those are few; once a bin holds no more than one wave's worth of keys the remaining digits
// are skipped and one wave ranks those keys directly.  The ordered pass scans 8 tiles per barrier.  No global atomics, no
// scratch memory, bit-exact and deterministic.
#include "common.h"

namespace strd {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / kWave;
constexpr int kBins = 2048;
constexpr int kTile = kThreads * 4;  // scores per tile
constexpr int kBatch = 8;            // tiles loaded together when streaming / scanned per barrier
// Copies of every histogram bin.  Clearing and summing 16 copies is 128 KB of LDS traffic each; up to two tiles
// of scores there are too few keys to queue on a counter for long.  With the tiles counted exactly and the scans at one
// barrier (every wave adds the wave totals up for itself) 1024 scores take 4.1 us for 6.4, 8192 6.1 for 7.6, 16384 9.7 for 13.6.
template <int TILES>
constexpr int kCopies = TILES == 1 || TILES == 2 ? 4 : TILES == 4 ? 8 : 16;
constexpr int kFewCopies = 2;        // copies in passes 1 and 2 when at most kFewKeys keys are still in play
constexpr int kFewKeys = 4096;
constexpr int kRankKeys = 64;        // at most this many keys still in play: one wave ranks them directly

// Monotone map float -> uint32 (larger float = larger key); -0.0 is folded onto +0.0.
// Every score maps above 0, the key given to the slots past the end of the array: the one bit
// pattern whose image would be 0 (a negative NaN, all bits set) shares key 1 with its neighbour,
// so that exactly K indices are written whatever the input holds.  NaNs are ordered by their
// bits: positive ones above +inf, negative ones below -inf.
__device__ __forceinline__ uint32_t order_key(float f) {
    uint32_t b = __float_as_uint(f);
    if (b == 0x80000000u) b = 0u;
    return max((b & 0x80000000u) ? ~b : (b | 0x80000000u), 1u);
}

// Keys of the 4 scores this lane owns in tile `t` (0 past the end).
__device__ __forceinline__ void load_tile(const float *__restrict__ scores, int N, int t, uint32_t (&key)[4]) {
    const int i0 = t * kTile + threadIdx.x * 4;
    if (i0 + 3 < N) {
        const float4 v = *reinterpret_cast<const float4 *>(scores + i0);
        key[0] = order_key(v.x); key[1] = order_key(v.y); key[2] = order_key(v.z); key[3] = order_key(v.w);
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) key[u] = (i0 + u < N) ? order_key(scores[i0 + u]) : 0u;
    }
}

// hist[bin] += 1 in this lane's copy of the bin (COPIES copies per bin, adjacent words).
template <int COPIES>
__device__ __forceinline__ void hist_add(uint32_t *hist, uint32_t bin, bool valid) {
    if (valid) atomicAdd(&hist[bin * COPIES + (threadIdx.x & (COPIES - 1))], 1u);
}

// Inclusive prefix sum over the 64 lanes of a wave with DPP moves (no LDS round trips):
// Kogge-Stone inside each row of 16 lanes, then the row totals are broadcast forward.
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v) {
#define STRD_DPP_ADD(ctrl, row_mask) \
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, row_mask, 0xF, true)
    STRD_DPP_ADD(0x111, 0xF);  // row_shr:1
    STRD_DPP_ADD(0x112, 0xF);  // row_shr:2
    STRD_DPP_ADD(0x114, 0xF);  // row_shr:4
    STRD_DPP_ADD(0x118, 0xF);  // row_shr:8
    STRD_DPP_ADD(0x142, 0xA);  // row_bcast:15 into rows 1 and 3
    STRD_DPP_ADD(0x143, 0xC);  // row_bcast:31 into rows 2 and 3
#undef STRD_DPP_ADD
    return v;
}

__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
#define STRD_DPP_MAX(ctrl, row_mask) \
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, ctrl, row_mask, 0xF, false))
    STRD_DPP_MAX(0x111, 0xF);
    STRD_DPP_MAX(0x112, 0xF);
    STRD_DPP_MAX(0x114, 0xF);
    STRD_DPP_MAX(0x118, 0xF);
    STRD_DPP_MAX(0x142, 0xA);
    STRD_DPP_MAX(0x143, 0xC);
#undef STRD_DPP_MAX
    return (uint32_t)__builtin_amdgcn_readlane((int)v, kWave - 1);
}

// Smallest and largest key of the workgroup; a barrier.  buf is not written again without another one.
__device__ __forceinline__ void block_range(uint32_t (&buf)[2][kWaves], uint32_t &kmin, uint32_t &kmax) {
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const uint32_t inv = wave_max(~kmin), top = wave_max(kmax);
    if (lane == 0) {
        buf[0][wave] = inv;
        buf[1][wave] = top;
    }
    __syncthreads();
    kmin = ~wave_max(buf[0][lane & (kWaves - 1)]);
    kmax = wave_max(buf[1][lane & (kWaves - 1)]);
}

// Cross-wave step of up to kBatch workgroup scans that share one barrier.  Before the call every wave
// has stored the inclusive total of scan b in sums[b][wave].  Every wave turns the rows of 16 wave totals into
// offsets for itself, four rows at a time (a DPP row of 16 lanes is exactly one scan): exclusive
// offset of this wave and grand total of every scan.  The sums may be written again after one more barrier.
struct ScanScratch {
    uint32_t sums[kBatch][kWaves];
};
template <int B>
__device__ __forceinline__ void finish_scans(const ScanScratch &sc, uint32_t (&base)[B], uint32_t (&total)[B]) {
    static_assert(kWaves == 16 && B <= kBatch, "a scan is one row of 16 lanes");
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    __syncthreads();
#pragma unroll
    for (int b0 = 0; b0 < B; b0 += 4) {
        const uint32_t v = sc.sums[b0 + lane / kWaves][lane % kWaves];
        uint32_t inc = v;
#define STRD_DPP_ADD(ctrl) inc += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)inc, ctrl, 0xF, 0xF, true)
        STRD_DPP_ADD(0x111);
        STRD_DPP_ADD(0x112);
        STRD_DPP_ADD(0x114);
        STRD_DPP_ADD(0x118);
#undef STRD_DPP_ADD
#pragma unroll
        for (int b = b0; b < (b0 + 4 < B ? b0 + 4 : B); ++b) {
            base[b] = (uint32_t)__builtin_amdgcn_readlane((int)(inc - v), (b - b0) * kWaves + wave);
            total[b] = (uint32_t)__builtin_amdgcn_readlane((int)inc, (b - b0) * kWaves + kWaves - 1);
        }
    }
}

// After a histogram pass: find the bin (scanning from the top) that holds the k-th largest key
// and reduce k to its rank inside that bin.  All threads return the same (bin, k).  Thread t owns
// bins 2047 - t and 1023 - t, so neighbouring threads read neighbouring 64-byte groups of copies.
template <int COPIES>
__device__ __forceinline__ void pick_bin(const uint32_t *hist, ScanScratch &sc, uint32_t *found, uint32_t &k,
                                         uint32_t &bin) {
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int d_hi = kBins - 1 - threadIdx.x, d_lo = d_hi - kThreads;
    uint32_t c_hi = 0, c_lo = 0;
    if (COPIES >= 4) {
#pragma unroll
        for (int c = 0; c < COPIES; c += 4) {
            const uint4 a = *reinterpret_cast<const uint4 *>(&hist[d_hi * COPIES + c]);
            const uint4 b = *reinterpret_cast<const uint4 *>(&hist[d_lo * COPIES + c]);
            c_hi += a.x + a.y + a.z + a.w;
            c_lo += b.x + b.y + b.z + b.w;
        }
    } else {
#pragma unroll
        for (int c = 0; c < COPIES; ++c) {
            c_hi += hist[d_hi * COPIES + c];
            c_lo += hist[d_lo * COPIES + c];
        }
    }
    const uint32_t i_hi = wave_inclusive_scan(c_hi), i_lo = wave_inclusive_scan(c_lo);
    if (lane == kWave - 1) {
        sc.sums[0][wave] = i_hi;
        sc.sums[1][wave] = i_lo;
    }
    uint32_t base[2], total[2];
    finish_scans(sc, base, total);
    // keys in higher bins than this thread's: all upper-half bins come before any lower-half bin
    const uint32_t above_hi = base[0] + i_hi - c_hi;
    const uint32_t above_lo = total[0] + base[1] + i_lo - c_lo;
    if (above_hi < k && k <= above_hi + c_hi) {
        found[0] = (uint32_t)d_hi;
        found[1] = k - above_hi;
        found[2] = c_hi;
    } else if (above_lo < k && k <= above_lo + c_lo) {
        found[0] = (uint32_t)d_lo;
        found[1] = k - above_lo;
        found[2] = c_lo;
    }
    __syncthreads();
    bin = found[0];
    k = found[1];
}

// The k-th largest of the c <= kRankKeys values in cand (LDS, published by a barrier before the call) and how many
// values equal to it are kept: every lane of wave 0 counts the values above and equal to its own.  A barrier.
__device__ __forceinline__ void rank_few(const uint32_t *cand, uint32_t c, uint32_t k, uint32_t (&ranked)[2]) {
    const int tid = threadIdx.x;
    if (tid < kWave) {
        c = (uint32_t)__builtin_amdgcn_readfirstlane((int)c);
        const uint32_t mine = (uint32_t)tid < c ? cand[tid] : 0u;
        uint32_t above = 0, equal = 0;
        for (uint32_t j = 0; j < c; ++j) {
            const uint32_t other = (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)j);
            above += other > mine ? 1u : 0u;
            equal += other == mine ? 1u : 0u;
        }
        if ((uint32_t)tid < c && above < k && k <= above + equal) {  // lanes with equal keys agree
            ranked[0] = mine;
            ranked[1] = k - above;
        }
    }
    __syncthreads();
}

// TILES > 0: N <= TILES * kTile and every key stays in registers.  TILES == 0: streaming.
// SEQ = SeqTab: one workgroup per sequence of a packed batch (scores of sequence b start at
// scores + b * ld, its indices at idx + koff[b]; N and K are the table's).
template <int TILES, class SEQ = OneSeq>
__global__ __launch_bounds__(kThreads) void select_topk_kernel(const float *__restrict__ scores, int N, int K,
                                                               int32_t *__restrict__ idx, SEQ seq, int ld) {
    if constexpr (is_varlen<SEQ>()) {
        const int b = blockIdx.x;
        N = seq.N[b];
        K = seq.K[b];
        scores += (size_t)b * ld;
        idx += seq.koff[b];
    }
    constexpr int kCop = kCopies<TILES>;
    extern __shared__ __attribute__((aligned(16))) uint32_t hist[];  // [kBins][kCop]
    __shared__ ScanScratch scan[2];          // taken in turn by the batches of the write-out
    __shared__ uint32_t range[2][kWaves];
    __shared__ uint32_t found[3][3];         // (bin, rank inside the bin, keys in the bin) of each pass
    __shared__ uint32_t cand[kRankKeys];     // direct ranking: the keys (less kmin) still in play
    __shared__ uint32_t ncand, ranked_key[2];
    const int tid = threadIdx.x;
    if (tid == 0) ncand = 0u;                // published by the first barrier below
    const int ntiles = (N + kTile - 1) / kTile;
    auto zero_hist = [&](int copies) {
        for (int b = tid * 4; b < kBins * copies; b += kThreads * 4)
            *reinterpret_cast<uint4 *>(&hist[b]) = make_uint4(0, 0, 0, 0);
    };
    zero_hist(kCop);

    constexpr int kHeld = TILES > 0 ? TILES : 1;
    uint32_t held[kHeld][4];
    if (TILES > 0) {
#pragma unroll
        for (int t = 0; t < kHeld; ++t) load_tile(scores, N, t, held[t]);
    }
    // Visit every key this lane owns; f is inlined into both variants.
    auto for_each_key = [&](auto &&f) {
        if (TILES > 0) {
#pragma unroll
            for (int t = 0; t < kHeld; ++t)
#pragma unroll
                for (int u = 0; u < 4; ++u) f(held[t][u]);
        } else {
            for (int t0 = 0; t0 < ntiles; t0 += kBatch) {
                uint32_t key[kBatch][4];
#pragma unroll
                for (int b = 0; b < kBatch; ++b) load_tile(scores, N, t0 + b, key[b]);  // past-the-end tiles give 0
#pragma unroll
                for (int b = 0; b < kBatch; ++b)
#pragma unroll
                    for (int u = 0; u < 4; ++u) f(key[b][u]);
            }
        }
    };

    // ---- radix select: exact key of the K-th largest score --------------------------------
    // Importance scores are close together (all scores of a layer within a factor of two is
    // normal), so the leading bits of the keys say nothing: the digits are taken from
    // rel = key - (smallest key) instead, whose nbits significant bits are cut into 11-bit digits
    // from the top.  Scores within a factor of two need two passes instead of three, and the keys
    // spread over the bins instead of crowding a few.
    // (When the keys do not fit the registers, finding the smallest key would cost one more pass
    // over memory, as much as the digit it may save: the raw keys are used then.)
    uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
    if (TILES > 0) {
        for_each_key([&](uint32_t key) {
            if (key) {  // 0 marks the slots past the end of the array
                kmin = min(kmin, key);
                kmax = max(kmax, key);
            }
        });
    } else {
        kmin = 0u;
        kmax = 0xFFFFFFFFu;
    }
    block_range(range, kmin, kmax);  // its barrier also publishes the cleared histogram
    const int nbits = 32 - __clz(kmax - kmin);     // 0 when all scores are equal
    const int npass = (nbits + 10) / 11;           // uniform
    // Pass 0 sees every key: 16 copies per bin, whatever the distribution.  A later pass only counts
    // the keys of one bin of the pass before; when those are few, their digits rarely collide and a
    // histogram with 2 copies per bin is 8 times cheaper to clear and to scan.
    uint32_t k = (uint32_t)K, prefix = 0;          // prefix: the digits of rel fixed so far, in place
    int shift_prev = 32;
    bool few = false, ranked = false;
    for (int pass = 0; pass < npass; ++pass) {
        if (pass > 0 && found[pass - 1][2] <= (uint32_t)kRankKeys) {  // uniform
            // The bin of the pass before holds a wave's worth of keys at most: collect them and let every
            // lane of wave 0 count the keys above and equal to its own -- two barriers instead of one or
            // two more histogram passes of five each.
            const uint32_t pfx = prefix >> shift_prev;
            for_each_key([&](uint32_t key) {
                const uint32_t rel = key - kmin;
                if (key != 0 && (rel >> shift_prev) == pfx) cand[atomicAdd(&ncand, 1u)] = rel;
            });
            __syncthreads();
            rank_few(cand, ncand, k, ranked_key);
            ranked = true;
            break;
        }
        const int shift = max(nbits - 11 * (pass + 1), 0);
        const uint32_t dmask = (1u << min(11, nbits - 11 * pass)) - 1u;
        uint32_t bin;
        if (pass > 0) {  // every lane has read its bins before the barrier inside pick_bin
            zero_hist(few ? kFewCopies : kCop);
            __syncthreads();
        }
        const uint32_t pfx = shift_prev < 32 ? prefix >> shift_prev : 0u;
        if (few) {
            for_each_key([&](uint32_t key) {
                const uint32_t rel = key - kmin;
                hist_add<kFewCopies>(hist, (rel >> shift) & dmask, key != 0 && (shift_prev >= 32 || (rel >> shift_prev) == pfx));
            });
            __syncthreads();
            pick_bin<kFewCopies>(hist, scan[0], found[pass], k, bin);
        } else {
            for_each_key([&](uint32_t key) {
                const uint32_t rel = key - kmin;
                hist_add<kCop>(hist, (rel >> shift) & dmask, key != 0 && (shift_prev >= 32 || (rel >> shift_prev) == pfx));
            });
            __syncthreads();
            pick_bin<kCop>(hist, scan[0], found[pass], k, bin);
        }
        prefix |= bin << shift;
        few = found[pass][2] <= kFewKeys;  // uniform
        shift_prev = shift;
    }
    // key of the K-th largest score (a real score: > 0) and how many keys equal to it survive (the first ones)
    const uint32_t thresh = kmin + (ranked ? ranked_key[0] : prefix);
    const uint32_t keep_eq = ranked ? ranked_key[1] : k;

    // ---- ordered write-out: kHold tiles per barrier -----------------------------------------
    constexpr int kHold = TILES > 0 ? TILES : kBatch;
    static_assert(kHold <= kBatch, "one batch when the keys stay in registers");
    uint32_t out_base = 0, eq_base = 0;  // survivors / duplicates of thresh seen in earlier tiles
    auto emit_batch = [&](int t0, const uint32_t (&key)[kHold][4], ScanScratch &sc) {
        const int lane = tid & (kWave - 1), wave = tid / kWave;
        uint32_t cnt[kHold], inc[kHold], base[kHold], total_of[kHold];  // low 16 bits: keys > thresh, high 16 bits: keys == thresh
#pragma unroll
        for (int b = 0; b < kHold; ++b) {
            cnt[b] = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u)
                cnt[b] += (key[b][u] > thresh ? 1u : 0u) + (key[b][u] == thresh ? 0x10000u : 0u);
            inc[b] = wave_inclusive_scan(cnt[b]);
            if (lane == kWave - 1) sc.sums[b][wave] = inc[b];
        }
        finish_scans(sc, base, total_of);
#pragma unroll
        for (int b = 0; b < kHold; ++b) {
            if (t0 + b < ntiles) {  // uniform
                const uint32_t total = total_of[b];
                const uint32_t ex = base[b] + inc[b] - cnt[b];
                const int i0 = (t0 + b) * kTile + tid * 4;
                uint32_t gt_before = ex & 0xFFFFu, eq_before = eq_base + (ex >> 16);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const bool gt = key[b][u] > thresh, eq = key[b][u] == thresh;
                    if (gt || (eq && eq_before < keep_eq)) {
                        const uint32_t eq_kept = min(eq_before, keep_eq) - min(eq_base, keep_eq);
                        idx[out_base + gt_before + eq_kept] = i0 + u;
                    }
                    gt_before += gt ? 1u : 0u;
                    eq_before += eq ? 1u : 0u;
                }
                const uint32_t eq_tile = total >> 16;
                out_base += (total & 0xFFFFu) + (min(eq_base + eq_tile, keep_eq) - min(eq_base, keep_eq));
                eq_base += eq_tile;
            }
        }
    };
    if constexpr (TILES > 0) {
        emit_batch(0, held, scan[0]);
    } else {
        for (int t0 = 0; t0 < ntiles; t0 += kHold) {
            uint32_t key[kHold][4];
#pragma unroll
            for (int b = 0; b < kHold; ++b) load_tile(scores, N, t0 + b, key[b]);
            emit_batch(t0, key, scan[(t0 / kHold) & 1]);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Wide form, 32768 < N <= kWideMax * 4096: one workgroup per 4096-score tile and a chain of five short launches
// instead of one workgroup that streams the scores four times.  At these sizes the time is the
// launches, so there are as few as the dependences allow without one workgroup waiting for another:
//   range    smallest and largest key of every tile (and the histograms cleared)
//   hist     histogram of the first 11-bit digit of key - min(key), one for all tiles
//   collect  every workgroup picks the bin that holds the K-th key for itself; the keys of that bin ("candidates":
//            their remaining bits and tile) go into one list, every tile leaves its counts of keys above the bin and
//            in it.  More candidates than the list holds (close scores beside zeros or an outlier) are counted by the
//            next digit instead, and
//   collect  is made again for that one (otherwise, 2 us, it has nothing to do).  Still too many: only the last 10 bits
//            are open then, and every tile leaves a table of how many of its candidates lie at or above each value.
//   emit     every workgroup ranks the candidates for itself, from the list or by a third digit, counts what the
//            tiles before it keep -- the keys above the bin from their counts, the others from the list or their
//            tables -- and writes its tile in order.
// Candidates that are all one value need neither.  No workgroup reads another's scores, whatever their values, and no
// more than kWideCand equal keys meet on one counter in emit (a list of 32768 without the tables took 45 us instead of 21 at
// 65536 close scores and a zero, 343 instead of 33 at 2^20, 51 instead of 16 where half the scores are one value).  (Appends,
// table reads and writes are bounded: calls that overlap on the array of the form without a
// workspace race, with wrong results but inside their buffers.)  The list is in no particular order, only the values in it
// count: the result is bit-exact and deterministic.  Six launches, with a global histogram per digit of the raw
// keys and the survivors counted in a launch of their own, took 24 us at 36864 to 131072 scores and 52
// at 2^20 (back to back, workspace from an allocator); these take 16 to 17 (21 where a second digit is needed), 24 to 33.
constexpr int kWideMax = 256;     // tiles (workgroups) at most
constexpr int kWideCopies = 4;    // copies of a bin in the local histogram of one tile
constexpr int kWideCand = 4096;   // candidates the list holds
constexpr int kLowBits = 21;      // a candidate is its bits below the first digit (at most 21) and, above them, its tile
constexpr int kLastBins = 1024;   // values of the bits below the second digit
static_assert(kWideMax <= 1 << (32 - kLowBits), "the tile fits above the low bits");

struct WideWs {
    uint32_t ghist[3][kBins];      // histograms of the first digit and, where they are needed, the second and the third
    uint32_t ncand;                // candidates in the list
    uint32_t low_inv, low_max;     // complement of their smallest low bits, their largest; these three follow ghist
    uint32_t kmin;                 // smallest key of all
    struct {
        uint32_t shift, bin;       // bits below the digits picked so far, the picked bin: (key - kmin) >> shift
        uint32_t k, count;         // rank of the K-th key inside the bin, keys in the bin
    } pick[2];                     // after one digit, after two
    uint32_t range[kWideMax][2];   // per tile: smallest and largest key
    uint32_t counts[kWideMax][2];  // per tile: keys above the bin, keys in it
    uint32_t cand[kWideCand];
    uint16_t from[kWideMax][kLastBins];  // per tile, two digits picked: keys in the bin whose low bits are at least so much
};

__global__ __launch_bounds__(kThreads) void topk_wide_range_kernel(const float *__restrict__ scores, int N, WideWs *ws) {
    __shared__ uint32_t buf[2][kWaves];
    uint32_t key[4];
    load_tile(scores, N, blockIdx.x, key);
    for (int i = blockIdx.x * kThreads + threadIdx.x; i < 3 * kBins; i += gridDim.x * kThreads) ws->ghist[i / kBins][i % kBins] = 0u;
    if (blockIdx.x == 0 && threadIdx.x == 0) ws->ncand = ws->low_inv = ws->low_max = 0u;
    uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (key[u]) {
            kmin = min(kmin, key[u]);
            kmax = max(kmax, key[u]);
        }
    block_range(buf, kmin, kmax);
    if (threadIdx.x == 0) {
        ws->range[blockIdx.x][0] = kmin;
        ws->range[blockIdx.x][1] = kmax;
    }
}

// Smallest key of all tiles and the number of bits below the first digit; a barrier.
__device__ __forceinline__ void wide_range(const WideWs *ws, uint32_t (&buf)[2][kWaves], uint32_t &kmin, int &shift) {
    uint32_t kmax = 0u;
    kmin = 0xFFFFFFFFu;
    if (threadIdx.x < gridDim.x) {
        kmin = ws->range[threadIdx.x][0];
        kmax = ws->range[threadIdx.x][1];
    }
    block_range(buf, kmin, kmax);
    shift = max(32 - __clz(kmax - kmin) - 11, 0);
}

__global__ __launch_bounds__(kThreads) void topk_wide_hist_kernel(const float *__restrict__ scores, int N, WideWs *ws) {
    __shared__ __attribute__((aligned(16))) uint32_t hist[kBins * kWideCopies];
    __shared__ uint32_t buf[2][kWaves];
    const int tid = threadIdx.x;
    uint32_t key[4], kmin;
    load_tile(scores, N, blockIdx.x, key);
    for (int b = tid * 4; b < kBins * kWideCopies; b += kThreads * 4)
        *reinterpret_cast<uint4 *>(&hist[b]) = make_uint4(0, 0, 0, 0);
    int shift;
    wide_range(ws, buf, kmin, shift);  // its barrier publishes the cleared histogram
#pragma unroll
    for (int u = 0; u < 4; ++u) hist_add<kWideCopies>(hist, (key[u] - kmin) >> shift, key[u] != 0);
    __syncthreads();
    for (int b = tid; b < kBins; b += kThreads) {
        const uint4 c = *reinterpret_cast<const uint4 *>(&hist[b * kWideCopies]);
        const uint32_t n = c.x + c.y + c.z + c.w;
        if (n) atomicAdd(&ws->ghist[0][b], n);
    }
}

template <int PASS>
__global__ __launch_bounds__(kThreads) void topk_wide_collect_kernel(const float *__restrict__ scores, int N, int K,
                                                                       WideWs *ws) {
    __shared__ __attribute__((aligned(16))) uint32_t hist[kBins * kWideCopies];  // the picked digit's, then the next one's
    __shared__ uint32_t buf[2][kWaves];
    __shared__ ScanScratch scan;
    __shared__ uint32_t found[3], list_base;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    uint32_t key[4], kmin, bin, k = (uint32_t)K;
    if constexpr (PASS == 1) {
        const uint32_t c = ws->pick[0].count;
        if (c <= (uint32_t)kWideCand || ~ws->low_inv == ws->low_max) return;  // uniform, the same in every workgroup
    }
    load_tile(scores, N, blockIdx.x, key);
    for (int b = tid; b < kBins; b += kThreads) hist[b] = ws->ghist[PASS][b];
    int shift;
    wide_range(ws, buf, kmin, shift);  // its barrier publishes the bins
    uint32_t prefix = 0;
    if constexpr (PASS == 1) {
        prefix = ws->pick[0].bin << (shift - max(shift - 11, 0));
        k = ws->pick[0].k;
        shift = max(shift - 11, 0);
    }
    pick_bin<1>(hist, scan, found, k, bin);
    const uint32_t count = found[2];
    bin |= prefix;
    uint32_t cnt = 0, low_min = 0xFFFFFFFFu, low_max = 0u;  // cnt: low 16 bits: keys above the bin, high 16 bits: keys in it
    const uint32_t low = (1u << shift) - 1u;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const uint32_t rel = key[u] - kmin, d = rel >> shift;
        if (key[u]) cnt += (d > bin ? 1u : 0u) + (d == bin ? 0x10000u : 0u);
        if (key[u] && d == bin) {
            low_min = min(low_min, rel & low);
            low_max = max(low_max, rel & low);
        }
    }
    const uint32_t inc = wave_inclusive_scan(cnt);
    if (lane == kWave - 1) scan.sums[0][wave] = inc;
    uint32_t base[1], total[1];
    finish_scans(scan, base, total);
    const bool listed = count <= (uint32_t)kWideCand;  // the same in every workgroup
    if (tid == 0) {
        ws->counts[blockIdx.x][0] = total[0] & 0xFFFFu;
        ws->counts[blockIdx.x][1] = total[0] >> 16;
        list_base = listed ? atomicAdd(&ws->ncand, total[0] >> 16) : 0u;
        if (blockIdx.x == 0) {
            ws->kmin = kmin;
            ws->pick[PASS].shift = (uint32_t)shift;
            ws->pick[PASS].bin = bin;
            ws->pick[PASS].k = k;
            ws->pick[PASS].count = count;
        }
    }
    if (total[0] >> 16 == 0) return;  // uniform
    if (listed) {
        __syncthreads();
        uint32_t at = list_base + ((base[0] + inc - cnt) >> 16);  // all tiles together append `count` <= kWideCand keys
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t rel = key[u] - kmin;
            if (key[u] && rel >> shift == bin && at < (uint32_t)kWideCand) ws->cand[at++] = (rel & low) | blockIdx.x << kLowBits;
        }
    } else if (PASS == 0 || shift > 0) {
        const int next = PASS == 0 ? max(shift - 11, 0) : 0;
        for (int b = tid * 4; b < kBins * kWideCopies; b += kThreads * 4)  // (all have read their bins: barriers in pick_bin)
            *reinterpret_cast<uint4 *>(&hist[b]) = make_uint4(0, 0, 0, 0);
        block_range(buf, low_min, low_max);  // its barrier publishes the cleared histogram
        if (PASS == 0 && tid == 0) {
            atomicMax(&ws->low_inv, ~low_min);
            atomicMax(&ws->low_max, low_max);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t rel = key[u] - kmin;
            hist_add<kWideCopies>(hist, (rel & low) >> next, key[u] != 0 && rel >> shift == bin);
        }
        __syncthreads();
        auto bin_count = [&](int b) {
            const uint4 c = *reinterpret_cast<const uint4 *>(&hist[b * kWideCopies]);
            return c.x + c.y + c.z + c.w;
        };
        for (int b = tid; b < kBins; b += kThreads) {
            const uint32_t n = bin_count(b);
            if (n) atomicAdd(&ws->ghist[PASS + 1][b], n);
        }
        if constexpr (PASS == 1) {  // thread t: the value kLastBins - 1 - t, so that the scan adds up from the top
            static_assert(kLastBins == kThreads, "a value per thread");
            const int b = kLastBins - 1 - tid;
            const uint32_t at_least = wave_inclusive_scan(bin_count(b));
            if (lane == kWave - 1) scan.sums[0][wave] = at_least;
            finish_scans(scan, base, total);
            ws->from[blockIdx.x][b] = (uint16_t)(base[0] + at_least);
        }
    }
}

__global__ __launch_bounds__(kThreads) void topk_wide_emit_kernel(const float *__restrict__ scores, int N, int K,
                                                                    const WideWs *__restrict__ ws,
                                                                    int32_t *__restrict__ idx) {
    __shared__ __attribute__((aligned(16))) uint32_t hist[kBins * kFewCopies];
    __shared__ ScanScratch scan[2];
    __shared__ uint32_t found[2][3], cand[kRankKeys], ncand, ranked[2];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    uint32_t key[4];
    load_tile(scores, N, blockIdx.x, key);
    uint32_t before_gt = 0, before_eq = 0;  // this thread's share of the keys above / in the bin in earlier tiles
    if (tid < (int)blockIdx.x) {
        before_gt = ws->counts[tid][0];
        before_eq = ws->counts[tid][1];
    }
    // one digit was enough, or the candidates are one value, or a second was picked
    const bool over = ws->pick[0].count > (uint32_t)kWideCand, one_value = over && ~ws->low_inv == ws->low_max;
    const int last = over && !one_value ? 1 : 0;
    const uint32_t kmin = ws->kmin, bin = ws->pick[last].bin, count = ws->pick[last].count;
    const int shift = (int)ws->pick[last].shift;
    uint32_t k = ws->pick[last].k;                 // -> how many keys equal to the threshold survive
    uint32_t t_low = one_value ? ws->low_max : 0;  // -> the threshold's low bits
    if (tid == 0) ncand = 0u;
    // f(low bits) of every key in the list that is in one of the first `tiles` tiles
    auto for_each_candidate = [&](int tiles, auto &&f) __attribute__((always_inline)) {
        for (uint32_t i = tid; i < count; i += kThreads) {
            const uint32_t c = ws->cand[i];
            if (c >> kLowBits < (uint32_t)tiles) f(c & ((1u << kLowBits) - 1u));
        }
    };
    // uniform, as everything below: the low bits decide, ...
    if (shift > 0 && !one_value && count > (uint32_t)kWideCand) {  // ... by one more digit and the tiles' tables
        for (int b = tid; b < kBins; b += kThreads) hist[b] = ws->ghist[2][b];
        __syncthreads();
        pick_bin<1>(hist, scan[0], found[0], k, t_low);
        if (tid < (int)blockIdx.x) {
            const uint32_t at = min(t_low, (uint32_t)kLastBins - 1), above = at + 1 < kLastBins ? ws->from[tid][at + 1] : 0u;
            const bool any = before_eq > 0;  // (a tile without keys in the bin leaves no table)
            before_gt += any ? above : 0u;
            before_eq = any ? ws->from[tid][at] - above : 0u;
        }
    } else if (shift > 0 && !one_value) {  // ... by digits of the list until few keys are left
        uint32_t left = count;
        int known = shift;  // the bits of t_low from here on are fixed
        for (int pass = 0; pass < 2 && known > 0 && left > (uint32_t)kRankKeys; ++pass) {
            const int sh = max(known - 11, 0);
            for (int b = tid * 4; b < kBins * kFewCopies; b += kThreads * 4)
                *reinterpret_cast<uint4 *>(&hist[b]) = make_uint4(0, 0, 0, 0);
            __syncthreads();
            for_each_candidate((int)gridDim.x, [&](uint32_t c) {
                hist_add<kFewCopies>(hist, (c >> sh) & (kBins - 1), c >> known == t_low >> known);
            });
            __syncthreads();
            uint32_t digit;
            pick_bin<kFewCopies>(hist, scan[0], found[pass], k, digit);
            t_low |= digit << sh;
            left = found[pass][2];
            known = sh;
        }
        if (known > 0) {
            __syncthreads();  // ncand
            for_each_candidate((int)gridDim.x, [&](uint32_t c) {
                if (c >> known == t_low >> known) cand[atomicAdd(&ncand, 1u) & (kRankKeys - 1)] = c;
            });
            __syncthreads();
            rank_few(cand, left, k, ranked);
            t_low = ranked[0];
            k = ranked[1];
        }
        before_eq = 0;
        for_each_candidate((int)blockIdx.x, [&](uint32_t c) {
            before_gt += c > t_low ? 1u : 0u;
            before_eq += c == t_low ? 1u : 0u;
        });
    }
    const uint32_t thresh = kmin + (bin << shift | t_low), keep_eq = k;
    uint32_t cnt = 0;  // low 16 bits: keys > thresh, high 16 bits: keys == thresh
#pragma unroll
    for (int u = 0; u < 4; ++u) cnt += (key[u] > thresh ? 1u : 0u) + (key[u] == thresh ? 0x10000u : 0u);
    const uint32_t inc = wave_inclusive_scan(cnt), inc_gt = wave_inclusive_scan(before_gt), inc_eq = wave_inclusive_scan(before_eq);
    if (lane == kWave - 1) {
        scan[1].sums[0][wave] = inc;
        scan[1].sums[1][wave] = inc_gt;
        scan[1].sums[2][wave] = inc_eq;
    }
    uint32_t base[3], total[3];
    finish_scans(scan[1], base, total);
    const uint32_t eq_base = total[2], out_base = total[1] + min(eq_base, keep_eq);
    const uint32_t ex = base[0] + inc - cnt;
    const int i0 = blockIdx.x * kTile + tid * 4;
    uint32_t gt_before = ex & 0xFFFFu, eq_before = eq_base + (ex >> 16);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const bool gt = key[u] > thresh, eq = key[u] == thresh;
        if (gt || (eq && eq_before < keep_eq)) {
            const uint32_t eq_kept = min(eq_before, keep_eq) - min(eq_base, keep_eq);
            const uint32_t o = out_base + gt_before + eq_kept;
            if (o < (uint32_t)K) idx[o] = i0 + u;
        }
        gt_before += gt ? 1u : 0u;
        eq_before += eq ? 1u : 0u;
    }
}

template <int TILES, class SEQ>
int launch_select(const float *scores, int N, int K, int32_t *idx, const SEQ &seq, int ld, int nseq, hipStream_t s) {
    const size_t smem = (size_t)kBins * kCopies<TILES> * sizeof(uint32_t);
    if (!allow_dynamic_lds(reinterpret_cast<const void *>(&select_topk_kernel<TILES, SEQ>), smem)) return STRD_EHIP;
    select_topk_kernel<TILES, SEQ><<<nseq, kThreads, smem, s>>>(scores, N, K, idx, seq, ld);
    return launch_status();
}

}  // namespace

size_t select_topk_ws(int N) {
    return (N > 8 * kTile && N <= kWideMax * kTile) ? align_up(sizeof(WideWs), 256) : 0;
}

int select_topk_varlen_max_n() { return 8 * kTile; }

int select_topk_varlen_launch(const float *scores, int ld, const SeqTab &tab, int nseq, int max_n, int32_t *idx,
                              hipStream_t s) {
    return max_n <= kTile       ? launch_select<1>(scores, 0, 0, idx, tab, ld, nseq, s)
           : max_n <= 2 * kTile ? launch_select<2>(scores, 0, 0, idx, tab, ld, nseq, s)
           : max_n <= 4 * kTile ? launch_select<4>(scores, 0, 0, idx, tab, ld, nseq, s)
                                : launch_select<8>(scores, 0, 0, idx, tab, ld, nseq, s);
}

int select_topk_launch(const float *scores, int N, int K, int32_t *idx, void *ws, hipStream_t s) {
    if (select_topk_ws(N)) {
        WideWs *w = reinterpret_cast<WideWs *>(ws);
        const int G = ceil_div(N, kTile);
        topk_wide_range_kernel<<<G, kThreads, 0, s>>>(scores, N, w);
        topk_wide_hist_kernel<<<G, kThreads, 0, s>>>(scores, N, w);
        topk_wide_collect_kernel<0><<<G, kThreads, 0, s>>>(scores, N, K, w);
        topk_wide_collect_kernel<1><<<G, kThreads, 0, s>>>(scores, N, K, w);
        topk_wide_emit_kernel<<<G, kThreads, 0, s>>>(scores, N, K, w, idx);
        return launch_status();
    }
    return N <= kTile       ? launch_select<1>(scores, N, K, idx, OneSeq(), 0, 1, s)
           : N <= 2 * kTile ? launch_select<2>(scores, N, K, idx, OneSeq(), 0, 1, s)
           : N <= 4 * kTile ? launch_select<4>(scores, N, K, idx, OneSeq(), 0, 1, s)
           : N <= 8 * kTile ? launch_select<8>(scores, N, K, idx, OneSeq(), 0, 1, s)
                            : launch_select<0>(scores, N, K, idx, OneSeq(), 0, 1, s);
}

// ---- the same selection for callers that cannot allocate --------------------------------------
// The histograms and per-tile counts of the many-workgroup form live in an array that is part of
// the library's image instead of a caller-provided workspace: every GPU the library runs on
// holds its own copy at its own address for the life of the process.  In host code the array's
// name is only a handle for hipGetSymbolAddress; kernels are given the address that call returns
// for the current device.
constexpr int kStaticMaxN = kWideMax * kTile;   // 2^20 scores
constexpr size_t kStaticBytes = (sizeof(WideWs) + 255) / 256 * 256;
static __device__ __align__(256) __attribute__((used)) unsigned char scratch[kStaticBytes];

int select_topk_static_max_n() { return kStaticMaxN; }

int select_topk_static_launch(const float *scores, int N, int K, int32_t *idx, hipStream_t s) {
    constexpr int kMaxDev = 64;
    static std::mutex mu;
    static void *ptr[kMaxDev];   // device address of `scratch` on each GPU, looked up once
    if (N > kStaticMaxN || select_topk_ws(N) > kStaticBytes) return STRD_EUNSUPPORTED;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDev) return STRD_EHIP;
    void *p = nullptr;
    {
        std::lock_guard<std::mutex> lock(mu);
        if (!ptr[dev]) {
            void *q = nullptr;
            if (hipGetSymbolAddress(&q, HIP_SYMBOL(scratch)) != hipSuccess || !q) {
                (void)hipGetLastError();
                return STRD_EHIP;
            }
            ptr[dev] = q;
        }
        p = ptr[dev];
    }
    // every launch of the chain starts from a kernel that clears the histograms; the counts and
    // picked digits are written before they are read
    return select_topk_launch(scores, N, K, idx, p, s);
}

}  // namespace strd
