// ssd_prefill on bf16 matrix cores, four heads of a group per workgroup: the Mamba-2 recurrence (paper
// Eqs. "ssm_state_update", "ssm_output") in its chunked form, cut into segments that run side by side.
//
// Decomposition.  One workgroup owns four whole heads (P = 64) of one group and one segment of the sequence,
// which it walks in 32-token steps.  Per step and head, with l_t the in-step cumulative sum of dt*A (log2 units):
//   (a) G^T[j,t] = b_j . c_t                                      contraction over the state dim n
//   (b) M[t,j]   = G^T[j,t] * 2^(l_t-l_j) * dt_j  for j <= t, else 0;  M[t,t] += D   (fp32, then bf16)
//   (d) Y^T[p,t] = 2^(l_t) * sum_n S[p,n] c_t[n]                  S = state before the step
//   (c) Y^T[p,t] += sum_j x_j[p] M[t,j]                           contraction over tokens
//   (e) S^T[n,p] = 2^(l_Q) S^T[n,p] + sum_j b_j[n] (w_j x_j[p]),  w_j = dt_j 2^(l_Q-l_j)
// every product a v_mfma_f32_16x16x32_bf16: 32 tokens are one contraction of (c) and (e).
//
// Waves (12, three per SIMD, 168 registers each).  Eight compute waves, two per head, each with a slab of 32 channels whose state
// S^T[n, 32] stays in fp32 accumulator registers for the whole segment; they do (d), (c), (e) and store the outputs, so an output is summed
// in fp32 from its first term to its last and rounded once.  Two G waves make the weights M of two heads each, one step ahead, and leave them
// in LDS in the operand layout of (c): (a) is the same for every head of a group.  One wave requests the asynchronous global -> LDS copies
// of the B, C and x tiles (three steps ahead), one helper wave dt, the scans l_t with everything that follows from them (two steps ahead) and
// the row tables of the gather form.  One LDS-only barrier per step.
//
// The accumulator layout of (e) is at the same time the A-operand layout of (d) (the contraction index n runs over the
// accumulator rows a lane holds), so the state is converted to bf16 in registers and never passes through LDS.  Column m of a
// slab's 16-channel tile pt is channel 8 (m / 4) + 4 pt + m % 4: a lane then holds 8 consecutive channels of its token and stores 16 bytes.
//
// Why four heads and 32 tokens.  With two heads per workgroup (ssd_seg) a step of 64 tokens takes 5400 cycles, this one of twice the heads and
// half the tokens 3400: the tiles of B and C cross the CU's copy path half as often and the b.c products are made for two heads at once
// instead of for each; every output is added up where its accumulators are, without a way through LDS and back through 16 bits; and each SIMD has two
// compute waves whose stalls the other fills.  What bounds a step: the vector instructions and products of the two compute waves of a SIMD do
// not overlap on this machine (36 products and 190 vector instructions each: 576 + 820 cycles of issue, 2600 measured for the pair without any
// LDS read, 2900 with them, 3160 with the G wave; copies, stores and G waves cost no cycles of a step but clock: 2.2 -> 1.85 GHz).
// Orders that changed nothing: products and vector work in turn or in blocks, with and without wave priorities, every LDS read a phase earlier, the
// copies dealt to three waves.
//
// Segments.  Each starts from a zero state (the first from S_in) and leaves its final local state and its total decay in the
// workspace; a second, small kernel adds what the true incoming state contributes to the tokens of each later segment,
//   y_t += 2^(l_t) * E c_t,   E = state at the segment's start, l_t = decay since then,
// for as long as 2^(l_t) is not zero in fp32, and completes S_out.  The first kSeamTok outputs of a later segment wait for that in fp32, so that
// where a head forgets within that many tokens no output is rounded twice.  Values that are not finite are never forgotten: a
// segment whose final state holds one says so, and the later segments then add it to all their tokens.
//
// GATHER: token t of the sequence is row idx[t] (t < K) or N + t - K of the tensors, i.e. the
// kernel reads the uncompacted x, dt, B, C through the kept-index list instead of a compacted copy.
#include "common.h"

namespace strd {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr int kQ = 32;      // tokens per step
constexpr int kHeads = 4;   // heads per workgroup
constexpr int kP = 64;      // channels per head
constexpr int kThreads = 768;
constexpr int kRB = 4;      // B / C tiles in LDS: of this step (compute waves), the next (G waves), two on their way
constexpr int kRX = 4;      // x tiles in LDS: of this step, three on their way
constexpr int kRD = 4;      // dt rows in LDS
constexpr int kSeamTok = 64;   // outputs of a later segment that are kept in fp32 for the seam (a multiple of the fix kernel's tile)
constexpr float kLog2e = 1.4426950408889634f;

struct QuadArgs {
    const bf16_t *x;
    const float *dt, *A;
    const bf16_t *B, *C;
    const float *D, *S_in;
    bf16_t *y;
    float *S_out;       // final state [H, P, n] or null
    float *lend;        // [nseg - 1, H, P, n]: final local state of every segment but the last
    float *ltot;        // [nseg, H]: total log2 decay of every segment
    uint32_t *lost;     // [nseg - 1, H, 2]: 1 where the final local state of a slab holds a value that is not finite
    float *seam;        // [nseg - 1, H, seg_steps * 32]: log2 decay of the tokens of a later segment since its start, while it is not zero
    int32_t *life;      // [nseg - 1, H]: for how many steps that is
    float *ybuf;        // [nseg - 1, kSeamTok, H * P]: first outputs of the later segments, before the seam
    const int32_t *idx;
    int N, K, T, H, G;
    int nseg, seg_steps;  // segments and 32-token steps per segment (the last may be shorter)
    int wg_per_seg;       // H / 4
};

template <int NS>
struct LdsQ {
    // A tile is filled 1 KB at a time (one copy instruction: lane l writes 16 bytes at 16 l): kRows rows of a tile after one another, then
    // 64 bytes nobody reads.  Inside a row of B or C the 16-byte pieces are permuted, piece v lies at v ^ (row % 4).  With that, the 8
    // rows two apart that a half wave passes to a transposing read share no bank, nor do the 16 rows of an 8-byte read.
    template <int ROW_BYTES>
    struct Tile {
        static constexpr int kRows = 1024 / ROW_BYTES;     // rows per copy instruction
        static constexpr int kIssues = kQ / kRows;
        static constexpr int kBlock = 16 / kRows * 1088;   // bytes between rows r and r + 16
        static __device__ __forceinline__ int row_at(int r) { return r / kRows * 1088 + r % kRows * ROW_BYTES; }
        alignas(64) char v[kIssues * 1088];
    };
    using TB = Tile<NS * 2>;
    using TX = Tile<kHeads * kP * 2>;
    struct alignas(16) Scan {
        float ell[kQ];    // inclusive cumulative sum of dt*A*log2(e) inside the step
        float dtv[kQ];    // dt (0 past the end of the sequence)
        float fw[16];     // key factors of the second query block: dt_j * 2^(l_15 - l_j), j < 16
        float w[kQ];      // weights of the state update, w_j = dt_j * 2^(l_Q - l_j), in slot order (slot_of)
        float carry[kQ];  // 2^(l_t); carry[kQ - 1] is the decay of the state over the step
    };
    bf16x8 m1[2][kHeads][64];  // weights of step i: [i % 2][head][lane], the B operand of (c) for the second query block
    bf16x4 m0[2][kHeads][64];  // ... for the first (token slots 0-3; the others are later tokens: zero)
    Scan scan[3][kHeads];
    float dt[kRD][2][64];    // [pair of heads][32 * (head % 2) + token]
    uint32_t rowtab[4][kQ];  // gather mode: source row of every token of local step i, i % 4 = slot
    int32_t rawidx[4][64];   // gather mode: entries of the kept-index list for local step i, i % 4 = slot (twice)
    TB b[kRB], c[kRB];
    TX x[kRX];
};
static_assert(sizeof(LdsQ<128>) <= 160 * 1024, "one workgroup must fit the 160 KB of LDS of a CU");

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ float fast_exp2(float v) { return __builtin_amdgcn_exp2f(v); }
__device__ __forceinline__ float read_lane_f32(float v, int l) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}
__device__ __forceinline__ bf16x8 cat8(bf16x4 lo, bf16x4 hi) {
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}
__device__ __forceinline__ bf16x4 to_bf16x4(f32x4 v) {
    return bf16x4{(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
}
// s_waitcnt immediate that waits until at most n vector-memory operations are outstanding
// (gfx9 layout: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[5:4] << 14); n < 64.
constexpr int lgkm_wait_imm(int n) { return 0xC07F | n << 8; }
constexpr int vm_wait_imm(int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }

// The contractions over tokens, (c) and (e), take the 32 tokens of a step in one order: k slot s of lane group lb is token
// 16 (s / 4) + state_tok(lb, s % 4), so that a half wave passes every other row of a tile to a transposing read (8 rows
// two apart share no bank at the pitches above).
__device__ __forceinline__ int state_tok(int lb, int j) { return 8 * (lb & 1) + 2 * j + (lb >> 1); }
// ... and the place of token j (< 32) in that order: 8 lb + s
__device__ __forceinline__ int slot_of(int j) { return 8 * (((j >> 3) & 1) + 2 * (j & 1)) + 4 * (j >> 4) + ((j & 7) >> 1); }

// The 8-byte pieces of one c row that a lane needs as B operand of (d): elements 32 ks + 4 lb .. + 3 (at e + 64 ks) and
// the same 16 further on (at o + 64 ks), for every k-step -- 2 KS plain reads (two in one instruction run at less than half
// the rate), requested together and waited for separately (same contract as lds_issue_tr8 / lds_settle8).
template <int KS, int OFF>
__device__ __forceinline__ void issue_c_pieces(uint32_t e, uint32_t o, strd_s16x4 (&r)[2 * KS]) {
    static_assert(KS == 2 || KS == 4, "state sizes 64 and 128");
    if constexpr (KS == 4)
        asm volatile(
            "ds_read_b64 %0, %8 offset:%10\n\tds_read_b64 %1, %9 offset:%10\n\tds_read_b64 %2, %8 offset:%11\n\t"
            "ds_read_b64 %3, %9 offset:%11\n\tds_read_b64 %4, %8 offset:%12\n\tds_read_b64 %5, %9 offset:%12\n\t"
            "ds_read_b64 %6, %8 offset:%13\n\tds_read_b64 %7, %9 offset:%13"
            : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7])
            : "v"(e), "v"(o), "i"(OFF), "i"(OFF + 64), "i"(OFF + 128), "i"(OFF + 192)
            : "memory");
    else
        asm volatile(
            "ds_read_b64 %0, %4 offset:%6\n\tds_read_b64 %1, %5 offset:%6\n\tds_read_b64 %2, %4 offset:%7\n\tds_read_b64 %3, %5 offset:%7"
            : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3])
            : "v"(e), "v"(o), "i"(OFF), "i"(OFF + 64)
            : "memory");
}
template <int KS>
__device__ __forceinline__ void settle_c_pieces(strd_s16x4 (&r)[2 * KS]) {
    if constexpr (KS == 4)
        lds_settle8(r);
    else
        lds_settle4(r);
}

// b^T fragments of four state tiles: transposing reads at e (tiles 0, 2) and o (1, 3), OFF bytes on, two 16-token blocks BLK bytes apart.
template <int OFF, int BLK>
__device__ __forceinline__ void issue_b_frags(uint32_t e, uint32_t o, strd_s16x4 (&r)[8]) {
    asm volatile(
        "ds_read_b64_tr_b16 %0, %8 offset:%10\n\t"
        "ds_read_b64_tr_b16 %1, %8 offset:%11\n\t"
        "ds_read_b64_tr_b16 %2, %9 offset:%10\n\t"
        "ds_read_b64_tr_b16 %3, %9 offset:%11\n\t"
        "ds_read_b64_tr_b16 %4, %8 offset:%12\n\t"
        "ds_read_b64_tr_b16 %5, %8 offset:%13\n\t"
        "ds_read_b64_tr_b16 %6, %9 offset:%12\n\t"
        "ds_read_b64_tr_b16 %7, %9 offset:%13"
        : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7])
        : "v"(e), "v"(o), "i"(OFF), "i"(OFF + BLK), "i"(OFF + 64), "i"(OFF + 64 + BLK)
        : "memory");
}

// The scheduler's order for the code before it: eight products, four vector instructions behind each (which also keeps the
// registers of the region within bounds).
__device__ __forceinline__ void eight_products_with_vector_work() {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x2, 4, 0);
    }
}

// Channel (in the head) of column m of tile pt of slab cw.
__device__ __forceinline__ int chan_of(int cw, int pt, int m) { return 32 * cw + 8 * (m >> 2) + 4 * pt + (m & 3); }

// ---- compute wave: slab cw (32 channels) of head hh of the workgroup: (d), (c), (e), the outputs ----
template <int NS>
__device__ __forceinline__ void compute_wave(LdsQ<NS> &lds, const QuadArgs &a, int hh, int cw, int h, int seg, int tok0, int nloc,
                                             const float *s_src, float *s_dst) {
    using L = LdsQ<NS>;
    constexpr int KS = NS / 32;  // k-steps of the products contracted over n
    constexpr int NT = NS / 16;  // 16-row tiles of the state
    const int lane = threadIdx.x & 63, lr = lane & 15, lb = lane >> 4;

    // state: S^T[n][p] tiles, rows n = 16 nt + 4 lb + i, columns p = chan_of(cw, pt, lr)
    f32x4 sacc[NT][2];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int pt = 0; pt < 2; ++pt) {
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            if (s_src) v = *reinterpret_cast<const f32x4 *>(s_src + ((size_t)h * kP + chan_of(cw, pt, lr)) * NS + 16 * nt + 4 * lb);
            sacc[nt][pt] = v;
        }
    const uint32_t HP = (uint32_t)a.H * kP;
    // Places of this lane in the tiles (bytes): 8 channels of x and 4 columns of b of the row it passes to the transposing reads of a 16-token
    // block, in even and in odd tiles of the state; the first and second 8-byte piece of a k-step of its own row of c.
    using TB = typename L::TB;
    using TX = typename L::TX;
    const int trow = state_tok(lb, lr >> 2), q4 = lr & 3;
    const int x_at = TX::row_at(trow) + 2 * (kP * hh + 32 * cw + 8 * q4);
    const int b_at = TB::row_at(trow) + 16 * ((q4 >> 1) ^ (trow & 3)) + 8 * (q4 & 1);  // odd tiles: ^ 32
    const int c_at = TB::row_at(lr) + 16 * ((lb >> 1) ^ (lr & 3)) + 8 * (lb & 1);      // second piece: ^ 32
    // this lane's 8 channels of its token in the first rows of a step's outputs (elements)
    const uint32_t y_at = lr * HP + (uint32_t)(h * kP + 32 * cw + 8 * lb);
    bf16_t *yp = a.y + (size_t)tok0 * HP;                                             // uniform
    float *yf = seg > 0 ? a.ybuf + (size_t)(seg - 1) * kSeamTok * HP : nullptr;        // uniform
    const int nseam = seg > 0 ? kSeamTok / kQ : 0;

    strd_s16x4 cr[2][2 * KS];  // c pieces of a step's two query blocks, requested a step ahead (as are the tiles, for the G waves)
    using First = std::integral_constant<int, 0>;
    using Second = std::integral_constant<int, 1>;
    auto request_c = [&](int i, auto tt) __attribute__((always_inline)) {
        const uint32_t ct = lds_offset(lds.c[i % kRB].v) + c_at;
        issue_c_pieces<KS, tt.value * TB::kBlock>(ct, ct ^ 32, cr[tt.value]);
    };
    lds_barrier();  // row tables |
    lds_barrier();  // first copies landed, scans of steps 0 and 1 |
    request_c(0, First());
    request_c(0, Second());
    lds_barrier();  // weights of step 0

    for (int i = 0; i < nloc; ++i) {
        settle_c_pieces<KS>(cr[0]);  // (the barrier before has waited for them)
        settle_c_pieces<KS>(cr[1]);
        const typename L::Scan &sc = lds.scan[i % 3][hh];
        const uint32_t bt = lds_offset(lds.b[i % kRB].v) + b_at;
        // Everything that (d), (c) and the weights of (e) need is requested at the start of the step.
        strd_s16x4 xr[4];
        lds_issue_tr4<0, TX::kBlock, 8, TX::kBlock + 8>(lds.x[i % kRX].v + x_at, xr);
        const float dq = sc.carry[kQ - 1];
        const f32x4 w0 = *reinterpret_cast<const f32x4 *>(&sc.w[8 * lb]), w1 = *reinterpret_cast<const f32x4 *>(&sc.w[8 * lb + 4]);
        const float cr0 = sc.carry[lr], cr1 = sc.carry[16 + lr];
        __builtin_amdgcn_sched_barrier(0);
        // (d): Y^T[p, t] = sum_n S[p, n] c_t[n].  A operand straight from the accumulators: the lane holds rows
        // 4 lb .. 4 lb + 3 of state tiles 2 ks and 2 ks + 1 for column p = lr, i.e. the k slots n = 32 ks + 4 lb + s (s < 4),
        // 32 ks + 16 + 4 lb + s - 4 (s >= 4); the c fragments are read in the same slot order (two 8-byte reads).
        // The vector work of a step is dealt out between its products, four or five instructions to each: the state's conversion and the
        // weights of x here, the state's decay in (e).
        f32x4 yacc[2][2];  // [query block][tile]
        bf16x8 xf[2], xwf[2];
        auto decay = [&](int nt, int pt) __attribute__((always_inline)) { sacc[nt][pt] *= dq; };
        auto half = [&](int ks, int pt, int hi) __attribute__((always_inline)) { return to_bf16x4(sacc[2 * ks + hi][pt]); };
        bf16x4 sb[2][2][2];  // [ks % 2][tile][half]: the state's fragments of this k-step and the next
#pragma unroll
        for (int pt = 0; pt < 2; ++pt)
#pragma unroll
            for (int hi = 0; hi < 2; ++hi) sb[0][pt][hi] = half(0, pt, hi);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int tt = j >> 1, pt = j & 1;
                yacc[tt][pt] = mfma16(cat8(sb[ks & 1][pt][0], sb[ks & 1][pt][1]), tr_pair(cr[tt][2 * ks], cr[tt][2 * ks + 1]), ks ? yacc[tt][pt] : f32x4{0.f, 0.f, 0.f, 0.f});
                if (ks + 1 < KS) sb[(ks + 1) & 1][pt][tt] = half(ks + 1, pt, tt);
                if (ks == 0) {
                    decay(tt, pt);
                } else {
                    // a twelfth (n = 64: a quarter) of the weights of x
                    constexpr int kSlots = 4 * (KS - 1);
                    const int from = 16 * (4 * (ks - 1) + j) / kSlots, to = 16 * (4 * (ks - 1) + j + 1) / kSlots;
#pragma unroll
                    for (int e = from; e < to; ++e) xwf[e >> 3][e & 7] = (bf16_t)((float)xf[e >> 3][e & 7] * ((e & 7) < 4 ? w0[e & 3] : w1[e & 3]));
                }
                if (ks == 0 && j == 3) {
                    // x fragments: A operand of (c) as they are, B operand of (e) once weighted
                    __builtin_amdgcn_s_waitcnt(lgkm_wait_imm(0));  // (in the compiler's books, too: a wait of its own later on would count the b fragments)
                    lds_settle4(xr);
                    xf[0] = tr_pair(xr[0], xr[1]);
                    xf[1] = tr_pair(xr[2], xr[3]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        strd_s16x4 ba[8], bb[8], m0;
        i32x4 m1;
        asm volatile("ds_read_b64 %0, %2\n\tds_read_b128 %1, %3"
                     : "=&v"(m0), "=&v"(m1) : "v"(lds_offset(&lds.m0[i & 1][hh][lane])), "v"(lds_offset(&lds.m1[i & 1][hh][lane])) : "memory");
        issue_b_frags<0, TB::kBlock>(bt, bt ^ 32, ba);
        if constexpr (NT == 8) issue_b_frags<128, TB::kBlock>(bt, bt ^ 32, bb);
        // (c) on top of the carried part
#pragma unroll
        for (int pt = 0; pt < 2; ++pt) {
            yacc[0][pt] *= cr0;
            yacc[1][pt] *= cr1;
        }
        asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(m0), "+v"(m1) : "i"(NT == 8 ? 15 : 8) : "memory");  // the b fragments after them may be on their way
#pragma unroll
        for (int pt = 0; pt < 2; ++pt) {
            yacc[0][pt] = mfma16(xf[pt], cat8(__builtin_bit_cast(bf16x4, m0), bf16x4{}), yacc[0][pt]);
            yacc[1][pt] = mfma16(xf[pt], __builtin_bit_cast(bf16x8, m1), yacc[1][pt]);
        }
        __builtin_amdgcn_sched_barrier(0);
        // (e): S^T = 2^(l_Q) S^T + b^T (w x)
        if constexpr (NT == 8)
            lds_settle8_but<8>(ba);
        else {
            lds_settle8(ba);
            request_c(i + 1, Second());
        }
        // the c pieces of the next step (the last step reads a tile that was never requested, into registers that nobody uses)
        request_c(i + 1, First());
#pragma unroll
        for (int d = 0; d < 4; ++d) {
#pragma unroll
            for (int pt = 0; pt < 2; ++pt) sacc[d][pt] = mfma16(tr_pair(ba[2 * d], ba[2 * d + 1]), xwf[pt], sacc[d][pt]);
            if (d + 2 < NT) decay(d + 2, 0), decay(d + 2, 1);
        }
        eight_products_with_vector_work();
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (NT == 8) {
            lds_settle8_but<2 * KS>(bb);
            request_c(i + 1, Second());
#pragma unroll
            for (int d = 4; d < 8; ++d) {
#pragma unroll
                for (int pt = 0; pt < 2; ++pt)
                    sacc[d % NT][pt] = mfma16(tr_pair(bb[2 * (d - 4)], bb[2 * (d - 4) + 1]), xwf[pt], sacc[d % NT][pt]);
                if (d + 2 < NT) decay(d + 2, 0), decay(d + 2, 1);
            }
            eight_products_with_vector_work();
            __builtin_amdgcn_sched_barrier(0);
        }
        // outputs: 16 bytes of this lane's token
        const int left = a.T - (tok0 + i * kQ);  // uniform: tokens from the step's first to the sequence's end
        if (i < nseam) {
#pragma unroll
            for (int tt = 0; tt < 2; ++tt)
                if (left >= kQ || lr + 16 * tt < left) {
                    float *dst = yf + (size_t)16 * tt * HP;
                    *reinterpret_cast<f32x4 *>(dst + y_at) = yacc[tt][0];
                    *reinterpret_cast<f32x4 *>(dst + y_at + 4) = yacc[tt][1];
                }
            yf += (size_t)kQ * HP;
        } else {
            bf16x8 out[2];
#pragma unroll
            for (int tt = 0; tt < 2; ++tt) out[tt] = cat8(to_bf16x4(yacc[tt][0]), to_bf16x4(yacc[tt][1]));
            if (left >= kQ) {
#pragma unroll
                for (int tt = 0; tt < 2; ++tt) *reinterpret_cast<bf16x8 *>(yp + (size_t)16 * tt * HP + y_at) = out[tt];
            } else {
#pragma unroll
                for (int tt = 0; tt < 2; ++tt)
                    if (lr + 16 * tt < left) *reinterpret_cast<bf16x8 *>(yp + (size_t)16 * tt * HP + y_at) = out[tt];
            }
        }
        yp += (size_t)kQ * HP;
        lds_barrier();  // the step is over
    }

    if (s_dst) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int pt = 0; pt < 2; ++pt)
                *reinterpret_cast<f32x4 *>(s_dst + ((size_t)h * kP + chan_of(cw, pt, lr)) * NS + 16 * nt + 4 * lb) = sacc[nt][pt];
    }
    if (seg < a.nseg - 1) {
        bool lost = false;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int pt = 0; pt < 2; ++pt)
#pragma unroll
                for (int e = 0; e < 4; ++e) lost |= !(__builtin_fabsf(sacc[nt][pt][e]) < __builtin_inff());
        const unsigned long long any = __ballot(lost);
        if (lane == 0) a.lost[((size_t)seg * a.H + h) * 2 + cw] = any != 0;
    }
}

// ---- G wave gw: the weights M of heads 2 gw and 2 gw + 1 of the workgroup, one step ahead ----
template <int NS>
__device__ __forceinline__ void g_wave(LdsQ<NS> &lds, const QuadArgs &a, int gw, int h0, int nloc) {
    using L = LdsQ<NS>;
    constexpr int KS = NS / 32;
    const int lane = threadIdx.x & 63, lr = lane & 15, lb = lane >> 4;
    f32x4 dskip[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const float Dh = a.D ? a.D[h0 + 2 * gw + q] : 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) dskip[q][e] = 4 * lb + e == lr ? Dh : 0.f;
    }
    using TB = typename L::TB;
    const int at = TB::row_at(lr) + 16 * (lb ^ (lr & 3));  // this lane's 16 bytes of the first k-step of its row
    auto weights = [&](int i) __attribute__((always_inline)) {
        const char *bt = lds.b[i % kRB].v + at, *ct = lds.c[i % kRB].v + at;
        // (a): key block 0 x query blocks 0 and 1, key block 1 x query block 1
        f32x4 g00 = {0.f, 0.f, 0.f, 0.f}, g01 = g00, g11 = g00;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const bf16x8 b0 = *reinterpret_cast<const bf16x8 *>(bt + 64 * ks), b1 = *reinterpret_cast<const bf16x8 *>(bt + TB::kBlock + 64 * ks);
            const bf16x8 c0 = *reinterpret_cast<const bf16x8 *>(ct + 64 * ks), c1 = *reinterpret_cast<const bf16x8 *>(ct + TB::kBlock + 64 * ks);
            g00 = mfma16(b0, c0, g00);
            g01 = mfma16(b0, c1, g01);
            g11 = mfma16(b1, c1, g11);
        }
        // (b): the diagonal blocks directly, masked; the block below the diagonal as 2^(l_t - l_15) * fw[j], both exponents <= 0.
        // A lane's four keys 4 lb + e of a block belong to two lanes of the operand layout: even ones to lane group lb / 2, odd
        // ones to lb / 2 + 2, in slots 2 (lb % 2) and + 1.
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const typename L::Scan &sc = lds.scan[i % 3][2 * gw + q];
            const float el0 = sc.ell[lr], el1 = sc.ell[16 + lr], ref = sc.ell[15];
            const f32x4 elj0 = *reinterpret_cast<const f32x4 *>(&sc.ell[4 * lb]), elj1 = *reinterpret_cast<const f32x4 *>(&sc.ell[16 + 4 * lb]);
            const f32x4 dtj0 = *reinterpret_cast<const f32x4 *>(&sc.dtv[4 * lb]), dtj1 = *reinterpret_cast<const f32x4 *>(&sc.dtv[16 + 4 * lb]);
            const f32x4 fj = *reinterpret_cast<const f32x4 *>(&sc.fw[4 * lb]);
            const float er = fast_exp2(el1 - ref);
            bf16x4 m00, m01, m11;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool causal = 4 * lb + e <= lr;
                const float v0 = g00[e] * fast_exp2(el0 - elj0[e]) * dtj0[e] + dskip[q][e];
                const float v1 = g11[e] * fast_exp2(el1 - elj1[e]) * dtj1[e] + dskip[q][e];
                m00[e] = (bf16_t)(causal ? v0 : 0.f);
                m11[e] = (bf16_t)(causal ? v1 : 0.f);
                m01[e] = (bf16_t)(g01[e] * er * fj[e]);
            }
            bf16_t *m0 = reinterpret_cast<bf16_t *>(&lds.m0[i & 1][2 * gw + q][16 * (lb >> 1) + lr]) + 2 * (lb & 1);
            bf16_t *m1 = reinterpret_cast<bf16_t *>(&lds.m1[i & 1][2 * gw + q][16 * (lb >> 1) + lr]) + 2 * (lb & 1);
            *reinterpret_cast<bf16x2 *>(m0) = bf16x2{m00[0], m00[2]};
            *reinterpret_cast<bf16x2 *>(m0 + 32 * 4) = bf16x2{m00[1], m00[3]};
            *reinterpret_cast<bf16x2 *>(m1) = bf16x2{m01[0], m01[2]};
            *reinterpret_cast<bf16x2 *>(m1 + 32 * 8) = bf16x2{m01[1], m01[3]};
            *reinterpret_cast<bf16x2 *>(m1 + 4) = bf16x2{m11[0], m11[2]};
            *reinterpret_cast<bf16x2 *>(m1 + 32 * 8 + 4) = bf16x2{m11[1], m11[3]};
        }
    };
    lds_barrier();
    lds_barrier();
    weights(0);
    lds_barrier();
    for (int i = 0; i < nloc; ++i) {
        if (i + 1 < nloc) weights(i + 1);
        lds_barrier();
    }
}

// Source row of token t of the sequence (gather form); an index outside [0, N) is clamped into
// the tensors instead of faulting.
__device__ __forceinline__ uint32_t gather_row(const QuadArgs &a, int t, int32_t kept) {
    const uint32_t last_row = (uint32_t)(a.N + (a.T - a.K) - 1);
    return min((uint32_t)(t < a.K ? kept : a.N + (t - a.K)), last_row);
}

// ---- helper wave: dt copies, the scans of the workgroup's heads (two at a time, lane = 32 * (head % 2) + token), the row
// tables of the gather form ----
template <int NS, bool GATHER>
__device__ __forceinline__ void helper_wave(LdsQ<NS> &lds, const QuadArgs &a, int h0, int tok0, int nloc, int seg) {
    using L = LdsQ<NS>;
    const int lane = threadIdx.x & 63, half = lane >> 5, j = lane & 31;
    float Al2[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) Al2[k] = a.A[h0 + 2 * k + half] * kLog2e;
    __builtin_amdgcn_s_setprio(3);
    auto token_of = [&](int i) { return min(tok0 + i * kQ + j, a.T - 1); };
    auto kept_of = [&](int i) -> int32_t { return a.idx[min(token_of(i), a.K - 1)]; };  // K >= 1 in gather mode
    auto request_kept = [&](int i) __attribute__((always_inline)) {
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(a.idx + min(token_of(i), a.K - 1)),
                                         (__attribute__((address_space(3))) void *)lds.rawidx[i & 3], 4, 0, 0);
    };
    auto request_dt = [&](int i) __attribute__((always_inline)) {  // 64 lanes x 4 bytes per pair; rows past T re-read the last row
        const uint32_t row = GATHER ? lds.rowtab[i & 3][j] : (uint32_t)token_of(i);
#pragma unroll
        for (int k = 0; k < 2; ++k)
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void *)(reinterpret_cast<const char *>(a.dt) + (size_t)row * ((uint32_t)a.H * 4) + (uint32_t)(h0 + 2 * k + half) * 4),
                (__attribute__((address_space(3))) void *)lds.dt[i % kRD][k], 4, 0, 0);
    };
    float ltot[2] = {0.f, 0.f};
    int life[2] = {0, 0};
    auto make_scan = [&](int k, int i, float raw) __attribute__((always_inline)) {
        const float dv = (tok0 + i * kQ + j < a.T) ? raw : 0.f;
        float inc = dv * Al2[k];  // inclusive prefix sum over the 32 lanes of a head
#define STRD_DPP_FADD(ctrl, row_mask) \
    inc += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, inc), ctrl, row_mask, 0xF, true))
        STRD_DPP_FADD(0x111, 0xF);  // row_shr:1
        STRD_DPP_FADD(0x112, 0xF);  // row_shr:2
        STRD_DPP_FADD(0x114, 0xF);  // row_shr:4
        STRD_DPP_FADD(0x118, 0xF);  // row_shr:8
        STRD_DPP_FADD(0x142, 0xA);  // row_bcast:15 into rows 1 and 3
#undef STRD_DPP_FADD
        typename L::Scan &m = lds.scan[i % 3][2 * k + half];
        const float tot = half ? read_lane_f32(inc, 63) : read_lane_f32(inc, 31);
        const float l15 = half ? read_lane_f32(inc, 47) : read_lane_f32(inc, 15);
        m.ell[j] = inc;
        m.dtv[j] = dv;
        m.w[slot_of(j)] = dv * fast_exp2(tot - inc);
        m.carry[j] = fast_exp2(inc);
        if (j < 16) m.fw[j] = dv * fast_exp2(l15 - inc);  // the exponent is <= 0 for these
        // for the seam, while anything of what lies before the segment is left: without a gap, since every entry before life * 32 is read
        // (a dt that is not finite makes exp2(ltot) other than zero again, long after it was)
        if (seg > 0 && life[k] == i && fast_exp2(ltot[k]) != 0.f) {
            a.seam[((size_t)(seg - 1) * a.H + h0 + 2 * k + half) * (a.seg_steps * kQ) + i * kQ + j] = ltot[k] + inc;
            life[k] = i + 1;
        }
        ltot[k] += tot;
    };
    constexpr int kNewest = 2 + (GATHER ? 1 : 0);  // copies requested per step

    if (GATHER) {
#pragma unroll
        for (int i = 0; i < 4; ++i) lds.rowtab[i][j] = gather_row(a, token_of(i), kept_of(i));
        lds.rawidx[5 & 3][lane] = kept_of(5);  // read in steps 0 and 1, before the first copied entries
        lds.rawidx[6 & 3][lane] = kept_of(6);
    }
    const int32_t kept4 = GATHER ? kept_of(4) : 0;
    lds_barrier();  // row tables of steps 0..3 written
#pragma unroll
    for (int i = 0; i < kRD; ++i)
        if (i < nloc) request_dt(i);
    async_tile_wait();
#pragma unroll
    for (int i = 0; i < 2; ++i)
        if (i < nloc) {
#pragma unroll
            for (int k = 0; k < 2; ++k) make_scan(k, i, lds.dt[i][k][lane]);
        }
    lds_barrier();  // first copies landed, scans of steps 0 and 1
    if (GATHER) lds.rowtab[0][j] = gather_row(a, token_of(4), kept4);  // the prologue's requests have read table 0
    lds_barrier();

    for (int i = 0; i < nloc; ++i) {
        // dt of step i + 2 landed before the barrier that ended the previous step (or in the prologue)
        float raw[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) raw[k] = lds.dt[(i + 2) % kRD][k][lane];
        int32_t kept = 0;
        if (GATHER) kept = lds.rawidx[(i + 5) & 3][lane];
        __builtin_amdgcn_sched_barrier(0);
        const bool more = i + 4 < nloc;  // uniform; nothing past the segment is requested
        if (more) {
            request_dt(i + 4);                // slot last read in step i - 2
            if (GATHER) request_kept(i + 7);  // slot last read in step i - 2
        }
        if (i + 2 < nloc) {                   // slot last read in step i - 1
#pragma unroll
            for (int k = 0; k < 2; ++k) make_scan(k, i + 2, raw[k]);
        }
        if (GATHER) lds.rowtab[(i + 5) & 3][j] = gather_row(a, token_of(i + 5), kept);  // slot last used in step i - 1
        if (more)
            __builtin_amdgcn_s_waitcnt(vm_wait_imm(kNewest));  // everything requested in earlier steps has landed
        else
            async_tile_wait();
        lds_barrier();
    }
    if (j == 0) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            a.ltot[(size_t)seg * a.H + h0 + 2 * k + half] = ltot[k];
            if (seg > 0) a.life[(size_t)(seg - 1) * a.H + h0 + 2 * k + half] = life[k];
        }
    }
}

// One copy instruction: 16 bytes per lane from `src` to `dst` + 16 * lane.
__device__ __forceinline__ void copy16(const char *src, void *dst) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                     (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
}

// ---- copy wave: the B, C and x tiles three steps ahead of the compute waves (B and C two ahead of the G waves) ----
template <int NS, bool GATHER>
__device__ __forceinline__ void copy_wave(LdsQ<NS> &lds, const QuadArgs &a, int g, int h0, int tok0, int nloc) {
    using L = LdsQ<NS>;
    using TB = typename L::TB;
    using TX = typename L::TX;
    const int lane = threadIdx.x & 63;
    __builtin_amdgcn_s_setprio(3);
    const uint32_t x_row = (uint32_t)a.H * kP * 2, bc_row = (uint32_t)a.G * NS * 2;
    const char *xs = reinterpret_cast<const char *>(a.x) + (size_t)h0 * kP * 2;
    const char *bs = reinterpret_cast<const char *>(a.B) + (size_t)g * NS * 2, *cs = reinterpret_cast<const char *>(a.C) + (size_t)g * NS * 2;
    // The row this lane copies from with its first instruction of a tile, and where in the row; the k-th one is k * kRows rows on.
    const int xr0 = lane / (64 / TX::kRows), br0 = lane / (64 / TB::kRows);
    const uint32_t xc = lane % (64 / TX::kRows) * 16, bc = ((lane % (64 / TB::kRows)) ^ (br0 & 3)) * 16;
    uint32_t xo[TX::kIssues], bo[TB::kIssues];  // dense form: byte offsets inside the rows of a step, which are a uniform pointer
#pragma unroll
    for (int k = 0; k < TX::kIssues; ++k) xo[k] = (xr0 + k * TX::kRows) * x_row + xc;
#pragma unroll
    for (int k = 0; k < TB::kIssues; ++k) bo[k] = (br0 + k * TB::kRows) * bc_row + bc;
    auto stream = [&](auto *tile, const char *src, uint32_t row_bytes, const uint32_t *off, int r0, uint32_t col, int i) __attribute__((always_inline)) {
        using TT = typename std::remove_pointer<decltype(tile)>::type;
        const int t0 = tok0 + i * kQ;
        if (!GATHER && t0 + kQ <= a.T) {  // uniform: every row of the step exists
            const char *base = src + (size_t)t0 * row_bytes;
#pragma unroll
            for (int k = 0; k < TT::kIssues; ++k) copy16(base + off[k], tile->v + 1088 * k);
        } else {  // rows from the table, or past T: the last row again
#pragma unroll
            for (int k = 0; k < TT::kIssues; ++k) {
                const uint32_t row = GATHER ? lds.rowtab[i & 3][r0 + k * TT::kRows] : (uint32_t)min(t0 + r0 + k * TT::kRows, a.T - 1);
                copy16(src + (size_t)row * row_bytes + col, tile->v + 1088 * k);
            }
        }
    };
    auto request_x = [&](int i) __attribute__((always_inline)) { stream(&lds.x[i % kRX], xs, x_row, xo, xr0, xc, i); };
    auto request_bc = [&](int i) __attribute__((always_inline)) {
        stream(&lds.b[i % kRB], bs, bc_row, bo, br0, bc, i);
        stream(&lds.c[i % kRB], cs, bc_row, bo, br0, bc, i);
    };
    constexpr int kX = TX::kIssues, kBC = 2 * TB::kIssues;
    constexpr int kAll = 3 * kX + 2 * kBC;
    static_assert(2 * kX + kBC < 64, "vmcnt has 6 bits");

    lds_barrier();  // row tables of steps 0..3 written
    request_bc(0);
    request_x(0);
    if (nloc > 1) request_bc(1);
    if (nloc > 1) request_x(1);
    if (nloc > 2) request_bc(2);
    if (nloc > 2) request_x(2);
    if (nloc > 2)
        __builtin_amdgcn_s_waitcnt(vm_wait_imm(kAll < 63 ? kAll : 63));  // b and c of step 0
    else
        async_tile_wait();
    lds_barrier();
    if (nloc > 2) __builtin_amdgcn_s_waitcnt(vm_wait_imm(2 * kX + kBC));  // x of step 0, b and c of step 1
    lds_barrier();

    for (int i = 0; i < nloc; ++i) {
        // At the end of step i there are x of step i + 1 and b and c of step i + 2: of what was requested later, x of steps i + 2 and
        // i + 3 and b and c of step i + 3 may still be on their way (b and c of step i + 2 were requested before x of step i + 2).
        if (i + 3 < nloc) {                   // slots last read in step i - 1
            request_bc(i + 3);
            request_x(i + 3);
            __builtin_amdgcn_s_waitcnt(vm_wait_imm(2 * kX + kBC));
        } else if (i + 2 < nloc) {
            __builtin_amdgcn_s_waitcnt(vm_wait_imm(kX));
        } else {
            async_tile_wait();
        }
        lds_barrier();  // publishes it; the copies stay in flight
    }
}

template <int NS, bool GATHER>
__global__ __launch_bounds__(kThreads) void ssd_quad_kernel(QuadArgs a, int nunits) {
    using L = LdsQ<NS>;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    L &lds = *reinterpret_cast<L *>(smem_raw);

    const int unit = xcd_swizzle(blockIdx.x, nunits);
    if (unit >= nunits) return;
    const int seg = unit / a.wg_per_seg, h0 = unit % a.wg_per_seg * kHeads, g = h0 / (a.H / a.G);
    const int nsteps = (a.T + kQ - 1) / kQ;
    const int s0 = seg * a.seg_steps;
    const int nloc = min(a.seg_steps, nsteps - s0);
    const int tok0 = s0 * kQ;
    // where the segment's state comes from and goes to
    const float *s_src = seg == 0 ? a.S_in : nullptr;
    float *s_dst = seg == a.nseg - 1 ? a.S_out : a.lend + (size_t)seg * a.H * kP * NS;
    // Wave i runs on SIMD i % 4: every SIMD has two compute waves and one of the others.
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (wave < 8)
        compute_wave<NS>(lds, a, wave >> 1, wave & 1, h0 + (wave >> 1), seg, tok0, nloc, s_src, s_dst);
    else if (wave < 10)
        g_wave<NS>(lds, a, wave - 8, h0, nloc);
    else if (wave == 10)
        copy_wave<NS, GATHER>(lds, a, g, h0, tok0, nloc);
    else
        helper_wave<NS, GATHER>(lds, a, h0, tok0, nloc, seg);
}

// ---- the contribution of the incoming state to the tokens of segments 1.. and S_out -----
// One workgroup per (four heads of a group, boundary b = 1..nseg); b < nseg: y of segment b; b == nseg: S_out.  A wave per head and slab of 32
// channels, with the scan's order of channels, so that a lane reads and writes 16 bytes of a token's outputs.  Where the heads forget within a
// tile the kernel is a launch and a chain of loads: the last segment's state, the outputs that wait in fp32 and the decays, which the
// segment's own scan has left, are requested first, then four times in turn what says whether a head's states hold a value that is not
// finite, then the states before (one value at a time, each waited for); the c rows, which the waves share, go through LDS (each wave with its own copy
// of them took 10 us longer for 7 boundaries of 128 heads, 23.5 us at 2176 tokens, this 14).  Where they remember for longer it is bound by the way of the
// outputs from memory and back: c rows, outputs and decays are requested two tiles ahead, the outputs 16 bytes at a time (8448 tokens of 128 heads with decays
// of 0.003 per token, the whole call: 263 us with ssd_seg, 162 here, 15 % more one tile ahead with 8-byte accesses).  In the compiled code a tile
// waits for all of that, its successor's loads and the stores before it included, not for its own alone: the compiler, not the count below, waits for y
// and the decays, and the gather form's index entries on their way to an address drain the same queue.
// The boundaries of a head lie on one XCD: their states E are sums over the same final states.
constexpr int kFixThreads = 512;
constexpr int kFixTile = 64;  // tokens per tile: a lane per token
static_assert(kSeamTok == kFixTile, "the outputs of the first tile wait in fp32");
constexpr float kTiny = 1.17549435e-38f;  // smallest normal number

template <int NS, bool GATHER>
__global__ __launch_bounds__(kFixThreads) void ssd_quad_fix_kernel(QuadArgs a, int nunits) {
    using TB = typename LdsQ<NS>::TB;
    constexpr int KS = NS / 32;
    __shared__ TB ct[3][kFixTile / kQ];  // c rows of this tile and the next two
    const int unit = xcd_swizzle(blockIdx.x, nunits);
    if (unit >= nunits) return;
    const int b = 1 + unit % a.nseg, h0 = unit / a.nseg * kHeads;
    const int lane = threadIdx.x & 63, lr = lane & 15, lb = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), cw = wave & 1;  // slab of this wave
    const int h = h0 + (wave >> 1);
    const size_t seg_elems = (size_t)a.H * kP * NS;
    // A value that is not finite in an earlier segment's state reaches everything behind it, whatever the decays: then no weight below
    // is less than the smallest normal number and no tile is skipped.
    auto any_lost = [&](int head, int n) {  // in the final states of segments 0 .. n - 1
        bool lost = false;
        for (int s0 = 0; s0 < n; s0 += 64) {
            const uint32_t *p = a.lost + ((size_t)min(s0 + lane, n - 1) * a.H + head) * 2;
            lost |= __ballot((p[0] | p[1]) != 0) != 0;
        }
        return lost;
    };
    auto weight = [](bool lost, float f) { return lost && f < kTiny ? kTiny : f; };
    // weight of segment s' < b in the state at the start of segment b: prod_{s' < u < b} 2^(ltot[u])
    // (uniform; the loops below stop at the first segment whose weight is zero)
    if (b == a.nseg) {
        if (!a.S_out) return;
        const bool lost = any_lost(h, b - 1);
        float f = weight(lost, fast_exp2(a.ltot[(size_t)(b - 1) * a.H + h]));
        constexpr int per = kP * NS / 4, kStep = kFixThreads / kHeads;  // float4s of the head's state, threads of the head
        f32x4 *dst = reinterpret_cast<f32x4 *>(a.S_out + (size_t)h * kP * NS);
        for (int s = b - 2; s >= 0 && f != 0.f; --s) {
            const f32x4 *src = reinterpret_cast<const f32x4 *>(a.lend + (size_t)s * seg_elems + (size_t)h * kP * NS);
            for (int e = threadIdx.x % kStep; e < per; e += kStep) dst[e] += f * src[e];
            f = weight(lost, f * fast_exp2(a.ltot[(size_t)s * a.H + h]));
        }
        return;
    }
    const uint32_t HP = (uint32_t)a.H * kP;
    const int g = h / (a.H / a.G);
    const int seg_tok = a.seg_steps * kQ, tok0 = b * seg_tok, tend = min(a.T, tok0 + seg_tok);
    const int ntiles = (tend - tok0 + kFixTile - 1) / kFixTile;
    auto row_of = [&](int t) -> size_t {
        t = min(t, a.T - 1);
        return GATHER ? (size_t)gather_row(a, t, a.idx[min(t, a.K - 1)]) : (size_t)t;
    };
    // c rows of tile k, 1 KB per instruction, the pieces of a row permuted as in the scan's tiles
    constexpr int kWaves = kFixThreads / 64, kCopies = (kFixTile / TB::kRows + kWaves - 1) / kWaves;
    static_assert(kFixTile / TB::kRows % kWaves == 0, "every wave issues as many copies");
    auto copy_c = [&](int k, TB *dst) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < kCopies; ++q) {
            const int j = q * kWaves + wave, row0 = lane / (64 / TB::kRows);
            copy16(reinterpret_cast<const char *>(a.C + (row_of(tok0 + k * kFixTile + j * TB::kRows + row0) * a.G + g) * NS) + ((lane % (64 / TB::kRows)) ^ (row0 & 3)) * 16,
                   dst[j / TB::kIssues].v + 1088 * (j % TB::kIssues));
        }
    };
    // uniform pointers, to which a lane adds an offset of 32 bits
    auto state_of = [&](int s) { return a.lend + (size_t)s * seg_elems + ((size_t)h * kP + 32 * cw) * NS; };
    const int col = h * kP + 32 * cw;
    auto in_tile = [&](int k, int tt) { return (uint32_t)min(16 * tt + lr, a.T - 1 - (tok0 + k * kFixTile)); };  // tokens past T: the last
    auto y_of = [&](int k) { return a.y + (size_t)(tok0 + k * kFixTile) * HP + col; };
    const float *seam = a.seam + ((size_t)(b - 1) * a.H + h) * seg_tok;
    copy_c(0, ct[0]);
    // E = state at the start of segment b, as A-operand fragments: rows p = chan_of(0, pt, lr) of the slab, k slots n = 32 ks + 4 lb + s
    // (s < 4), 32 ks + 16 + 4 lb + s - 4 (s >= 4)
    f32x4 e[2][KS][2];
    auto each_e = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
        for (int pt = 0; pt < 2; ++pt)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int hi = 0; hi < 2; ++hi) f(e[pt][ks][hi], (uint32_t)(chan_of(0, pt, lr) * NS + 32 * ks + 16 * hi + 4 * lb));
    };
    each_e([&](f32x4 &v, uint32_t at) { v = *reinterpret_cast<const f32x4 *>(state_of(b - 1) + at); });
    // Outputs and decays of a tile and the next one.  A tile's are requested when the one two before it is done with its registers.
    bf16x8 y[2][4];
    f32x4 y0[4][2];  // the first tile's outputs
    float inc[2];    // lane = token: decay since the segment's start
    auto load = [&](int k, auto p) __attribute__((always_inline)) {
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) y[p.value][tt] = *reinterpret_cast<const bf16x8 *>(y_of(k) + (in_tile(k, tt) * HP + 8 * lb));
        inc[p.value] = seam[min(k * kFixTile + lane, seg_tok - 1)];
    };
    constexpr int kLoads = kCopies + 5;  // a wave's loads per tile
    std::integral_constant<int, 0> P0;
    std::integral_constant<int, 1> P1;
    const float *yw = a.ybuf + (size_t)(b - 1) * kSeamTok * HP + col;
#pragma unroll
    for (int tt = 0; tt < 4; ++tt)
#pragma unroll
        for (int pt = 0; pt < 2; ++pt) y0[tt][pt] = *reinterpret_cast<const f32x4 *>(yw + ((16 * tt + lr) * HP + 8 * lb + 4 * pt));
    inc[0] = seam[min(lane, seg_tok - 1)];
    const float lt = a.ltot[(size_t)(b - 1) * a.H + h];
    // tiles that anything of E reaches, for this head and for all four; the outputs of the first tile are written in any case
    int mine = 1, most = 1;
    bool lost = false;
#pragma unroll
    for (int q = 0; q < kHeads; ++q) {
        const bool l = any_lost(h0 + q, b);
        const int n = l ? ntiles : min(ntiles, (a.life[(size_t)(b - 1) * a.H + h0 + q] * kQ + kFixTile - 1) / kFixTile);
        most = max(most, n);
        if (h0 + q == h) mine = max(n, 1), lost = l;
    }
    const int life_tok = a.life[(size_t)(b - 1) * a.H + h] * kQ;  // tokens whose decays are there; behind them they are zero
    if (most > 1) {
        copy_c(1, ct[1]);
        load(1, P1);
    }
    float f = weight(lost, fast_exp2(lt));
    for (int s = b - 2; s >= 0 && f != 0.f; --s) {
        const float *src = state_of(s);
        each_e([&](f32x4 &v, uint32_t at) { v += f * *reinterpret_cast<const f32x4 *>(src + at); });
        f = weight(lost, f * fast_exp2(a.ltot[(size_t)s * a.H + h]));
    }
    bf16x8 ef[2][KS];
#pragma unroll
    for (int pt = 0; pt < 2; ++pt)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) ef[pt][ks] = cat8(to_bf16x4(e[pt][ks][0]), to_bf16x4(e[pt][ks][1]));
    const int c_at = TB::row_at(lr) + 16 * ((lb >> 1) ^ (lr & 3)) + 8 * (lb & 1);
    bf16x8 out[4];
    auto store = [&](int k) __attribute__((always_inline)) {
#pragma unroll
        for (int tt = 0; tt < 4; ++tt)
            if (tok0 + k * kFixTile + 16 * tt + lr < tend) *reinterpret_cast<bf16x8 *>(y_of(k) + (in_tile(k, tt) * HP + 8 * lb)) = out[tt];
    };
    int k = 0, buf = 0, last = -1;  // last: the tile whose outputs wait to be stored
    bool ahead = false;             // the loads of the tile after this one are the newest of the wave
    // One tile, outputs in slot p; false after the last.
    auto tile = [&](auto p) __attribute__((always_inline)) {
        if (ahead)
            __builtin_amdgcn_s_waitcnt(vm_wait_imm(kLoads));
        else
            async_tile_wait();
        lds_barrier();  // the c rows of this tile are there, and everyone is done with those of the tile before
        if (last >= 0) store(last);
        last = -1;
        if (k < mine) {
            const float cr = k * kFixTile + lane < life_tok ? weight(lost, fast_exp2(inc[p.value])) : lost ? kTiny : 0.f;
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) {
                const float crt = __shfl(cr, 16 * tt + lr, 64);
                const uint32_t c0 = lds_offset(ct[buf][tt >> 1].v) + c_at + (tt & 1) * TB::kBlock;
                strd_s16x4 cr8[2 * KS];
                issue_c_pieces<KS, 0>(c0, c0 ^ 32, cr8);
                settle_c_pieces<KS>(cr8);
                f32x4 acc[2] = {};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                    for (int pt = 0; pt < 2; ++pt) acc[pt] = mfma16(ef[pt][ks], tr_pair(cr8[2 * ks], cr8[2 * ks + 1]), acc[pt]);
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const float yv = k == 0 ? y0[tt][q >> 2][q & 3] : (float)y[p.value][tt][q];
                    out[tt][q] = (bf16_t)(crt != 0.f ? yv + crt * acc[q >> 2][q & 3] : yv);
                }
            }
            last = k;
        }
        ahead = k + 2 < most;
        if (ahead) {
            copy_c(k + 2, ct[buf == 0 ? 2 : buf - 1]);
            load(k + 2, p);
        }
        ++k;
        buf = buf == 2 ? 0 : buf + 1;
        return k < most;
    };
    while (tile(P0) && tile(P1)) {
    }
    if (last >= 0) store(last);
}

template <int NS, bool GATHER>
int launch(const QuadArgs &a, hipStream_t st) {
    const int nunits = a.nseg * a.wg_per_seg;
    const size_t smem = sizeof(LdsQ<NS>);
    if (!allow_dynamic_lds(reinterpret_cast<const void *>(&ssd_quad_kernel<NS, GATHER>), smem)) return STRD_EHIP;
    ssd_quad_kernel<NS, GATHER><<<xcd_grid(nunits), kThreads, smem, st>>>(a, nunits);
    // (as many units again: a boundary per segment, the last one for S_out)
    ssd_quad_fix_kernel<NS, GATHER><<<xcd_grid(nunits), kFixThreads, 0, st>>>(a, nunits);
    return launch_status();
}

struct Plan {
    int nseg, seg_steps;
    size_t lend, ltot, lost, seam, life, ybuf;  // bytes of the parts of the workspace
    size_t bytes() const { return lend + ltot + lost + seam + life + ybuf; }
};

// How the sequence is cut: as many segments as it takes to give every CU a workgroup, each at least kMinSegSteps steps long; two at least
// (ssd_quad_preferred).
Plan plan_of(int T, int H, int n) {
    constexpr int kMinSegSteps = 8, kCUs = 256;
    const int nsteps = (T + kQ - 1) / kQ, wg = H / kHeads;
    const int s = max(1, min(kCUs / wg, nsteps / kMinSegSteps));  // (one round of the chip)
    Plan p;
    p.seg_steps = (nsteps + s - 1) / s;
    p.nseg = (nsteps + p.seg_steps - 1) / p.seg_steps;
    p.lend = align_up((size_t)(p.nseg - 1) * H * kP * n * sizeof(float), 256);
    p.ltot = align_up((size_t)p.nseg * H * sizeof(float), 256);
    p.lost = align_up((size_t)(p.nseg - 1) * H * 2 * sizeof(uint32_t), 256);
    p.seam = align_up((size_t)(p.nseg - 1) * H * p.seg_steps * kQ * sizeof(float), 256);
    p.life = align_up((size_t)(p.nseg - 1) * H * sizeof(int32_t), 256);
    p.ybuf = (size_t)(p.nseg - 1) * kSeamTok * H * kP * sizeof(float);
    return p;
}

}  // namespace

size_t ssd_quad_ws(int T, int H, int n) { return plan_of(T, H, n).bytes(); }

// `rows` = number of rows of the source tensors (T for the dense call, N + M for the gather call)
bool ssd_quad_supported(int T, int rows, int H, int P, int G, int n, strd_dtype io) {
    return P == kP && H / G % kHeads == 0 && ssd_seg_supported(T, rows, H, P, G, n, io);
}

// Where this kernel is taken: in the place of ssd_seg's two-head form, where that one would be taken with segments of 32 steps of 64
// tokens and more, and the segments here, twice as many, still leave the few CUs that they need (64 heads).  us of a call, before -> here, n = 128,
// with decays of one per token and more (A = -1 to -7, dt = 0.8) / with
// 0.003 of those: 128 heads, 8448 tokens 119 -> 99 / 263 -> 162, 33280 tokens 356 -> 287 / 1087 -> 505; 64 heads, 16640 tokens 106 -> 97 / 268 ->
// 197; 256 heads, 8448 tokens 196 -> 157 / 545 -> 268; 96 heads, 12000 tokens 164 -> 107 / 391 -> 189; 508 heads, 4500 tokens 213 -> 161 / 556 -> 259; n = 64:
// 128 heads, 8448 tokens 87.5 -> 80.7 / 188 -> 126, 33280 tokens 282 -> 254 / 864 -> 471.  Error against 64 bits (2-norm), decays of one per token / 0.1 / 0.003 of
// that: 128 heads, 8448 tokens 2.3440 -> 2.3435e-3 / 2.410 -> 2.404 / 3.28 -> 3.11; no larger at any of 1 to 0.0003 for 64 to 508 heads, n = 64 and 128.
// Not taken: shorter sequences of fewer heads, where one workgroup per (head, 32 channels) is the slower one while heads forget (128 heads, 5630
// tokens 89 -> 67) and the faster one while they do not (90 -> 114: seven eighths of the outputs are read and written again); up to 32 heads
// neither gains (16 heads, 2176 tokens 31 -> 36).  512 heads and more, where ssd_seg is not taken either: here they are faster, 2176 tokens of
// 512 heads 172 -> 97, of 1024 345 -> 146, but further from 64 bits than the kernel that adds up 64 tokens of every output from unrounded x: steps of 32
// leave more of an output to the state and its weighted x, both rounded (2176 tokens of 512 heads in two segments 2.334 -> 2.335e-3, with slow
// decays 2.73 -> 2.98e-3; in one segment, of 1024 heads, 2.347 -> 2.348 and 2.73 -> 2.79e-3).
bool ssd_quad_preferred(int T, int H, int P, int G) { return H >= 64 && ssd_seg_preferred(T, H, P, G); }

int ssd_quad(const void *x, const float *dt, const float *A, const void *B, const void *C, const float *D, const float *S_in,
             void *y, float *S_out, const int32_t *idx, int N, int K, int T, int H, int G, int n, void *ws, hipStream_t st) {
    QuadArgs a;
    a.x = (const bf16_t *)x; a.dt = dt; a.A = A; a.B = (const bf16_t *)B; a.C = (const bf16_t *)C; a.D = D; a.S_in = S_in;
    a.y = (bf16_t *)y; a.S_out = S_out; a.idx = idx; a.N = N; a.K = K; a.T = T; a.H = H; a.G = G;
    const Plan p = plan_of(T, H, n);
    a.nseg = p.nseg;
    a.seg_steps = p.seg_steps;
    a.wg_per_seg = H / kHeads;
    if (!ws) return STRD_EWORKSPACE;
    char *w = (char *)ws;
    a.lend = (float *)w;
    a.ltot = (float *)(w + p.lend);
    a.lost = (uint32_t *)(w + p.lend + p.ltot);
    a.seam = (float *)(w + p.lend + p.ltot + p.lost);
    a.life = (int32_t *)(w + p.lend + p.ltot + p.lost + p.seam);
    a.ybuf = (float *)(w + p.lend + p.ltot + p.lost + p.seam + p.life);
    if (n == 128) return idx ? launch<128, true>(a, st) : launch<128, false>(a, st);
    return idx ? launch<64, true>(a, st) : launch<64, false>(a, st);
}

}  // namespace strd
