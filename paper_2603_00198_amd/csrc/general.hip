// General-shape kernels: fp32 arithmetic on fp32 or bf16 tensors, any head count, head dimension
// and state size.  They serve fp32 I/O (whose 1e-4 tolerance rules out bf16 matrix cores) and the
// shapes the bf16 kernels of the *_mfma.hip files are not tiled for.
//
// Every contraction (but those of a few tokens: the recurrence, and attention row by row) runs on v_mfma_f32_16x16x4_f32: fp32 products and sums, so nothing is lost
// against vector arithmetic, while a wave owns a 16 x 16 tile and reads each operand row once per
// tile instead of once per element.  An operand lane (row r = lane % 16, lane group lb = lane / 16)
// holds the four elements 16 j + 4 lb .. + 3 of its row as one 16-byte load and feeds them to four
// consecutive products; both operands take the contraction index in that order, so the sum is
// the same.  Accumulator element i of a lane is row 4 lb + i, column r of the tile -- exactly the
// operand layout of the next product over those rows, so that probabilities (attention) and decay
// weights (scan) go from one product into the next without leaving the registers.
// Operands come straight from global memory: the shapes these kernels see in practice (a few
// thousand tokens, a handful of heads) live in L2 and are bound by latency, i.e. by how many
// loads are in flight and how many workgroups share the work, not by bandwidth.
#include <algorithm>

#include "common.h"

namespace strd {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ float ex2(float v) { return __builtin_amdgcn_exp2f(v); }
__device__ __forceinline__ bool finite(float v) { return fabsf(v) < INFINITY; }
__device__ __forceinline__ f32x4 zero4() { return f32x4{0.f, 0.f, 0.f, 0.f}; }
__device__ __forceinline__ int wave_index() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); }
// Sum / max over the four lane groups that share a column of an accumulator tile.
__device__ __forceinline__ float groups_sum(float v) {
    v += __shfl_xor(v, 16, kWave);
    return v + __shfl_xor(v, 32, kWave);
}
__device__ __forceinline__ float groups_max(float v) {
    v = fmaxf(v, __shfl_xor(v, 16, kWave));
    return fmaxf(v, __shfl_xor(v, 32, kWave));
}

// Elements c .. c + W - 1 of a row of `len`, zeros from len on (FULL: the caller never asks past len).  W > 1
// needs len % W == 0 and an aligned row, so a vector lies wholly inside the row or wholly past it.  No
// branch around the load: behind one, the compiler waits for every outstanding load at the first use of any.
template <int W, bool FULL, typename T>
__device__ __forceinline__ void load_row(const T *__restrict__ row, int c, int len, float (&out)[W]) {
    const int at = FULL ? c : min(c, len - W);
    if constexpr (W == 1) {
        out[0] = to_f32(row[at]);
    } else if constexpr (std::is_same<T, float>::value) {
        typedef typename std::conditional<W == 4, f32x4, f32x2>::type V;
        const V v = *reinterpret_cast<const V *>(row + at);
#pragma unroll
        for (int i = 0; i < W; ++i) out[i] = v[i];
    } else {
        typedef typename std::conditional<W == 4, bf16x4, bf16x2>::type V;
        const V v = *reinterpret_cast<const V *>(row + at);
#pragma unroll
        for (int i = 0; i < W; ++i) out[i] = static_cast<float>(v[i]);
    }
    if constexpr (!FULL)
#pragma unroll
        for (int i = 0; i < W; ++i) out[i] = c < len ? out[i] : 0.f;
}
template <int W, typename T>
__device__ __forceinline__ void store_row(T *__restrict__ row, int c, int len, const float (&in)[W]) {
    if (c >= len) return;
    if constexpr (W == 1) {
        row[c] = from_f32<T>(in[0]);
    } else if constexpr (std::is_same<T, float>::value) {
        typedef typename std::conditional<W == 4, f32x4, f32x2>::type V;
        V v;
#pragma unroll
        for (int i = 0; i < W; ++i) v[i] = in[i];
        *reinterpret_cast<V *>(row + c) = v;
    } else {
        typedef typename std::conditional<W == 4, bf16x4, bf16x2>::type V;
        V v;
#pragma unroll
        for (int i = 0; i < W; ++i) v[i] = static_cast<bf16_t>(in[i]);
        *reinterpret_cast<V *>(row + c) = v;
    }
}

// One lane's share of an operand row: elements 16 j + 4 lb .. + 3 for j < KJ (rows up to 16 KJ
// elements stay in registers; FULL: exactly 16 KJ), or only the row's address for KJ = 0 (longer rows, or
// rows whose length or alignment does not allow vectors: element by element, read again for every product).
template <typename T, int KJ, bool FULL>
struct Operand {
    float v[KJ > 0 ? KJ : 1][4];
    const T *row;
    int len;
    __device__ __forceinline__ void load(const T *__restrict__ r, int lb, int n) {
        if constexpr (KJ > 0) {
#pragma unroll
            for (int j = 0; j < KJ; ++j) load_row<4, FULL>(r, 16 * j + 4 * lb, n, v[j]);
        } else {
            row = r;
            len = n;
        }
    }
};
// c += A . B^T for the 16 rows of each operand.
template <typename TA, typename TB, int KJ, bool FULL>
__device__ __forceinline__ f32x4 product(const Operand<TA, KJ, FULL> &a, const Operand<TB, KJ, FULL> &b, int lb, f32x4 c) {
    if constexpr (KJ > 0) {
#pragma unroll
        for (int j = 0; j < KJ; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) c = mfma4(a.v[j][i], b.v[j][i], c);
    } else {
        for (int e0 = 0; e0 < a.len; e0 += 16) {
            float av[4], bv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int e = e0 + 4 * i + lb;
                av[i] = e < a.len ? to_f32(a.row[e]) : 0.f;
                bv[i] = e < a.len ? to_f32(b.row[e]) : 0.f;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) c = mfma4(av[i], bv[i], c);
        }
    }
    return c;
}

// The same for NT row tiles against one B operand, the tiles taking turns: a product issues while the
// others' results are still on their way.
template <typename TA, typename TB, int KJ, bool FULL, int NT>
__device__ __forceinline__ void products(const Operand<TA, KJ, FULL> (&a)[NT], const Operand<TB, KJ, FULL> &b, int lb,
                                         f32x4 (&c)[NT]) {
    if constexpr (KJ > 0) {
#pragma unroll
        for (int j = 0; j < KJ; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int t = 0; t < NT; ++t) c[t] = mfma4(a[t].v[j][i], b.v[j][i], c[t]);
    } else {
#pragma unroll
        for (int t = 0; t < NT; ++t) c[t] = product(a[t], b, lb, c[t]);
    }
}

// The same product in double, from chains of at most 16 elements in single precision: in one chain the rounding grows
// with the row's length (128 elements: twice that of a sum in pieces of 16).
template <typename TA, typename TB, int KJ, bool FULL>
__device__ __forceinline__ void product_f64(const Operand<TA, KJ, FULL> &a, const Operand<TB, KJ, FULL> &b, int lb,
                                            double (&sum)[4]) {
    if constexpr (KJ > 0) {
        constexpr int kChains = KJ > 4 ? KJ : 4;  // (a chain of one element's four products waits for each of them)
        f32x4 c[kChains];
#pragma unroll
        for (int m = 0; m < kChains; ++m) c[m] = zero4();
#pragma unroll
        for (int j = 0; j < KJ; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) c[(4 * j + i) % kChains] = mfma4(a.v[j][i], b.v[j][i], c[(4 * j + i) % kChains]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            sum[e] = 0.0;
#pragma unroll
            for (int m = 0; m < kChains; ++m) sum[e] += (double)c[m][e];
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[e] = 0.0;
        // `M` chains at a time, all their elements requested before the first product
        auto step = [&](auto chains, int e0) __attribute__((always_inline)) {
            constexpr int M = decltype(chains)::value;
            float av[M][4], bv[M][4];
#pragma unroll
            for (int m = 0; m < M; ++m)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int at = min(e0 + 16 * m + 4 * u + lb, a.len - 1);
                    av[m][u] = to_f32(a.row[at]);
                    bv[m][u] = to_f32(b.row[at]);
                }
            f32x4 c[M];
#pragma unroll
            for (int m = 0; m < M; ++m) c[m] = zero4();
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    const bool in = e0 + 16 * m + 4 * u + lb < a.len;
                    c[m] = mfma4(in ? av[m][u] : 0.f, in ? bv[m][u] : 0.f, c[m]);
                }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int m = 0; m < M; ++m) sum[e] += (double)c[m][e];
        };
        int e0 = 0;
        for (; e0 + 48 < a.len; e0 += 64) step(std::integral_constant<int, 4>(), e0);
        for (; e0 < a.len; e0 += 16) step(std::integral_constant<int, 1>(), e0);
    }
}

// Query row r of kv head kvh (r = m * rep + j) is row m * Hq + kvh * rep + j of q.
__device__ __forceinline__ size_t qrow_index(int r, int rep, int Hq, int kvh) {
    return (size_t)(r / rep) * Hq + kvh * rep + r % rep;
}

// ------------------------------------------------------------------ score_attn -------------
// Two launches.  Pass 1: per query row the running max and sum of 2^z over a slice of the keys
// (z = scale log2(e) q.k); a wave holds 16 query rows in registers and walks the slice, tile
// transposed (keys on accumulator rows), so a lane's softmax state is one (max, sum) pair.
// Pass 2: a workgroup owns 16 keys and all query rows; it first combines the slices' statistics of
// its rows into log-sum-exps in LDS (every workgroup for itself: a few thousand cached loads
// instead of a launch), then its 8 waves deal the row tiles among themselves.
// 1024 keys, 128 query rows of 64: 11 + 928 us in the direct evaluation (one thread per key walked
// all rows) -> 6 + 5.6 us.
// SEQ = SeqTab (packed batch, blockIdx.y = sequence): q and k both point at the packed tensors, the
// statistics of sequence b start at b * seq_stride.
constexpr int kStatRows = 64;      // query rows per workgroup of pass 1 (4 waves)
constexpr int kColThreads = 512;   // pass 2 and score_mamba: 8 waves
constexpr int kColRows = 2048;     // rows whose log-sum-exp are in LDS at a time
constexpr int kMaxScoreRow = 14992;  // longest row taken

template <typename T, int KJ, bool FULL, class SEQ>
__global__ __launch_bounds__(256) void attn_stats_kernel(const T *__restrict__ q, const T *__restrict__ k,
                                                         float *__restrict__ pmax, float *__restrict__ psum, int M, int N,
                                                         int Hq, int Hkv, int d, float scale2, int nrb, int keys_per_slice,
                                                         SEQ seq, size_t seq_stride) {
    constexpr int KT = KJ == 1 || KJ == 4 ? 4 : 2;  // key tiles per trip: that many rows' loads in flight
    if constexpr (is_varlen<SEQ>()) {
        const int b = blockIdx.y;
        N = seq.N[b];
        M = seq.M[b];
        k += (size_t)seq.row0[b] * Hkv * d;
        q += (size_t)(seq.row0[b] + N) * Hq * d;
        pmax += b * seq_stride;
        psum += b * seq_stride;
    }
    const int lane = threadIdx.x & 63, lr = lane & 15, lb = lane >> 4, w = wave_index();
    const int rep = Hq / Hkv, R = M * rep;
    const int rb = blockIdx.x % nrb, kvh = (blockIdx.x / nrb) % Hkv, sl = blockIdx.x / nrb / Hkv;
    const int row = rb * kStatRows + w * 16 + lr;
    if (rb * kStatRows + w * 16 >= R) return;  // uniform per wave; there are no barriers
    const int key0 = sl * keys_per_slice, key1 = min(N, key0 + keys_per_slice);
    Operand<T, KJ, FULL> qf;
    qf.load(q + qrow_index(min(row, R - 1), rep, Hq, kvh) * d, lb, d);
    float run_m = -INFINITY, run_s = 0.f;
    for (int kb = key0; kb < key1; kb += 16 * KT) {
        Operand<T, KJ, FULL> kf[KT];
#pragma unroll
        for (int t = 0; t < KT; ++t) kf[t].load(k + ((size_t)min(kb + 16 * t + lr, N - 1) * Hkv + kvh) * d, lb, d);
        f32x4 z[KT];
#pragma unroll
        for (int t = 0; t < KT; ++t) z[t] = zero4();
        products(kf, qf, lb, z);
        float tmax = -INFINITY;
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (kb + 16 * t + 4 * lb + i >= key1) z[t][i] = -INFINITY;
                tmax = fmaxf(tmax, z[t][i]);
            }
        const float nm = fmaxf(run_m, tmax * scale2);
        const float ref = nm == -INFINITY ? 0.f : nm;
        float ts = 0.f;
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) ts += ex2(fmaf(z[t][i], scale2, -ref));
        run_s = run_s * ex2(run_m - ref) + ts;
        run_m = nm;
    }
    // the four lane groups saw disjoint keys of the same query
    const float m = groups_max(run_m), ref = m == -INFINITY ? 0.f : m;
    const float tot = groups_sum(run_s * ex2(run_m - ref));
    if (lb == 0 && row < R) {
        const size_t o = (size_t)sl * M * Hq + qrow_index(row, rep, Hq, kvh);
        pmax[o] = m;
        psum[o] = tot;
    }
}

template <typename T, int KJ, bool FULL, class SEQ>
__global__ __launch_bounds__(kColThreads) void attn_col_sum_kernel(const T *__restrict__ q, const T *__restrict__ k,
                                                                   const float *__restrict__ pmax,
                                                                   const float *__restrict__ psum, float *__restrict__ s,
                                                                   int M, int N, int Hq, int Hkv, int d, float scale2,
                                                                   int nslice, SEQ seq, size_t seq_stride, int ld) {
    __shared__ __attribute__((aligned(16))) float lse[kColRows];
    __shared__ float red[kColThreads / kWave][16];
    if constexpr (is_varlen<SEQ>()) {
        const int b = blockIdx.y;
        N = seq.N[b];
        M = seq.M[b];
        if ((int)blockIdx.x * 16 >= N) return;  // uniform
        k += (size_t)seq.row0[b] * Hkv * d;
        q += (size_t)(seq.row0[b] + N) * Hq * d;
        pmax += b * seq_stride;
        psum += b * seq_stride;
        s += (size_t)b * ld;
    }
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lb = lane >> 4, w = wave_index();
    const int rep = Hq / Hkv, R = M * rep, rows = M * Hq;
    // all query rows, kv head after kv head, every kv head padded to whole tiles of 16
    const int Rp = (R + 15) / 16 * 16;
    const long long F = (long long)Rp * Hkv;
    const int key = blockIdx.x * 16 + lr;
    Operand<T, KJ, FULL> kf, qf;
    int kf_head = -1;
    auto load_tile = [&](long long f) {  // f: first row of a tile (uniform)
        const int kvh = (int)(f / Rp), r = min((int)(f - (long long)kvh * Rp) + lr, R - 1);
        if (kvh != kf_head) kf.load(k + ((size_t)min(key, N - 1) * Hkv + kvh) * d, lb, d);
        kf_head = kvh;
        qf.load(q + qrow_index(r, rep, Hq, kvh) * d, lb, d);
    };
    float col = 0.f;
    for (long long f0 = 0; f0 < F; f0 += kColRows) {
        const int cnt = (int)min((long long)kColRows, F - f0);
        if (w * 16 < cnt) load_tile(f0 + w * 16);  // requested before the statistics are waited for
        if (f0 > 0) __syncthreads();               // everybody is done with the previous rows
        for (int e = tid; e < cnt; e += kColThreads) {
            const int kvh = (int)((f0 + e) / Rp), r = (int)(f0 + e - (long long)kvh * Rp);
            float v = INFINITY;  // padding rows: probability 0
            if (r < R) {
                const size_t o = qrow_index(r, rep, Hq, kvh);
                float m = -INFINITY, t = 0.f;
#pragma unroll 8
                for (int sl = 0; sl < nslice; ++sl) {
                    const float pm = pmax[(size_t)sl * rows + o], ps = psum[(size_t)sl * rows + o];
                    const float nm = fmaxf(m, pm), ref = nm == -INFINITY ? 0.f : nm;
                    t = t * ex2(m - ref) + ps * ex2(pm - ref);
                    m = nm;
                }
                v = m + __builtin_amdgcn_logf(t);
            }
            lse[e] = v;
        }
        __syncthreads();
        for (int ft = w * 16; ft < cnt; ft += kColThreads / kWave * 16) {
            const f32x4 z = product(qf, kf, lb, zero4());
            const f32x4 l = *reinterpret_cast<const f32x4 *>(&lse[ft + 4 * lb]);
            if (ft + kColThreads / kWave * 16 < cnt) load_tile(f0 + ft + kColThreads / kWave * 16);
#pragma unroll
            for (int i = 0; i < 4; ++i) col += ex2(fmaf(z[i], scale2, -l[i]));
        }
    }
    col = groups_sum(col);
    if (lb == 0) red[w][lr] = col;
    __syncthreads();
    if (tid < 16 && (int)blockIdx.x * 16 + tid < N) {
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < kColThreads / kWave; ++i) t += red[i][tid];  // fixed order
        s[blockIdx.x * 16 + tid] = t / ((float)M * (float)Hq);
    }
}

// ------------------------------------------------------------------ score_mamba ------------
// sum_g (sum_{h in g} dt_i^h) * sum_m |b_i^g . c_m^g|: a workgroup owns 16 tokens, its 8 waves deal the
// 16-row text tiles of all groups among themselves (1024 tokens, 32 text rows of 16: 58 us with one
// thread per token -> 3 us).
template <typename T, int KJ, bool FULL, class SEQ>
__global__ __launch_bounds__(kColThreads) void mamba_score_kernel(const T *__restrict__ Bv, const T *__restrict__ Ct,
                                                                  const float *__restrict__ dtv, float *__restrict__ s,
                                                                  int M, int N, int H, int G, int n, SEQ seq, int ld) {
    __shared__ float red[kColThreads / kWave][16];
    if constexpr (is_varlen<SEQ>()) {  // blockIdx.y = sequence; Bv, Ct, dtv are the packed tensors
        const int b = blockIdx.y;
        N = seq.N[b];
        M = seq.M[b];
        if ((int)blockIdx.x * 16 >= N) return;  // uniform
        Bv += (size_t)seq.row0[b] * G * n;
        Ct += (size_t)(seq.row0[b] + N) * G * n;
        dtv += (size_t)seq.row0[b] * H;
        s += (size_t)b * ld;
    }
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lb = lane >> 4, w = wave_index();
    const int hpg = H / G, tok = min((int)blockIdx.x * 16 + lr, N - 1);
    const int mt = (M + 15) / 16;  // text tiles per group
    float tot = 0.f, dts = 0.f;
    Operand<T, KJ, FULL> bf;
    int g_now = -1;
    for (long long u = w; u < (long long)mt * G; u += kColThreads / kWave) {
        const int g = (int)(u / mt), m0 = (int)(u - (long long)g * mt) * 16;
        if (g != g_now) {  // uniform
            bf.load(Bv + ((size_t)tok * G + g) * n, lb, n);
            dts = 0.f;
            for (int h = lb; h < hpg; h += 4) dts += dtv[(size_t)tok * H + g * hpg + h];
            dts = groups_sum(dts);
            g_now = g;
        }
        Operand<T, KJ, FULL> cf;
        cf.load(Ct + ((size_t)min(m0 + lr, M - 1) * G + g) * n, lb, n);
        const f32x4 z = product(cf, bf, lb, zero4());  // row = text row 4 lb + i, column = token
        float a = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) a += m0 + 4 * lb + i < M ? fabsf(z[i]) : 0.f;
        tot = fmaf(dts, a, tot);
    }
    tot = groups_sum(tot);
    if (lb == 0) red[w][lr] = tot;
    __syncthreads();
    if (tid < 16 && (int)blockIdx.x * 16 + tid < N) {
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < kColThreads / kWave; ++i) t += red[i][tid];
        s[blockIdx.x * 16 + tid] = t / ((float)M * (float)H);
    }
}

// ------------------------------------------------------------------ ssd ---------------------
// The scan in chunks of 64 tokens, all chunks side by side (the token-by-token recurrence is a serial
// chain of T steps: 830 us at 544 tokens, 8 heads of 32, n = 16; this form 13.9 in all).  Three launches:
//   state: per (head, chunk) what the chunk adds to the state, L = sum_s 2^(l_end - l_s) dt_s x_s b_s^T,
//          and its total decay,
//   pass:  per state element the recurrence over the chunks, leaving the state BEFORE every chunk in
//          place of L, and S_out,
//   out:   y_t = sum_{s<=t} 2^(l_t - l_s) dt_s (c_t.b_s) x_s + 2^(l_t) S_before c_t + D x_t.
// l is the running sum of dt A log2(e) inside the chunk, in double: it reaches several hundred, and a
// difference of two such numbers decides weights near 1 (in fp32 they would be off by 1e-5).
// The weights are products in double, rounded once, and the products c.b and S c sums of short chains: y is 5 to 40 %
// nearer to 64 bits than the recurrence's and S 2 to 50 %, at 16 to 1024 state entries and decays of 1 to 0.01 (with all
// of it in single precision y was 1.0 to 5 times as far off).  That costs 2 to 8 % (544 tokens 13.2 -> 13.9 us, 4096
// tokens of 128 heads 636 -> 676), and up to a quarter where many heads have a few chunks each.
constexpr int kChunk = 64;

// Inclusive sum over the lanes of a wave.
__device__ __forceinline__ double wave_scan_f64(double v) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const double u = __shfl_up(v, o, kWave);
        if (lane >= o) v += u;
    }
    return v;
}

// log2 of one token's decay.  2^-4096 is 0 like everything below it, and a sum of such terms has a difference where
// -inf (A = -inf: a head that forgets at once) has none.  A NaN stays one.
__device__ __forceinline__ double log2_decay(float dt, float A) {
    const double v = (double)dt * A * 1.4426950408889634;
    return v < -4096.0 ? -4096.0 : v;
}

// 2^v without the rounding of v to single precision (v is at least -64 x 4096).
__device__ __forceinline__ double ex2_f64(double v) {
    const double whole = rint(v);
    return (double)ldexpf(ex2((float)(v - whole)), (int)whole);
}

// What chunk c of head h adds to a block of 16 CPL channels x 16 NPL state columns, by one wave, into L[P][n], and (where
// `decay` is given) the chunk's total decay.  The weights go through LDS (`wt`, 64 entries) in two parts: their product with x is
// rounded once (in one, the states were 1 to 8 % further from 64 bits than the recurrence's).
template <typename T, int CPL, int NPL, bool FULL>
__device__ __forceinline__ void chunk_state(const T *__restrict__ x, const float *__restrict__ dt, const float *__restrict__ A,
                                            const T *__restrict__ B, float *L, float *decay, float2 *wt, int Tn, int H, int P, int G,
                                            int n, int h, int c, int p0, int n0) {
    const int lane = threadIdx.x & 63, lr = lane & 15, lb = lane >> 4, g = h / (H / G), t0 = c * kChunk;
    const float dtv = t0 + lane < Tn ? dt[(size_t)(t0 + lane) * H + h] : 0.f;
    float xv[4][4][CPL], bv[4][4][NPL];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const size_t t = min(t0 + 16 * kb + 4 * lb + i, Tn - 1);
            load_row<CPL, FULL>(x + (t * H + h) * P, p0 + CPL * lr, P, xv[kb][i]);
            load_row<NPL, FULL>(B + (t * G + g) * n, n0 + NPL * lr, n, bv[kb][i]);
        }
    const double l = wave_scan_f64(t0 + lane < Tn ? log2_decay(dtv, A[h]) : 0.0);
    const double end = __shfl(l, kWave - 1, kWave);
    const double weight = ex2_f64(end - l) * dtv;  // 0 past the last token
    const float most = (float)weight;
    wt[lane] = make_float2(most, fabsf(most) < INFINITY ? (float)(weight - most) : 0.f);
    if (decay && lane == 0) *decay = (float)ex2_f64(end);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // (LDS operations of a wave keep their order)
    if (t0 + kChunk > Tn) {  // uniform: the rows past the end are the last one again, which 0 does not take out if it is not finite
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (t0 + 16 * kb + 4 * lb + i >= Tn) {
#pragma unroll
                    for (int a = 0; a < CPL; ++a) xv[kb][i][a] = 0.f;
#pragma unroll
                    for (int b = 0; b < NPL; ++b) bv[kb][i][b] = 0.f;
                }
    }
    f32x4 acc[CPL][NPL];
#pragma unroll
    for (int a = 0; a < CPL; ++a)
#pragma unroll
        for (int b = 0; b < NPL; ++b) acc[a][b] = zero4();
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float2 wv = wt[16 * kb + 4 * lb + i];
#pragma unroll
            for (int a = 0; a < CPL; ++a) {
                const float rest = xv[kb][i][a] * wv.y;
                const float wx = fmaf(xv[kb][i][a], wv.x, finite(rest) ? rest : 0.f);
#pragma unroll
                for (int b = 0; b < NPL; ++b) acc[a][b] = mfma4(wx, bv[kb][i][b], acc[a][b]);
            }
        }
#pragma unroll
    for (int a = 0; a < CPL; ++a)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int p = p0 + CPL * (4 * lb + i) + a;
            float v[NPL];
#pragma unroll
            for (int b = 0; b < NPL; ++b) v[b] = acc[a][b][i];
            if (p < P) store_row<NPL>(L + p * n, n0 + NPL * lr, n, v);
        }
}

// One wave per (head, chunk, block of 16 CPL channels x 16 NPL state columns).
template <typename T, int CPL, int NPL, bool FULL>
__global__ __launch_bounds__(kWave) void ssd_chunk_state_kernel(const T *__restrict__ x, const float *__restrict__ dt,
                                                                const float *__restrict__ A, const T *__restrict__ B,
                                                                float *__restrict__ L, float *__restrict__ decay, int Tn,
                                                                int H, int P, int G, int n, int nc, int nst, int pblocks) {
    __shared__ float2 wt[kChunk];
    const int c = blockIdx.x % nst, h = (blockIdx.x / nst) % H, u = blockIdx.x / nst / H;
    chunk_state<T, CPL, NPL, FULL>(x, dt, A, B, L + ((size_t)h * nc + c) * P * n, u == 0 ? decay + (size_t)h * nc + c : nullptr, wt,
                                   Tn, H, P, G, n, h, c, u % pblocks * 16 * CPL, u / pblocks * 16 * NPL);
}

__global__ __launch_bounds__(kWave) void ssd_pass_kernel(float *__restrict__ L, const float *__restrict__ decay,
                                                         const float *__restrict__ S_in, float *__restrict__ S_out,
                                                         long long total, int pn, int nc, int nst) {
    const long long e = (long long)blockIdx.x * kWave + threadIdx.x;
    if (e >= total) return;
    const int h = (int)(e / pn);
    float *Lh = L + (size_t)h * nc * pn + (e - (long long)h * pn);
    const float *ah = decay + (size_t)h * nc;
    float run = S_in ? S_in[e] : 0.f;
    constexpr int kAhead = 8;
    for (int c0 = 0; c0 < nc; c0 += kAhead) {
        float v[kAhead], a[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int c = min(c0 + u, nst - 1);  // (nst = 0 only with nc = 1 and nothing to add: v is not used)
            v[u] = nst > 0 ? Lh[(size_t)c * pn] : 0.f;
            a[u] = nst > 0 ? ah[c] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (c0 + u < nc) {
                Lh[(size_t)(c0 + u) * pn] = run;
                run = fmaf(run, a[u], v[u]);
            }
    }
    if (S_out) S_out[e] = run;
}

// Outputs of the 64 tokens of chunk c of head h, by four waves: wave w owns tokens 16 w .. 16 w + 15 of the chunk as accumulator
// columns: weights W[s, t] = 2^(l_t - l_s) dt_s (c_t.b_s) for s <= t from the products b.c, then
// y^T[p, t] = sum_s x[s, p] W[s, t], a block of 16 CPL channels at a time.  `S`: the state before the chunk, [P][n] (`carried`:
// there is one), read with the first operands (EARLY) or after `publish`, which meets the other waves and makes the decays (ls: running
// sums, dts: dt) and the state theirs.
template <typename T, int CPL, int KN, bool FULL, bool EARLY, typename Publish>
__device__ __forceinline__ void chunk_out(const T *__restrict__ x, const T *__restrict__ B, const T *__restrict__ C,
                                          const float *__restrict__ D, const float *S, T *__restrict__ y, int Tn, int H, int P, int G,
                                          int n, int h, int c, int w, bool carried, const double *ls, const float *dts,
                                          Publish publish) {
    const int lane = threadIdx.x & 63, lr = lane & 15, lb = lane >> 4, g = h / (H / G), t0 = c * kChunk;
    const int tl = 16 * w + lr, t = t0 + tl;  // this lane's token (a column)
    Operand<T, KN, FULL> cf, bf[4];
    cf.load(C + ((size_t)min(t, Tn - 1) * G + g) * n, lb, n);
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (j <= w) bf[j].load(B + ((size_t)min(t0 + 16 * j + lr, Tn - 1) * G + g) * n, lb, n);
    // x and, where they are short enough for the registers, the state rows of a channel block: those of the
    // first block are on their way while the decays are scanned, those of the next while a block is summed
    float xv[4][4][CPL];
    Operand<float, KN, FULL> sf[CPL];
    constexpr bool kEarlyState = EARLY && CPL * KN <= 16;
    auto load_state = [&](int p0) {
        if (carried)
#pragma unroll
            for (int a = 0; a < CPL; ++a)
                sf[a].load(S + min(p0 + CPL * lr + a, P - 1) * n, lb, n);
    };
    auto load_block = [&](int p0) {
        if (kEarlyState) load_state(p0);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (j <= w)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    load_row<CPL, FULL>(x + ((size_t)min(t0 + 16 * j + 4 * lb + i, Tn - 1) * H + h) * P, p0 + CPL * lr, P, xv[j][i]);
    };
    load_block(0);
    publish();
    if (t0 + 16 * w >= Tn) return;  // uniform per wave, after the last barrier
    const double lt = ls[tl];
    const float et = ex2((float)lt);
    f32x4 W[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (j <= w) {
            double bc[4];
            product_f64(bf[j], cf, lb, bc);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int sl = 16 * j + 4 * lb + i;
                const double skip = D && sl == tl ? D[h] : 0.f;  // the skip term rides on the diagonal
                W[j][i] = sl <= tl ? (float)fma(bc[i], (double)ex2((float)(lt - ls[sl])) * dts[sl], skip) : 0.f;
            }
        }
    for (int p0 = 0; p0 < P; p0 += 16 * CPL) {
        f32x4 acc[CPL], from_state[CPL];
#pragma unroll
        for (int a = 0; a < CPL; ++a) acc[a] = from_state[a] = zero4();
        if (carried) {
            if (!kEarlyState) load_state(p0);
#pragma unroll
            for (int a = 0; a < CPL; ++a) {
                double sc[4];
                product_f64(sf[a], cf, lb, sc);
#pragma unroll
                for (int i = 0; i < 4; ++i) from_state[a][i] = (float)sc[i];
            }
        }
        // A weight of 0 takes a later token out of the sum only if its x is finite (0 x inf is NaN): on the diagonal
        // tile the values that are not are taken out of the operand and added token by token, where there are any.
        bool odd = false;  // uniform
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (j == w) {
                float z = 0.f;
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int a = 0; a < CPL; ++a) z = fmaf(xv[j][i][a], 0.f, z);
                odd = __any(z != 0.f);
                if (odd) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int a = 0; a < CPL; ++a) xv[j][i][a] = finite(xv[j][i][a]) ? xv[j][i][a] : 0.f;
                }
            }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (j <= w) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int a = 0; a < CPL; ++a) acc[a] = mfma4(xv[j][i][a], W[j][i], acc[a]);
            }
        if (odd) {
            f32x4 wd = W[0];
#pragma unroll
            for (int j = 1; j < 4; ++j)
                if (j == w) wd = W[j];
#pragma unroll 1
            for (int u = 0; u < 16; ++u) {
                const float mine = u & 2 ? (u & 1 ? wd[3] : wd[2]) : (u & 1 ? wd[1] : wd[0]);
                const float weight = __shfl(mine, 16 * (u >> 2) + lr, kWave);
                if (u > lr || t >= Tn) continue;
                const T *xr = x + ((size_t)(t0 + 16 * w + u) * H + h) * P;
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int a = 0; a < CPL; ++a) {
                        const int p = p0 + CPL * (4 * lb + i) + a;
                        const float val = p < P ? to_f32(xr[p]) : 0.f;
                        acc[a][i] = finite(val) ? acc[a][i] : fmaf(val, weight, acc[a][i]);
                    }
            }
        }
        if (carried) {
#pragma unroll
            for (int a = 0; a < CPL; ++a)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[a][i] = fmaf(from_state[a][i], et, acc[a][i]);
        }
        if (p0 + 16 * CPL < P) load_block(p0 + 16 * CPL);
        if (t < Tn)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float v[CPL];
#pragma unroll
                for (int a = 0; a < CPL; ++a) v[a] = acc[a][i];
                store_row<CPL>(y + ((size_t)t * H + h) * P, p0 + CPL * (4 * lb + i), P, v);
            }
    }
}

// l and dt of a chunk's tokens, by one wave.
__device__ __forceinline__ void chunk_decays(const float *__restrict__ dt, const float *__restrict__ A, int Tn, int H, int h, int t0,
                                             double *ls, float *dts) {
    const int lane = threadIdx.x & 63;
    const float dtv = t0 + lane < Tn ? dt[(size_t)(t0 + lane) * H + h] : 0.f;
    ls[lane] = wave_scan_f64(t0 + lane < Tn ? log2_decay(dtv, A[h]) : 0.0);
    dts[lane] = dtv;
}

// One workgroup per (head, chunk).
template <typename T, int CPL, int KN, bool FULL>
__global__ __launch_bounds__(256) void ssd_chunk_out_kernel(const T *__restrict__ x, const float *__restrict__ dt,
                                                            const float *__restrict__ A, const T *__restrict__ B,
                                                            const T *__restrict__ C, const float *__restrict__ D,
                                                            const float *__restrict__ S, T *__restrict__ y, int Tn, int H,
                                                            int P, int G, int n, int nc, int first_carried) {
    __shared__ double ls[kChunk];
    __shared__ float dts[kChunk];
    const int w = wave_index(), h = blockIdx.x % H, c = blockIdx.x / H;
    chunk_out<T, CPL, KN, FULL, true>(x, B, C, D, S + ((size_t)h * nc + c) * P * n, y, Tn, H, P, G, n, h, c, w, c >= first_carried, ls, dts, [&] {
        if (w == 0) chunk_decays(dt, A, Tn, H, h, c * kChunk, ls, dts);
        __syncthreads();
    });
}

// All three in one launch, for a few chunks of small states: a workgroup per (head, chunk) works out what every chunk before its own
// adds to the state (8 waves, a chunk each at a time), folds them up in the order of the pass, and has its four other waves' outputs.  The
// states of the chunks are made over and over, but none of it waits for another launch.
constexpr int kOnceChunks = 17;  // at most
constexpr int kOnceStateWaves = 8, kOnceThreads = (4 + kOnceStateWaves) * kWave;

template <typename T, int CPL, int KN, bool FULL>
__global__ __launch_bounds__(kOnceThreads) void ssd_once_kernel(const T *__restrict__ x, const float *__restrict__ dt,
                                                                const float *__restrict__ A, const T *__restrict__ B,
                                                                const T *__restrict__ C, const float *__restrict__ D,
                                                                const float *__restrict__ S_in, T *__restrict__ y,
                                                                float *__restrict__ S_out, int Tn, int H, int P, int G, int n, int nc) {
    extern __shared__ __attribute__((aligned(16))) float added[];  // [chunk][P][n]; chunk 0's place then holds the state before c
    __shared__ double ls[kChunk];
    __shared__ float dts[kChunk], decay[kOnceChunks];
    __shared__ float2 wt[kOnceStateWaves][kChunk];
    const int w = wave_index(), h = blockIdx.x % H, c = nc - 1 - (int)(blockIdx.x / H), pn = P * n;  // longest first
    const int want = c == nc - 1 && S_out ? c + 1 : c;  // chunks whose contribution is needed
    auto fold = [&] {
        __syncthreads();
        for (int e = threadIdx.x; e < pn; e += kOnceThreads) {
            float run = S_in ? S_in[(size_t)h * pn + e] : 0.f;
            for (int j = 0; j < c; ++j) run = fmaf(run, decay[j], added[j * pn + e]);
            if (want > c) S_out[(size_t)h * pn + e] = fmaf(run, decay[c], added[c * pn + e]);
            added[e] = run;
        }
        __syncthreads();
    };
    if (w >= 4) {
        const int v = w - 4, pblocks = (P + 16 * CPL - 1) / (16 * CPL), units = pblocks * ((n + 15) / 16);
        for (int u = v; u < want * units; u += kOnceStateWaves) {
            const int j = u / units, b = u % units;
            chunk_state<T, CPL, 1, FULL>(x, dt, A, B, added + j * pn, b == 0 ? &decay[j] : nullptr, wt[v], Tn, H, P, G, n, h, j,
                                         b % pblocks * 16 * CPL, b / pblocks * 16);
        }
        fold();
        return;
    }
    chunk_out<T, CPL, KN, FULL, false>(x, B, C, D, added, y, Tn, H, P, G, n, h, c, w, S_in || c > 0, ls, dts, [&] {
        if (w == 0) chunk_decays(dt, A, Tn, H, h, c * kChunk, ls, dts);
        fold();
    });
}

// The recurrence itself, for a few tokens, very large states and callers that bring no workspace: a state column (h, p) is held by
// `lanes` adjacent lanes, each with kSlice consecutive state entries in registers; y_t is reduced across those
// lanes.  A serial chain of T steps: 830 us at 544 tokens, 8 heads of 32, n = 16, where the chunks take 13.4.
constexpr int kSlice = 16, kRecThreads = 256;

template <typename T>
__global__ __launch_bounds__(kRecThreads) void ssd_recurrence_kernel(
    const T *__restrict__ x, const float *__restrict__ dt, const float *__restrict__ A, const T *__restrict__ B,
    const T *__restrict__ C, const float *__restrict__ D, const float *__restrict__ S_in, T *__restrict__ y,
    float *__restrict__ S_out, int Tn, int H, int P, int G, int n, int lanes) {
    const int gid = blockIdx.x * kRecThreads + threadIdx.x;
    const int col = gid / lanes, sub = gid % lanes;
    const bool live = col < H * P;
    const int h = live ? col / P : 0, p = live ? col % P : 0, g = h / (H / G);
    const int j0 = sub * kSlice;
    float S[kSlice];
#pragma unroll
    for (int e = 0; e < kSlice; ++e)
        S[e] = (live && S_in && j0 + e < n) ? S_in[((size_t)h * P + p) * n + j0 + e] : 0.f;
    const float Ah = A[h];
    const float Dh = D ? D[h] : 0.f;
    for (int t = 0; t < Tn; ++t) {
        const float dtt = dt[(size_t)t * H + h];
        const float a = expf(dtt * Ah);
        const float xv = to_f32(x[((size_t)t * H + h) * P + p]);
        const T *b = B + ((size_t)t * G + g) * n + j0;
        const T *c = C + ((size_t)t * G + g) * n + j0;
        float out = 0.f;
#pragma unroll
        for (int e = 0; e < kSlice; ++e)
            if (j0 + e < n) {
                S[e] = a * S[e] + xv * (dtt * to_f32(b[e]));
                out = fmaf(S[e], to_f32(c[e]), out);
            }
        for (int o = lanes / 2; o > 0; o >>= 1) out += __shfl_xor(out, o, kWave);
        if (live && sub == 0) y[((size_t)t * H + h) * P + p] = from_f32<T>(out + Dh * xv);
    }
    if (live && S_out)
#pragma unroll
        for (int e = 0; e < kSlice; ++e)
            if (j0 + e < n) S_out[((size_t)h * P + p) * n + j0 + e] = S[e];
}

// ------------------------------------------------------------------ attention --------------
// One workgroup per (16 query rows, query head), longest rows first; its NW waves take the key trips in
// turn, each with an online softmax of its own, and merge through LDS.  S^T = K Q^T keeps the queries
// on accumulator columns, so the probabilities of a tile are the operand of O^T += V^T P^T as they
// stand; V is read 4 channels a lane (channels 4 r .. of a block of 64 are rows r of four tiles).
// NW = 8 up to d = 64, 4 up to 128, 2 up to 256 (LDS).  544 tokens, 4 heads of 64: 54 us with one workgroup
// per row and no tiles -> 10.9 us; 2361 tokens: 46 us (51 when this was taken apart), of which the products alone take 32 and the loads
// alone 30 (16 KB per trip and wave from L2, the rate of a CU's path).  Four waves per SIMD overlap the
// two; a register set for the next trip in two waves per SIMD, two query tiles a wave (half the loads, but
// too few workgroups for the causal sweep to balance) and 4 or 16 waves were not faster.
template <typename T, bool VEC, bool FULL, int DJ, int NW, bool WIDE>
__global__ __launch_bounds__(NW *kWave) __attribute__((amdgpu_waves_per_eu(DJ == 1 ? 4 : 1))) void attn_tile_kernel(
    const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v, T *__restrict__ o, int Tn, int Hq, int Hkv,
    int d, float scale2) {
    constexpr int KJ = VEC ? 4 * DJ : 0, KT = DJ == 4 ? 1 : 2, kPitch = 64 * DJ + 4;
    __shared__ __attribute__((aligned(16))) float so[NW][16][kPitch];
    __shared__ float sm[NW][16], sl[NW][16];
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lb = lane >> 4, w = wave_index();
    const int nqt = (Tn + 15) / 16;
    const int q0 = (nqt - 1 - (int)(blockIdx.x / Hq)) * 16, h = blockIdx.x % Hq, hk = h / (Hq / Hkv);
    const int ntrip = (min(Tn, q0 + 16) + 16 * KT - 1) / (16 * KT);
    Operand<T, KJ, FULL> qf;
    qf.load(q + ((size_t)min(q0 + lr, Tn - 1) * Hq + h) * d, lb, d);
    f32x4 acc[DJ][4];
#pragma unroll
    for (int b = 0; b < DJ; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[b][e] = zero4();
    float run_m = -INFINITY, run_l = 0.f;
    // Rows of a trip: one address per workgroup and trip plus a 24-bit product per row (they lie within 32
    // rows of each other; WIDE, for rows of 16 MB and more: a full product); rows past the end of the sequence
    // re-read its last one.
    const size_t stride = (size_t)Hkv * d * sizeof(T);
    auto row_of = [&](const T *base, int r, int last) {
        const size_t off = WIDE ? (unsigned)min(r, last) * stride : __umul24((unsigned)min(r, last), (unsigned)stride);
        return reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + off);
    };
    auto body = [&](auto edge, int trip) __attribute__((always_inline)) {
        const int key0 = trip * KT * 16, last = Tn - 1 - key0;  // uniform
        const T *kb = k + ((size_t)key0 * Hkv + hk) * d, *vb = v + ((size_t)key0 * Hkv + hk) * d;
        Operand<T, KJ, FULL> kf[KT];
        float vf[KT][4][DJ][4];
#pragma unroll
        for (int u = 0; u < KT; ++u) {
            kf[u].load(row_of(kb, 16 * u + lr, last), lb, d);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const T *vr = row_of(vb, 16 * u + 4 * lb + i, last);
#pragma unroll
                for (int b = 0; b < DJ; ++b) {
                    if constexpr (VEC) {
                        load_row<4, FULL>(vr, 64 * b + 4 * lr, d, vf[u][i][b]);
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int ch = 64 * b + 4 * lr + e;
                            vf[u][i][b][e] = ch < d ? to_f32(vr[ch]) : 0.f;
                        }
                    }
                }
            }
        }
        f32x4 z[KT];
#pragma unroll
        for (int u = 0; u < KT; ++u) z[u] = zero4();
        products(kf, qf, lb, z);
        float tmax = -INFINITY;
#pragma unroll
        for (int u = 0; u < KT; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (key0 + 16 * u + 4 * lb + i > q0 + lr) z[u][i] = -INFINITY;
                tmax = fmaxf(tmax, z[u][i]);
            }
        // (a trip starts at or before the block's first query: every query sees a key of every trip)
        const float nm = fmaxf(run_m, groups_max(tmax) * scale2);
        const float ref = nm == -INFINITY ? 0.f : nm, corr = ex2(run_m - ref);
        float ts = 0.f;
#pragma unroll
        for (int u = 0; u < KT; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                z[u][i] = ex2(fmaf(z[u][i], scale2, -ref));
                ts += z[u][i];
            }
        run_l = run_l * corr + ts;
        run_m = nm;
#pragma unroll
        for (int b = 0; b < DJ; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[b][e][i] *= corr;
        // A probability of 0 takes a key's values out of the sum only if they are finite (0 x inf is NaN).  Tiles past
        // the block's queries are cleared; in the tile on the diagonal, which some of the queries see and some do not,
        // values that are not finite are taken out of the operand and added query by query, where there are any.
        bool odd = false;  // uniform
        if (edge) {
#pragma unroll
            for (int u = 0; u < KT; ++u) {
                const int ahead = key0 + 16 * u - q0;
                if (ahead < 0) continue;
                float t = 0.f;
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int b = 0; b < DJ; ++b)
#pragma unroll
                        for (int e = 0; e < 4; ++e) t = fmaf(vf[u][i][b][e], 0.f, t);
                if (!__any(t != 0.f)) continue;
                odd |= ahead == 0;
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int b = 0; b < DJ; ++b)
#pragma unroll
                        for (int e = 0; e < 4; ++e) vf[u][i][b][e] = finite(vf[u][i][b][e]) ? vf[u][i][b][e] : 0.f;
            }
        }
#pragma unroll
        for (int u = 0; u < KT; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int b = 0; b < DJ; ++b)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[b][e] = mfma4(vf[u][i][b][e], z[u][i], acc[b][e]);
        if (odd) {
            const int first = q0 - key0;  // the diagonal tile's first key, in the trip
            const f32x4 zd = KT > 1 && first ? z[KT - 1] : z[0];
#pragma unroll 1
            for (int s = 0; s < 16; ++s) {
                const float mine = s & 2 ? (s & 1 ? zd[3] : zd[2]) : (s & 1 ? zd[1] : zd[0]);
                const float pr = __shfl(mine, 16 * (s >> 2) + lr, kWave);
                const T *vr = row_of(vb, first + s, last);
                if (s > lr) continue;
#pragma unroll
                for (int b = 0; b < DJ; ++b)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int ch = 64 * b + 16 * lb + 4 * i + e;
                            const float val = ch < d ? to_f32(vr[ch]) : 0.f;
                            acc[b][e][i] = finite(val) ? acc[b][e][i] : fmaf(pr, val, acc[b][e][i]);
                        }
                        __builtin_amdgcn_sched_barrier(0);  // a few loads at a time: this must not cost the kernel registers
                    }
            }
        }
    };
    // The last trip holds the diagonal (and nothing past it but the rest of its keys).  Up to d = 64 it takes a branch
    // in the loop, which makes the compiler keep the values of a trip in registers from its start (544 tokens, 4 heads
    // 13.0 -> 10.9 us, 4096 of 8 heads 195 -> 179); longer rows have no room for that (4096 tokens, 8 heads of 128
    // 336 -> 410): there the last trip has code of its own and the others are as they were (336 -> 341).
    if constexpr (DJ > 1) {
        int trip = w;
        for (; trip < ntrip - 1; trip += NW) body(std::false_type(), trip);
        if (trip == ntrip - 1) body(std::true_type(), trip);
    } else {
        for (int trip = w; trip < ntrip; trip += NW) body(trip == ntrip - 1, trip);
    }
    run_l = groups_sum(run_l);
#pragma unroll
    for (int b = 0; b < DJ; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *reinterpret_cast<f32x4 *>(&so[w][lr][64 * b + 16 * lb + 4 * i]) =
                f32x4{acc[b][0][i], acc[b][1][i], acc[b][2][i], acc[b][3][i]};
    if (lb == 0) {
        sm[w][lr] = run_m;
        sl[w][lr] = run_l;
    }
    __syncthreads();
    for (int e = tid; e < 16 * d; e += NW * kWave) {
        const int r = e / d, ch = e - r * d;
        if (q0 + r >= Tn) break;
        float mx = sm[0][r];  // wave 0 always has a trip
#pragma unroll
        for (int u = 1; u < NW; ++u) mx = fmaxf(mx, sm[u][r]);
        const float ref = mx == -INFINITY ? 0.f : mx;
        float num = 0.f, den = 0.f;
#pragma unroll
        for (int u = 0; u < NW; ++u) {
            const float cw = ex2(sm[u][r] - ref);  // 0 for a wave without trips
            num = fmaf(cw, so[u][r][ch], num);
            den = fmaf(cw, sl[u][r], den);
        }
        o[((size_t)(q0 + r) * Hq + h) * d + ch] = from_f32<T>(num / den);
    }
}

// Short sequences: one workgroup per (query row, query head).  Keys are walked in tiles of kRowThreads, a thread each,
// with an online softmax; lane c < d accumulates output channel c.  A row's work is one short chain, where a tile's
// waves read 32 rows of K and V at a time, element by element if d is odd; see attn_by_rows.
constexpr int kRowThreads = 256;

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, kWave));
    return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

template <typename T>
__global__ __launch_bounds__(kRowThreads) void attn_row_kernel(const T *__restrict__ q, const T *__restrict__ k,
                                                               const T *__restrict__ v, T *__restrict__ o, int Hq, int Hkv,
                                                               int d, float scale2) {
    extern __shared__ float smem[];  // d (q) + kRowThreads (p) + waves (red)
    float *qs = smem, *ps = smem + d, *red = smem + d + kRowThreads;
    const int t = blockIdx.x / Hq, h = blockIdx.x % Hq, hk = h / (Hq / Hkv);
    for (int c = threadIdx.x; c < d; c += kRowThreads) qs[c] = to_f32(q[((size_t)t * Hq + h) * d + c]);
    __syncthreads();
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    float m_run = -INFINITY, l_run = 0.f, acc = 0.f;  // acc: channel threadIdx.x (< d)
    for (int j0 = 0; j0 <= t; j0 += kRowThreads) {
        const int j = j0 + threadIdx.x;
        float z = -INFINITY;
        if (j <= t) {
            const T *kv = k + ((size_t)j * Hkv + hk) * d;
            float dot[4] = {0.f, 0.f, 0.f, 0.f};  // four chains: less rounding, and a quarter of the wait
            int c = 0;
            for (; c + 4 <= d; c += 4)
#pragma unroll
                for (int i = 0; i < 4; ++i) dot[i] = fmaf(qs[c + i], to_f32(kv[c + i]), dot[i]);
            for (; c < d; ++c) dot[0] = fmaf(qs[c], to_f32(kv[c]), dot[0]);
            z = scale2 * ((dot[0] + dot[1]) + (dot[2] + dot[3]));
        }
        const float wm = wave_max(z);
        if (lane == 0) red[wave] = wm;
        __syncthreads();
        float tm = -INFINITY;
        for (int w = 0; w < kRowThreads / kWave; ++w) tm = fmaxf(tm, red[w]);
        const float m_new = fmaxf(m_run, tm), ref = m_new == -INFINITY ? 0.f : m_new;
        const float pj = j <= t ? ex2(z - ref) : 0.f;
        ps[threadIdx.x] = pj;
        const float wsum = wave_sum(pj);
        __syncthreads();  // ps complete, red (max) consumed
        if (lane == 0) red[wave] = wsum;
        __syncthreads();
        float tsum = 0.f;
        for (int w = 0; w < kRowThreads / kWave; ++w) tsum += red[w];
        const float corr = ex2(m_run - ref);  // 0 on the first tile (m_run = -inf)
        l_run = l_run * corr + tsum;
        m_run = m_new;
        if (threadIdx.x < d) {
            const int cnt = min(kRowThreads, t + 1 - j0);
            const T *vc = v + ((size_t)j0 * Hkv + hk) * d + threadIdx.x;
            const size_t pitch = (size_t)Hkv * d;
            float sum[4] = {0.f, 0.f, 0.f, 0.f};
            int jj = 0;
            for (; jj + 4 <= cnt; jj += 4)
#pragma unroll
                for (int i = 0; i < 4; ++i) sum[i] = fmaf(ps[jj + i], to_f32(vc[(jj + i) * pitch]), sum[i]);
            for (; jj < cnt; ++jj) sum[0] = fmaf(ps[jj], to_f32(vc[jj * pitch]), sum[0]);
            acc = fmaf(acc, corr, (sum[0] + sum[1]) + (sum[2] + sum[3]));
        }
        __syncthreads();  // before ps / red are overwritten
    }
    if (threadIdx.x < d) o[((size_t)t * Hq + h) * d + threadIdx.x] = from_f32<T>(acc / l_run);
}

// Rows of `len` elements from bases `p...` can be read 4 elements at a time.
template <typename T, typename... Ptr>
inline bool vec4(int len, const Ptr *...p) {
    return len % 4 == 0 && ((... | (uintptr_t)p) % (4 * sizeof(T))) == 0;
}
// LAUNCH(operand registers, exact): rows of `len` elements fill 1, 4 or 8 operand vectors a lane, exactly or
// with zeros behind them; 0: longer rows or no vectors, operands are read per product.
#define STRD_BY_ROW(LAUNCH, vec, len)                \
    if (!(vec) || (len) > 128) { LAUNCH(0, false); } \
    else if ((len) == 16) { LAUNCH(1, true); }       \
    else if ((len) < 16) { LAUNCH(1, false); }       \
    else if ((len) == 64) { LAUNCH(4, true); }       \
    else if ((len) < 64) { LAUNCH(4, false); }       \
    else if ((len) == 128) { LAUNCH(8, true); }      \
    else { LAUNCH(8, false); }

struct StatPlan {
    int nrb, nslice, keys_per_slice;
};
// About 1024 workgroups of pass 1 over all sequences, and at most 32 slices: pass 2 reads every slice's
// statistics once per workgroup.
StatPlan stat_plan(int M, int N, int Hq, int Hkv, int nseq) {
    StatPlan p;
    p.nrb = ceil_div(M * (Hq / Hkv), kStatRows);
    const long long units = (long long)p.nrb * Hkv * nseq;
    const int want = (int)std::max(1LL, std::min({32LL, 1024 / std::min(1024LL, units), (long long)ceil_div(N, 64)}));
    p.keys_per_slice = ceil_div(ceil_div(N, want), 64) * 64;
    p.nslice = ceil_div(N, p.keys_per_slice);
    return p;
}

}  // namespace

// ------------------------------------------------------------------ host launchers ---------
size_t score_attn_general_ws(int M, int N, int Hq, int Hkv, int nseq) {
    return align_up((size_t)2 * stat_plan(M, N, Hq, Hkv, nseq).nslice * M * Hq * nseq * sizeof(float), 256);
}

template <typename T, class SEQ>
static int score_attn_launch(const void *q, const void *k, float *s, int M, int N, int Hq, int Hkv, int d, float scale,
                             void *ws, const SEQ &seq, int nseq, int ld, hipStream_t st) {
    if (d > kMaxScoreRow) return STRD_EUNSUPPORTED;
    const StatPlan p = stat_plan(M, N, Hq, Hkv, nseq);
    const long long grid1 = (long long)p.nrb * Hkv * p.nslice;
    if (grid1 > 0x7FFFFFFFLL) return STRD_EUNSUPPORTED;
    const size_t stride = (size_t)p.nslice * M * Hq;
    float *pmax = (float *)ws, *psum = pmax + stride * nseq;
#define STRD_SCORE_ATTN(KJ, FULL)                                                                                         \
    attn_stats_kernel<T, KJ, FULL, SEQ><<<dim3((unsigned)grid1, nseq), 256, 0, st>>>(                                      \
        (const T *)q, (const T *)k, pmax, psum, M, N, Hq, Hkv, d, scale * kLog2e, p.nrb, p.keys_per_slice, seq, stride);  \
    attn_col_sum_kernel<T, KJ, FULL, SEQ><<<dim3(ceil_div(N, 16), nseq), kColThreads, 0, st>>>(                            \
        (const T *)q, (const T *)k, pmax, psum, s, M, N, Hq, Hkv, d, scale * kLog2e, p.nslice, seq, stride, ld)
    STRD_BY_ROW(STRD_SCORE_ATTN, vec4<T>(d, (const T *)q, (const T *)k), d)
#undef STRD_SCORE_ATTN
    return launch_status();
}

int score_attn_general(const void *q, const void *k, float *s, int M, int N, int Hq, int Hkv, int d,
                       float scale, strd_dtype io, void *ws, hipStream_t st) {
    if (io == STRD_F32) return score_attn_launch<float>(q, k, s, M, N, Hq, Hkv, d, scale, ws, OneSeq(), 1, 0, st);
    return score_attn_launch<bf16_t>(q, k, s, M, N, Hq, Hkv, d, scale, ws, OneSeq(), 1, 0, st);
}

// Packed batch: grids sized for the longest sequence, statistics of every sequence in a region of its own.
int score_attn_general_varlen(const void *q, const void *k, float *s, int ld, const SeqTab &tab, int nseq, int max_m,
                              int max_n, int Hq, int Hkv, int d, float scale, strd_dtype io, void *ws, hipStream_t st) {
    if (io == STRD_F32)
        return score_attn_launch<float>(q, k, s, max_m, max_n, Hq, Hkv, d, scale, ws, tab, nseq, ld, st);
    return score_attn_launch<bf16_t>(q, k, s, max_m, max_n, Hq, Hkv, d, scale, ws, tab, nseq, ld, st);
}

template <typename T, class SEQ>
static int score_mamba_launch(const void *B, const void *C, const float *dt, float *s, int M, int N, int H, int G, int n,
                              const SEQ &seq, int nseq, int ld, hipStream_t st) {
    const dim3 grid(ceil_div(N, 16), nseq);
#define STRD_SCORE_MAMBA(KJ, FULL)                                                                                 \
    mamba_score_kernel<T, KJ, FULL, SEQ><<<grid, kColThreads, 0, st>>>((const T *)B, (const T *)C, dt, s, M, N, H, G, n, \
                                                                       seq, ld)
    STRD_BY_ROW(STRD_SCORE_MAMBA, vec4<T>(n, (const T *)B, (const T *)C), n)
#undef STRD_SCORE_MAMBA
    return launch_status();
}

// The floats behind every sequence's scores, `ld` apart, become 0.
static __global__ __launch_bounds__(256) void scores_pad_kernel(float *__restrict__ s, SeqTab seq, int ld) {
    const int i = seq.N[blockIdx.y] + blockIdx.x * 256 + threadIdx.x;
    if (i < ld) s[(size_t)blockIdx.y * ld + i] = 0.f;
}
int scores_pad(float *s, int ld, const SeqTab &tab, int nseq, hipStream_t st) {
    int most = 0;
    for (int b = 0; b < nseq; ++b) most = std::max(most, ld - tab.N[b]);
    if (most > 0) scores_pad_kernel<<<dim3(ceil_div(most, 256), nseq), 256, 0, st>>>(s, tab, ld);
    return launch_status();
}
int score_mamba_general(const void *B, const void *C, const float *dt, float *s, int M, int N, int H,
                        int G, int n, strd_dtype io, hipStream_t st) {
    if (io == STRD_F32) return score_mamba_launch<float>(B, C, dt, s, M, N, H, G, n, OneSeq(), 1, 0, st);
    return score_mamba_launch<bf16_t>(B, C, dt, s, M, N, H, G, n, OneSeq(), 1, 0, st);
}

int score_mamba_general_varlen(const void *B, const void *C, const float *dt, float *s, int ld, const SeqTab &tab, int nseq, int max_n,
                               int H, int G, int n, strd_dtype io, hipStream_t st) {
    if (io == STRD_F32) return score_mamba_launch<float>(B, C, dt, s, 0, max_n, H, G, n, tab, nseq, ld, st);
    return score_mamba_launch<bf16_t>(B, C, dt, s, 0, max_n, H, G, n, tab, nseq, ld, st);
}

bool ssd_general_supported(int n) { return n >= 1 && n <= 1024; }

// Workspace: the state before every chunk [H][chunks][P][n] and the chunks' total decays [H][chunks].  Long
// sequences go through it in rounds of as many chunks as fit kRoundBytes (at 128 heads of 64 x 128: 4096 tokens, 8192
// workgroups a launch), the state handed on in two more buffers that take turns: 131072 tokens take 276 MB, not 8.6 GB.
constexpr size_t kRoundBytes = (size_t)256 << 20;
// The chunked form's launches count 32-bit threads per grid: states of up to 2^28 entries (1 GB) in fewer than 2^24
// heads.  Beyond, there are channels enough to fill the chip with the recurrence.  And it is two or three launches, of
// 10 us for the shortest sequence (16 state entries) to 32 (1024, whose rows are read per product), where a token of the
// recurrence takes 1.2 to 3.7: us in chunks / as a recurrence, 1 and 5 and 8 tokens: 8 heads of 32, n = 16 10.7 / 5.9,
// 10.7 / 10.7, 10.7 / 14.3; 128 heads of 64, n = 124 23.5 / 10.0, 23.7 / 18.4, 23.8 / 24.5; n = 1024, 8 heads 32 / 10, 34 / 25,
// 37 / 37; 128 heads of 64, n = 256, where every CU has its share of the lanes, 32 / 20, 32 / 47 and at 2 tokens 32 / 27.
static bool ssd_in_chunks(int T, int H, int P, int n) {
    if (H >= 1 << 24 || (long long)H * P > (1 << 28) / n) return false;
    if (n <= 128) return T > (n < 32 ? 5 : H < 256 ? 6 : 8);
    if ((long long)H * P * ceil_div(n, kSlice) > 1 << 16) return T > 2;
    return T > (n <= 256 ? 4 : n <= 512 ? 6 : 8);
}
struct ScanRounds {
    int chunks;  // per round
    size_t states, decays, carry;  // bytes
    size_t total() const { return states + decays + 2 * carry; }
};
static ScanRounds ssd_rounds(int T, int H, int P, int n) {
    const size_t state = (size_t)H * P * n * sizeof(float);
    const int nc = ceil_div(T, kChunk);
    ScanRounds r;
    r.chunks = (int)std::min<size_t>(nc, std::max<size_t>(1, kRoundBytes / std::max(state, (size_t)H * 64)));
    r.states = align_up(r.chunks * state, 256);
    r.decays = align_up((size_t)H * r.chunks * sizeof(float), 256);
    r.carry = nc > r.chunks ? align_up(state, 256) : 0;
    return r;
}
size_t ssd_general_ws(int T, int H, int P, int n) { return ssd_in_chunks(T, H, P, n) ? ssd_rounds(T, H, P, n).total() : 0; }

// Few chunks of small states go in one launch: while no state wave has more than two chunk states to make, and all workgroups
// together not many more than the chip has waves for.  us, three launches -> one (fp32, 16 state entries): 8 heads of 32, 65 tokens
// 11.9 -> 6.8, 544 13.5 -> 10.1, 800 13.8 -> 12.4 (1088 14.4 either way, 1600 15.3 / 18.3); 32 heads, 544 tokens 14.5 -> 13.2 (800
// 16.3 / 17.8); 64 heads of 64, 200 tokens 16.3 -> 10.8 (544 23.7 / 30.0); 256 of 32, 128 tokens 15.5 -> 14.1 (200 20.7 / 27.6).
// Of heads with many channels a workgroup has the blocks one after the other, which the separate launches share out: 512 channels, 9
// tokens 17 / 21, 128 30 / 33; 384, 9 15.6 / 16.3; 256, 128 21.2 / 22.6 (9 14.1 -> 12.3); 192, 128 18.9 -> 17.8.  And one chunk that starts
// from nothing and leaves nothing is one launch anyway (`carried`: there is a state carried in): 64 channels 5.3 / 5.6, 256 8.8 / 10.8.
// The workgroup has LDS for one state at least (the one before its chunk), also where no chunk's is asked for.
constexpr int once_states(int nst) { return nst > 1 ? nst : 1; }
constexpr size_t once_lds(int nst, int P, int n) { return (size_t)once_states(nst) * P * n * sizeof(float); }
constexpr bool ssd_at_once(int nc, int nst, bool carried, int H, int P, int n) {
    // blocks of 32 channels x 16 state entries, 2 KB of LDS each: 32 KB at most
    const long long states = (long long)once_states(nst) * (P / 32 + (P % 32 != 0));
    return (nst > 0 || carried) && (P <= 192 || (P <= 256 && nst <= 1)) && n <= 16 && nc <= kOnceChunks && states <= 2 * kOnceStateWaves && states * nc * H <= 3000;
}

template <typename T>
static int ssd_launch(const void *x, const float *dt, const float *A, const void *B, const void *C, const float *D,
                      const float *S_in, void *y, float *S_out, int Tn, int H, int P, int G, int n, float *L, float *decay,
                      hipStream_t st) {
    const int nc = ceil_div(Tn, kChunk), nst = S_out ? nc : nc - 1;  // chunks whose contribution to the state is needed
    const bool vec = vec4<T>(P, (const T *)x, (const T *)y) && vec4<T>(n, (const T *)B, (const T *)C);
    const int cpl = !vec ? 1 : P > 32 ? 4 : 2, npl = vec && n >= 64 ? 4 : 1;
    // (there every workgroup of a head reads S_in and one writes S_out: not in place)
    if (vec && ssd_at_once(nc, nst, S_in, H, P, n) && !overlap(S_in, S_out, (size_t)H * P * n * sizeof(float))) {
        const size_t lds = once_lds(nst, P, n);
#define STRD_SSD_ONCE(FF)                                                                                                    \
    ssd_once_kernel<T, 2, 1, FF><<<(unsigned)(nc * H), kOnceThreads, lds, st>>>((const T *)x, dt, A, (const T *)B, (const T *)C, D, \
                                                                               S_in, (T *)y, S_out, Tn, H, P, G, n, nc)
        if (P % 32 == 0 && n == 16) STRD_SSD_ONCE(true);
        else STRD_SSD_ONCE(false);
#undef STRD_SSD_ONCE
        return launch_status();
    }
    const int pblocks = ceil_div(P, 16 * cpl), nblocks = ceil_div(n, 16 * npl);
    const long long grid1 = (long long)nst * H * pblocks * nblocks, total = (long long)H * P * n, grid3 = (long long)nc * H;
    const long long grid2 = (total + kWave - 1) / kWave;
#define STRD_SSD_STATE(CC, NN, FF)                                                                                   \
    ssd_chunk_state_kernel<T, CC, NN, FF><<<(unsigned)grid1, kWave, 0, st>>>((const T *)x, dt, A, (const T *)B, L, decay, \
                                                                             Tn, H, P, G, n, nc, nst, pblocks)
#define STRD_SSD_STATE_N(CC, FF)                   \
    if (npl == 4) { STRD_SSD_STATE(CC, 4, FF); }   \
    else { STRD_SSD_STATE(CC, 1, FF); }
    if (nst > 0) {
        const bool full = P % (16 * cpl) == 0 && n % (16 * npl) == 0;
        if (cpl == 4 && full) { STRD_SSD_STATE_N(4, true) }
        else if (cpl == 4) { STRD_SSD_STATE_N(4, false) }
        else if (cpl == 2 && full) { STRD_SSD_STATE_N(2, true) }
        else if (cpl == 2) { STRD_SSD_STATE_N(2, false) }
        else STRD_SSD_STATE(1, 1, false);
    }
#undef STRD_SSD_STATE_N
#undef STRD_SSD_STATE
    // nothing to pass on where one chunk starts from zero and nobody asks for its state
    if (nst > 0 || S_in)
        ssd_pass_kernel<<<(unsigned)grid2, kWave, 0, st>>>(L, decay, S_in, S_out, total, P * n, nc, nst);
    const int first_carried = S_in ? 0 : 1;
#define STRD_SSD_OUT(CC, KK, FF)                                                                                     \
    ssd_chunk_out_kernel<T, CC, KK, FF><<<(unsigned)grid3, 256, 0, st>>>((const T *)x, dt, A, (const T *)B, (const T *)C, D, \
                                                                         L, (T *)y, Tn, H, P, G, n, nc, first_carried)
#define STRD_SSD_OUT4(KK, FF) STRD_SSD_OUT(4, KK, FF)
#define STRD_SSD_OUT2(KK, FF) STRD_SSD_OUT(2, KK, FF)
    const bool pfull = P % (16 * cpl) == 0;
    const int nn = pfull ? n : n - (n == 16 || n == 64 || n == 128);  // "exact" needs whole channel blocks as well
    if (cpl == 4) { STRD_BY_ROW(STRD_SSD_OUT4, true, nn) }
    else if (cpl == 2) { STRD_BY_ROW(STRD_SSD_OUT2, true, nn) }
    else STRD_SSD_OUT(1, 0, false);
#undef STRD_SSD_OUT2
#undef STRD_SSD_OUT4
#undef STRD_SSD_OUT
    return launch_status();
}

template <typename T>
static int ssd_in_rounds(const void *x, const float *dt, const float *A, const void *B, const void *C, const float *D,
                         const float *S_in, void *y, float *S_out, int Tn, int H, int P, int G, int n, void *ws,
                         hipStream_t st) {
    const ScanRounds r = ssd_rounds(Tn, H, P, n);
    char *p = (char *)ws;
    float *L = (float *)p, *decay = (float *)(p + r.states);
    float *carry[2] = {(float *)(p + r.states + r.decays), (float *)(p + r.states + r.decays + r.carry)};
    const int step = r.chunks * kChunk;
    for (long long t0 = 0, i = 0; t0 < Tn; t0 += step, ++i) {
        const bool last = Tn - t0 <= step;
        const int rc = ssd_launch<T>((const T *)x + t0 * H * P, dt + t0 * H, A, (const T *)B + t0 * G * n, (const T *)C + t0 * G * n, D,
                                     i ? carry[(i - 1) & 1] : S_in, (T *)y + t0 * H * P, last ? S_out : carry[i & 1],
                                     last ? (int)(Tn - t0) : step, H, P, G, n, L, decay, st);
        if (rc != STRD_OK) return rc;
    }
    return STRD_OK;
}

// ws = nullptr: a caller without a workspace gets the recurrence.
int ssd_general(const void *x, const float *dt, const float *A, const void *B, const void *C,
                const float *D, const float *S_in, void *y, float *S_out, int T, int H, int P, int G,
                int n, strd_dtype io, void *ws, hipStream_t st) {
    if (T == 0 || !ws || !ssd_in_chunks(T, H, P, n)) {
        int lanes = 1;
        while (lanes * kSlice < n) lanes <<= 1;  // power of two <= 64, so a column never straddles a wave
        const long long threads = (long long)H * P * lanes;
        if (threads > (1LL << 30)) return STRD_EUNSUPPORTED;
        const int grid = (int)((threads + kRecThreads - 1) / kRecThreads);
        if (io == STRD_F32)
            ssd_recurrence_kernel<float><<<grid, kRecThreads, 0, st>>>((const float *)x, dt, A, (const float *)B, (const float *)C, D,
                                                                       S_in, (float *)y, S_out, T, H, P, G, n, lanes);
        else
            ssd_recurrence_kernel<bf16_t><<<grid, kRecThreads, 0, st>>>((const bf16_t *)x, dt, A, (const bf16_t *)B,
                                                                        (const bf16_t *)C, D, S_in, (bf16_t *)y, S_out, T, H, P, G,
                                                                        n, lanes);
        return launch_status();
    }
    if (io == STRD_F32) return ssd_in_rounds<float>(x, dt, A, B, C, D, S_in, y, S_out, T, H, P, G, n, ws, st);
    return ssd_in_rounds<bf16_t>(x, dt, A, B, C, D, S_in, y, S_out, T, H, P, G, n, ws, st);
}

bool attn_general_supported(int d) { return d >= 1 && d <= 256; }

// Short sequences go row by row.  The tiles' time is a chain that grows with T (and with d: 2 waves a workgroup above
// 128; and with every element of a row that vectors cannot read), the rows' with T * T * Hq, so the line lies at about
// T * (Hq + a few): us as tiles / as rows, fp32, 4 query heads: d = 200, 200 tokens 43 / 18, 600 113 / 113; d = 130, 600
// 109 / 92, 1000 177 / 230; d = 100, 100 10.3 / 8.1, 200 15.5 / 13.5, 300 20 / 22; d = 65, 300 25 / 20, 600 40 / 50; d = 33,
// 64 7.0 / 6.1, 100 7.4 / 7.3; bf16: d = 130, 1000 370 / 180, 1500 562 / 400; d = 33 200 12.1 / 12.7.  (Rows of up to 64
// elements that vectors read: equal within 0.7 us up to 16 tokens, tiles from there on.)
static bool attn_by_rows(int T, int Hq, int d, bool vec, bool half) {
    auto below = [&](int extra, int line) { return (long long)T * (Hq + extra) <= line; };
    if (d <= 64) return !vec && below(4, half ? 2320 : 450);
    if (d <= 128) return vec ? below(4, d == 128 ? 640 : 1300) : below(1, half ? 4960 : 2560);
    if (d == 256 && vec) return below(1, half ? 2200 : 1300);
    return vec ? below(0, half ? 3300 : 3000) : below(0, half ? 6600 : 3300);
}

template <typename T>
static int attn_launch(const void *q, const void *k, const void *v, void *o, int Tn, int Hq, int Hkv, int d, float scale,
                       hipStream_t st) {
    const long long grid = (long long)ceil_div(Tn, 16) * Hq;
    if ((long long)Tn * Hq > 0x7FFFFFFFLL) return STRD_EUNSUPPORTED;
    if (attn_by_rows(Tn, Hq, d, vec4<T>(d, (const T *)q, (const T *)k, (const T *)v), sizeof(T) == 2)) {
        attn_row_kernel<T><<<Tn * Hq, kRowThreads, (size_t)(d + kRowThreads + kRowThreads / kWave) * sizeof(float), st>>>(
            (const T *)q, (const T *)k, (const T *)v, (T *)o, Hq, Hkv, d, scale * kLog2e);
        return launch_status();
    }
    const bool wide = (long long)Hkv * d * (long long)sizeof(T) >= 1 << 24;  // rows that a 24-bit product does not reach
#define STRD_ATTN_W(VV, FF, DD, NN, WW)                                                                                  \
    attn_tile_kernel<T, VV, FF, DD, NN, WW><<<(unsigned)grid, NN * kWave, 0, st>>>(                                      \
        (const T *)q, (const T *)k, (const T *)v, (T *)o, Tn, Hq, Hkv, d, scale * kLog2e)
#define STRD_ATTN(VV, FF, DD, NN) STRD_ATTN_W(VV, FF, DD, NN, false)
    if (wide) {
        if (d <= 64) STRD_ATTN_W(false, false, 1, 8, true);
        else if (d <= 128) STRD_ATTN_W(false, false, 2, 4, true);
        else STRD_ATTN_W(false, false, 4, 2, true);
    } else if (!vec4<T>(d, (const T *)q, (const T *)k, (const T *)v)) {
        if (d <= 64) STRD_ATTN(false, false, 1, 8);
        else if (d <= 128) STRD_ATTN(false, false, 2, 4);
        else STRD_ATTN(false, false, 4, 2);
    } else if (d == 64) STRD_ATTN(true, true, 1, 8);
    else if (d < 64) STRD_ATTN(true, false, 1, 8);
    else if (d == 128) STRD_ATTN(true, true, 2, 4);
    else if (d < 128) STRD_ATTN(true, false, 2, 4);
    else if (d == 256) STRD_ATTN(true, true, 4, 2);
    else STRD_ATTN(true, false, 4, 2);
#undef STRD_ATTN
#undef STRD_ATTN_W
    return launch_status();
}

int attn_general(const void *q, const void *k, const void *v, void *o, int T, int Hq, int Hkv, int d,
                 float scale, strd_dtype io, hipStream_t st) {
    if (T == 0) return STRD_OK;
    if (io == STRD_F32) return attn_launch<float>(q, k, v, o, T, Hq, Hkv, d, scale, st);
    return attn_launch<bf16_t>(q, k, v, o, T, Hq, Hkv, d, scale, st);
}

}  // namespace strd
