// ssd_prefill on bf16 matrix cores: the Mamba-2 recurrence (paper Eqs. "ssm_state_update",
// "ssm_output") in its chunked form, i.e. the unrolled sum (Eq. "ssm_unrolled") split at
// 64-token boundaries, with the recurrent state of a head kept in the registers of the waves
// that own it for a whole segment of the sequence.
//
// Decomposition.  One workgroup owns 32*NC consecutive channels of one head (NC = 2: the whole
// head when P = 64) -- or, NH = 2, two whole heads of one group -- and one segment of the
// sequence, which it walks in 64-token steps.  Per step and head, with l_t the in-step cumulative
// sum of dt*A (log2 units):
//   (a) G^T[j,t] = b_j . c_t                                      contraction over the state dim n
//   (b) M[t,j]   = G^T[j,t] * 2^(l_t-l_j) * dt_j  for j <= t, else 0;  M[t,t] += D   (fp32, then bf16)
//   (c) Y^T[p,t] = sum_j x_j[p] M[t,j]                            contraction over tokens
//   (d) Y^T[p,t] += 2^(l_t) * sum_n S[p,n] c_t[n]                 S = state before the step
//   (e) S^T[n,p] = 2^(l_Q) S^T[n,p] + sum_j b_j[n] (w_j x_j[p]),  w_j = dt_j 2^(l_Q-l_j)
// every product a v_mfma_f32_16x16x32_bf16 (the skip term D x_t of the output rides on (c) through
// the diagonal of M).  (a) and (b) depend on the head only, not on the channel: two "G waves" per
// head do them once, two query blocks of 16 tokens each, keep the weights M in registers -- the
// accumulators of (a), rounded to bf16, are the B operand of (c) as they stand -- and go on to (c)
// for all the head's channels and to the outputs.  (d) and (e) belong to NC "compute waves" per
// head, one per slab of 32 channels, which hold their slab's state S^T[n, 32] in fp32 accumulator
// registers from the first step to the last.  The accumulator layout of (e) is at the same time
// the A-operand layout of (d) (the contraction index n runs over the accumulator rows a lane
// holds), so the state is converted to bf16 in registers and never passes through LDS; the
// carried part (d) of a step's outputs goes to the G waves through LDS in accumulator layout,
// rounded to bf16 (8 bytes per lane, no bank conflicts).
//
// Waves (NH (NC + 2) + 4): per head NC compute waves and 2 G waves; one wave each that only
// requests the asynchronous global -> LDS copies of the B tiles, the C tiles and the x tiles; a
// helper wave that requests dt three steps ahead and turns it into the scan l_t, the key factors
// of (b), the weights of (e) and the carries of (d) one step ahead (and keeps the row tables of
// the gather form).  One LDS-only barrier per step.  The outputs of a step leave one step late:
// the G waves keep (c) of step i in registers, the compute waves leave the carried part (d) of
// step i in LDS (bf16, double-buffered), the barrier that ends the step publishes it, and the G
// waves add the two and store them while the arithmetic of step i + 1 runs.
//
// One head per workgroup (NH = 1): 8 waves, two per SIMD, 256 registers each; tiles two steps
// ahead (rings of 3), every LDS read of a step requested at its start.  Two heads (NH = 2, P = 64
// and an even number of heads per group): 12 waves, three per SIMD -- a compute wave, a G wave
// and a copy wave -- so that the vector work of one arithmetic wave runs under the matrix
// products and LDS round trips of the other, and the B and C tiles cross the CU's copy path once
// for both heads.  That leaves 168 registers per wave and LDS for rings of 2 (tiles one step
// ahead): reads are requested where they are needed instead of at the start of the step.
//
// Segments.  A head is a serial chain over time; to fill the chip the sequence is cut into a few
// long segments that run side by side, each from a zero state (the first from S_in).  A segment
// leaves its final local state and its total decay in the workspace; a second, small kernel adds
// what the true incoming state contributes to the first tokens of each later segment,
//   y_t += 2^(l_t) * E c_t,   E = state at the segment's start, l_t = decay since then,
// for as many 64-token tiles as 2^(l_t) is not yet zero in fp32 (a handful at the decay rates of
// a trained layer, the whole segment if A = 0: always exact), and completes S_out.
//
// GATHER: token t of the sequence is row idx[t] (t < K) or N + t - K of the tensors, i.e. the
// kernel reads the uncompacted x, dt, B, C through the kept-index list instead of a compacted copy.
#include "ssd_seg.h"

namespace strd {
namespace {

using namespace seg;

template <int NS, int NC, int NH, bool GATHER>
__global__ __launch_bounds__(threads_for(NC, NH)) void ssd_seg_kernel(SegArgs a, int nunits) {
    using L = LdsS<NS, NC, NH>;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    L &lds = *reinterpret_cast<L *>(smem_raw);

    const int unit = xcd_swizzle(blockIdx.x, nunits);
    if (unit >= nunits) return;
    const int seg = unit / a.wg_per_seg, u = unit % a.wg_per_seg;
    const int chan0 = u * (32 * NC * NH);  // NH = 2: two whole heads of one group (P = 32 NC)
    const int h0 = chan0 / a.P, pin = chan0 % a.P, g = h0 / (a.H / a.G);
    const int nsteps = (a.T + kQ - 1) / kQ;
    const int s0 = seg * a.seg_steps;
    const int nloc = min(a.seg_steps, nsteps - s0);
    const int tok0 = s0 * kQ;
    // where the segment's state comes from and goes to
    const float *s_src = seg == 0 ? a.S_in : nullptr;
    float *s_dst = seg == a.nseg - 1 ? a.S_out : a.lend + (size_t)seg * a.H * a.P * NS;
    // Wave i runs on SIMD i % 4.  NH = 1, NC = 2: the compute waves have SIMDs 0 and 1, the G waves 2 and 3, each
    // with one copy wave beside it.  NH = 2: every SIMD has one compute wave, one G wave and one copy wave, so
    // the vector work of one overlaps the matrix products of the other.
    const int wave = threadIdx.x >> 6;
    if (wave < NH * NC) {
        const int hh = NH == 1 ? 0 : wave / NC, cw = NH == 1 ? wave : wave % NC;
        compute_wave<NS, NC, NH, GATHER>(lds, a, hh, cw, h0 + hh, pin, nloc, s_src, s_dst);
        return;
    }
    const int r = wave - NH * NC;
    if (r < 2 * NH) {
        const int hh = NH == 1 ? 0 : r >> 1;
        if (r & 1)
            g_wave<NS, NC, NH, 1, GATHER>(lds, a, hh, h0 + hh, chan0 + hh * 32 * NC, tok0, nloc);
        else
            g_wave<NS, NC, NH, 0, GATHER>(lds, a, hh, h0 + hh, chan0 + hh * 32 * NC, tok0, nloc);
        return;
    }
    switch (r - 2 * NH) {
        case 0: copy_wave<NS, NC, NH, 1, GATHER>(lds, a, g * NS * 2, tok0, nloc); break;
        case 1: copy_wave<NS, NC, NH, 2, GATHER>(lds, a, g * NS * 2, tok0, nloc); break;
        case 2: helper_wave<NS, NC, NH, GATHER>(lds, a, h0, tok0, nloc, seg); break;
        default: copy_wave<NS, NC, NH, 0, GATHER>(lds, a, chan0 * 2, tok0, nloc); break;
    }
}

// ---- the contribution of the incoming state to the first tokens of segments 1.. and S_out -----
// grid = (boundary b = 1..nseg, head, share z); b < nseg: y of segment b; b == nseg: S_out.
// One workgroup per (boundary, head), or a few that take its 64-token tiles in turn (see fix_shares), a wave per 16-channel
// tile.  At the decay rates of a trained layer the incoming state is gone after two or three tiles, so the kernel is
// a chain of loads: dt, the state E and the rows of the first tile travel together.  The rows of the next tile are fetched when their
// turn comes: held beside the current ones they cost the second workgroup of a CU.  (Always four workgroups per
// (boundary, head) read dt and E four times over and take four rounds of the chip at 128 heads; one takes one, and the scan
// 2 to 6 us less at 2500 to 33280 tokens.)
constexpr int kFixThreads = 256;
constexpr int kFixBatch = 4;  // tiles whose dt is read at once

template <int NS, bool GATHER>
__global__ __launch_bounds__(kFixThreads) void ssd_fix_kernel(SegArgs a) {
    constexpr int KS = NS / 32;
    const int b = 1 + blockIdx.x, h = blockIdx.y, z = blockIdx.z, nz = gridDim.z;
    const int lane = threadIdx.x & 63, lr = lane & 15, lb = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const size_t seg_elems = (size_t)a.H * a.P * NS;
    // weight of segment s' < b in the state at the start of segment b: prod_{s' < u < b} 2^(ltot[u])
    // (uniform; the loops below stop at the first segment whose weight is zero)
    if (b == a.nseg) {
        if (!a.S_out) return;
        float f = fast_exp2(a.ltot[(size_t)(b - 1) * a.H + h]);
        const int per = a.P * NS / 4;  // float4s of the head's state
        for (int s = b - 2; s >= 0 && f != 0.f; --s) {
            const float *src = a.lend + (size_t)s * seg_elems + (size_t)h * a.P * NS;
            float *dst = a.S_out + (size_t)h * a.P * NS;
            for (int e = z * kFixThreads + threadIdx.x; e < per; e += nz * kFixThreads) {
                f32x4 v = reinterpret_cast<const f32x4 *>(src)[e], o = reinterpret_cast<f32x4 *>(dst)[e];
                reinterpret_cast<f32x4 *>(dst)[e] = o + f * v;
            }
            f *= fast_exp2(a.ltot[(size_t)s * a.H + h]);
        }
        return;
    }
    const int HP = a.H * a.P, g = h / (a.H / a.G);
    const int tok0 = b * a.seg_steps * kQ;
    const int tend = min(a.T, (b + 1) * a.seg_steps * kQ);
    const int npt = a.P / 16;
    if (wave >= npt || tok0 + z * kQ >= tend) return;
    const float Al2 = a.A[h] * kLog2e;
    auto row_of = [&](int t) -> size_t {
        t = min(t, a.T - 1);
        return GATHER ? (size_t)gather_row(a, t, a.idx[min(t, a.K - 1)]) : (size_t)t;
    };
    float dv[kFixBatch];  // lane = token
    auto load_dt = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < kFixBatch; ++q) {
            const int t = tok0 + (k0 + q) * kQ + lane;
            dv[q] = t < tend ? a.dt[row_of(t) * a.H + h] : 0.f;
        }
    };
    // c rows of a tile (B operand: column = token 16 tt + lr) and the outputs they correct
    struct Rows {
        bf16x8 c[4][KS];
        bf16x4 y[4];
    };
    auto y_at = [&](int k, int tt, int pt) -> bf16x4 * {
        const int tq = min(tok0 + k * kQ + 16 * tt + lr, a.T - 1);
        return reinterpret_cast<bf16x4 *>(a.y + (size_t)tq * HP + (size_t)h * a.P + 16 * pt + 4 * lb);
    };
    auto load_rows = [&](int k, int pt, Rows &r) __attribute__((always_inline)) {
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            const bf16_t *crow = a.C + (row_of(tok0 + k * kQ + 16 * tt + lr) * a.G + g) * NS + 8 * lb;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) r.c[tt][ks] = *reinterpret_cast<const bf16x8 *>(crow + 32 * ks);
            r.y[tt] = *y_at(k, tt, pt);
        }
    };
    for (int pt = wave; pt < npt; pt += kFixThreads / 64) {
        load_dt(0);
        Rows r;
        load_rows(z, pt, r);
        // E = state at the start of segment b, as A-operand fragments (rows p = 16 pt + lr, k slots
        // n = 32 ks + 8 lb + s)
        bf16x8 ef[KS];
        {
            f32x4 acc[KS][2];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) acc[ks][0] = acc[ks][1] = f32x4{0.f, 0.f, 0.f, 0.f};
            float f = 1.f;
            for (int s = b - 1; s >= 0 && f != 0.f; --s) {
                const float *src = a.lend + (size_t)s * seg_elems + ((size_t)h * a.P + 16 * pt + lr) * NS + 8 * lb;
                f32x4 v[KS][2];
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    v[ks][0] = *reinterpret_cast<const f32x4 *>(src + 32 * ks);
                    v[ks][1] = *reinterpret_cast<const f32x4 *>(src + 32 * ks + 4);
                }
                const float lt = a.ltot[(size_t)s * a.H + h];
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    acc[ks][0] += f * v[ks][0];
                    acc[ks][1] += f * v[ks][1];
                }
                f *= fast_exp2(lt);
            }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) ef[ks] = cat8(to_bf16x4(acc[ks][0]), to_bf16x4(acc[ks][1]));
        }
        float prefix = 0.f;  // log2 decay from the segment's start to the tile's start
        bool dead = false;   // nothing reaches this tile, nor any later one (uniform)
        for (int k0 = 0; tok0 + k0 * kQ < tend && !dead; k0 += kFixBatch) {
            if (k0 > 0) load_dt(k0);
            float cr[kFixBatch];
            int alive = 0;  // tiles of the batch that something reaches
#pragma unroll
            for (int q = 0; q < kFixBatch; ++q) {
                const float inc = prefix + wave_inclusive_scan_f32(dv[q] * Al2);
                cr[q] = tok0 + (k0 + q) * kQ + lane < tend ? fast_exp2(inc) : 0.f;
                if (read_lane_f32(fast_exp2(inc), 0) == 0.f) dead = true;
                if (!dead) alive = q + 1;
                prefix = read_lane_f32(inc, kQ - 1);
            }
#pragma unroll
            for (int q = 0; q < kFixBatch; ++q) {
                if (q >= alive || tok0 + (k0 + q) * kQ >= tend) break;
                const int k = k0 + q;
                if ((k & (nz - 1)) != z) continue;
                if (k != z) load_rows(k, pt, r);
#pragma unroll
                for (int tt = 0; tt < 4; ++tt) {
                    const int tq = tok0 + k * kQ + 16 * tt + lr;  // this lane's token of the query block
                    const float crt = __shfl(cr[q], 16 * tt + lr, 64);
                    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) acc = mfma16(ef[ks], r.c[tt][ks], acc);
                    if (tq < tend && crt != 0.f) {
                        bf16x4 out;
#pragma unroll
                        for (int e = 0; e < 4; ++e) out[e] = (bf16_t)((float)r.y[tt][e] + crt * acc[e]);
                        *y_at(k, tt, pt) = out;
                    }
                }
            }
        }
    }
}

// Workgroups that share the tiles of a (boundary, head): as many as still find a CU to themselves, where the state may
// live through all tiles of a segment (us of a scan whose decays are slow, with 1 / 2 / 4: 24 heads of 64, 1000 tokens,
// 48 pairs 45.8 / 36.6 / 32.2; 2000, 96 pairs 50.5 / 42.2 / 45.4; 4000, 168 pairs 58.7 / 62.1 / 65.1), two where a few
// CUs would have two workgroups and the others wait for them (6000, 264 pairs 87.1 / 71.8 / 84.2), and four where heads of
// more than 64 channels take a wave two turns (30 heads of 128, 4000 tokens, 150 pairs 122 / 125 / 101).  With fast decays the
// shares cost 1 us at most.  The bits are the same.
int fix_shares(int nseg, int H, int P) {
    const long long pairs = (long long)nseg * H;
    return pairs <= 64 ? 4 : pairs <= 128 ? 2 : pairs <= 256 ? (P > 64 ? 4 : 1) : pairs <= 320 ? 2 : 1;
}

template <int NS, int NC, int NH, bool GATHER>
int launch(const SegArgs &a, hipStream_t st) {
    const int nunits = a.nseg * a.wg_per_seg;
    const size_t smem = sizeof(LdsS<NS, NC, NH>);
    if (!allow_dynamic_lds(reinterpret_cast<const void *>(&ssd_seg_kernel<NS, NC, NH, GATHER>), smem)) return STRD_EHIP;
    ssd_seg_kernel<NS, NC, NH, GATHER><<<xcd_grid(nunits), threads_for(NC, NH), smem, st>>>(a, nunits);
    if (a.nseg > 1) ssd_fix_kernel<NS, GATHER><<<dim3(a.nseg, a.H, fix_shares(a.nseg, a.H, a.P)), kFixThreads, 0, st>>>(a);
    return launch_status();
}

// channels per workgroup / 32: the whole head when that divides, else one slab
int slabs_per_wg(int P) { return P % 64 == 0 ? 2 : 1; }
// heads per workgroup: two heads of one group share the B and C tiles when a head is one workgroup's
// worth of channels and the group has an even number of heads
int heads_per_wg(int H, int P, int G) { return P == 64 && (H / G) % 2 == 0 ? 2 : 1; }

}  // namespace

// How the sequence is cut: as many segments as it takes to give every CU a workgroup, each at least
// kMinSegSteps steps long (a shorter segment costs more in its prologue and at its seam than it gains).
void ssd_seg_plan(int T, int H, int P, int G, int *nseg, int *seg_steps) {
    constexpr int kMinSegSteps = 8, kCUs = 256;
    const int nsteps = (T + kQ - 1) / kQ;
    const int wg = H * (P / 32) / slabs_per_wg(P) / heads_per_wg(H, P, G);
    int s = wg >= kCUs ? 1 : (kCUs + wg - 1) / wg;
    s = max(1, min(s, nsteps / kMinSegSteps));
    const int per = (nsteps + s - 1) / s;
    *seg_steps = max(per, 1);
    *nseg = max(1, (nsteps + *seg_steps - 1) / *seg_steps);
}

size_t ssd_seg_ws(int T, int H, int P, int G, int n) {
    int nseg, seg_steps;
    ssd_seg_plan(T, H, P, G, &nseg, &seg_steps);
    if (nseg <= 1) return 0;
    return align_up((size_t)(nseg - 1) * H * P * n * sizeof(float), 256) + align_up((size_t)nseg * H * sizeof(float), 256);
}

// `rows` = number of rows of the source tensors (T for the dense call, N + M for the gather call)
bool ssd_seg_supported(int T, int rows, int H, int P, int G, int n, strd_dtype io) {
    const unsigned long long lim = 1ull << 32, r = (unsigned long long)(rows > T ? rows : T) + 2 * kQ;
    return io == STRD_BF16 && T >= 1 && (n == 64 || n == 128) && P % 32 == 0 && (long long)H * (P / 32) < (1 << 22) &&
           r * H * 4 < lim && H <= 65535;
}

// Whether this kernel or the one that walks the whole sequence in one workgroup per (head, 32
// channels) (ssd_mfma) is taken.  This kernel moves about half the bytes per token through
// a CU's copy path (B and C tiles serve the whole head) and fills the chip with few heads, but pays
// for its segments with a longer prologue and a second launch -- and with a rounding: the carried part of an
// output passes through LDS in bf16 where ssd_mfma adds it in fp32, and a seam corrects outputs that are
// already rounded.  So it is kept to where ssd_mfma is no choice: segments of 32 steps and more, or few heads, when
// that kernel would leave CUs idle.  (In between, 43 to 124 steps of 128 heads, it is further from 64 bits than that kernel's
// walk, 2.348e-3 against 2.346e-3; the segments that ssd_mfma cuts for itself there are nearer, 1.67e-3.)
bool ssd_seg_preferred(int T, int H, int P, int G) {
    int nseg, seg_steps;
    ssd_seg_plan(T, H, P, G, &nseg, &seg_steps);
    return nseg >= 2 && (seg_steps >= 32 || H * (P / 32) < 128);
}

int ssd_seg(const void *x, const float *dt, const float *A, const void *B, const void *C, const float *D,
            const float *S_in, void *y, float *S_out, const int32_t *idx, int N, int K, int T, int H, int P, int G, int n,
            void *ws, hipStream_t st) {
    SegArgs a;
    a.x = (const bf16_t *)x; a.dt = dt; a.A = A; a.B = (const bf16_t *)B; a.C = (const bf16_t *)C; a.D = D; a.S_in = S_in;
    a.y = (bf16_t *)y; a.S_out = S_out; a.idx = idx; a.N = N; a.K = K; a.T = T; a.H = H; a.P = P; a.G = G;
    ssd_seg_plan(T, H, P, G, &a.nseg, &a.seg_steps);
    const int nc = slabs_per_wg(P), nh = heads_per_wg(H, P, G);
    a.wg_per_seg = H * (P / 32) / nc / nh;
    a.lend = a.ltot = nullptr;
    if (a.nseg > 1) {
        if (!ws) return STRD_EWORKSPACE;
        a.lend = (float *)ws;
        a.ltot = (float *)((char *)ws + align_up((size_t)(a.nseg - 1) * H * P * n * sizeof(float), 256));
    }
#define STRD_SEG_LAUNCH(NS_, NC_, NH_)                                                 \
    return idx ? launch<NS_, NC_, NH_, true>(a, st) : launch<NS_, NC_, NH_, false>(a, st)
    if (n == 128 && nc == 2 && nh == 2) { STRD_SEG_LAUNCH(128, 2, 2); }
    if (n == 64 && nc == 2 && nh == 2) { STRD_SEG_LAUNCH(64, 2, 2); }
    if (n == 128 && nc == 2) { STRD_SEG_LAUNCH(128, 2, 1); }
    if (n == 128 && nc == 1) { STRD_SEG_LAUNCH(128, 1, 1); }
    if (n == 64 && nc == 2) { STRD_SEG_LAUNCH(64, 2, 1); }
    if (n == 64 && nc == 1) { STRD_SEG_LAUNCH(64, 1, 1); }
#undef STRD_SEG_LAUNCH
    return STRD_EUNSUPPORTED;
}

}  // namespace strd
