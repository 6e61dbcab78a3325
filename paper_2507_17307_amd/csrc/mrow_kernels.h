// Multi-row kernels (2..128 token rows per call): the catch-up prefill of the
// tokens a model has not seen, and batched decode.  The weights are still read
// once per call, so the phases stay HBM-bound; the contraction over tokens runs
// on the matrix cores (v_mfma_f32_16x16x32_bf16, fp32 accumulate) so that ALU
// work never becomes the limiter.  Activations stay fp32 in memory; the consumer
// splits each value in registers into three bf16 planes (p0 = bf16(x), p1 =
// bf16(x - p0), p2 = x - p0 - p1, which is exact: 3 x 8 significant bits hold the
// 24 of an fp32) and multiplies each weight tile with all three, smallest first,
// so the product is that of the fp32 activation (4 bytes per element through the
// load path instead of the 6 of stored planes).  They lie in the order in which the
// matrix-core operands take them (frag_index), not row by row.
#pragma once

#include "device_utils.h"
#include "gemm_plan.h"
#include "model_kernels.h"

namespace rs {

constexpr int ROWK_THREADS = 1024;     // row norm: one workgroup per token row
constexpr int ROPE_THREADS = 256;      // rotary kernel: several

// x[i] (+ the other split-K partial sums of it): all requests are issued together, unconditionally
// (the split index is clamped, a duplicate is dropped by a select), so a row costs one round trip.
__device__ __forceinline__ float4 sum_splits4(const float *base, size_t i, int ksplit, size_t part_stride, float4 first) {
    float4 v[KSPLIT_MAX];
#pragma unroll
    for (int ks = 1; ks < KSPLIT_MAX; ++ks)
        v[ks] = *reinterpret_cast<const float4 *>(base + (size_t)min(ks, ksplit - 1) * part_stride + i);
#pragma unroll
    for (int ks = 1; ks < KSPLIT_MAX; ++ks)
        if (ks < ksplit) { first.x += v[ks].x; first.y += v[ks].y; first.z += v[ks].z; first.w += v[ks].w; }
    return first;
}

// RMSNorm of whole rows: grid n_out, block ROWK_THREADS; d a multiple of 4, at most 4 * NV * ROWK_THREADS.
// src row = gather ? gather[blockIdx.x] : blockIdx.x; the normalised row goes to out32[blockIdx.x] as fp32 (the
// matrix-core kernels split it into bf16 planes themselves), in operand order (frag_index).
// part != null: the projection before this norm left its result as `ksplit` partial sums
// part[ks][row][d] (split over K across workgroups); they are added to the residual row here, in a
// fixed order, and the row is written back before it is normalised.
// All of a thread's NV quads are requested before the first sum is written back: with a store between them the second quad of a row of 5120
// values was requested a round trip later (kernel times of both builds in turn: width 5120, 61 rows 6.9 -> 6.7 us, 29 rows 6.7 -> 6.4; with one quad the partial
// sums no longer wait for the residual: width 3584, 128 rows 7.2 -> 6.5; three quads, width 12288, 128 rows 14.8 and 15.0, width 8320, 61 rows 9.6 and 9.5).  A row's partial sums, 115 KB of eight splits, come through one CU: that is most of what is left.
template <int NV>
__global__ void __launch_bounds__(ROWK_THREADS)
k_rmsnorm_rows(float *__restrict__ h, const uint16_t *__restrict__ gain, float eps, int d,
               const int *__restrict__ gather, float *__restrict__ out32, int rsh,
               const float *__restrict__ part, int ksplit, size_t part_stride) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int src = gather ? gather[blockIdx.x] : blockIdx.x;
    float *hr = h + (size_t)src * d;
    __shared__ float red_ss[ROWK_THREADS / 64];
    const int n4 = d >> 2;
    float4 v[NV], p[NV][KSPLIT_MAX];
    uint2 gv[NV];
    float ss = 0.f;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int i4 = tid + k * ROWK_THREADS;
        v[k] = make_float4(0.f, 0.f, 0.f, 0.f); gv[k] = make_uint2(0, 0);
        if (i4 < n4) {
            v[k] = *reinterpret_cast<const float4 *>(hr + 4 * i4);
            gv[k] = *reinterpret_cast<const uint2 *>(gain + 4 * i4);
            if (part) {
#pragma unroll
                for (int ks = 0; ks < KSPLIT_MAX; ++ks) p[k][ks] = *reinterpret_cast<const float4 *>(part + (size_t)min(ks, ksplit - 1) * part_stride + (size_t)src * d + 4 * i4);
            }
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int i4 = tid + k * ROWK_THREADS;
        if (part && i4 < n4) {
            float4 t = p[k][0];
#pragma unroll
            for (int ks = 1; ks < KSPLIT_MAX; ++ks)
                if (ks < ksplit) { t.x += p[k][ks].x; t.y += p[k][ks].y; t.z += p[k][ks].z; t.w += p[k][ks].w; }
            v[k].x += t.x; v[k].y += t.y; v[k].z += t.z; v[k].w += t.w;
            *reinterpret_cast<float4 *>(hr + 4 * i4) = v[k];
        }
        ss = fmaf(v[k].x, v[k].x, ss); ss = fmaf(v[k].y, v[k].y, ss); ss = fmaf(v[k].z, v[k].z, ss); ss = fmaf(v[k].w, v[k].w, ss);
    }
    ss = wave_sum(ss);
    if (lane == 0) red_ss[wave] = ss;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < ROWK_THREADS / 64; ++w) tot += red_ss[w];
    const float inv = 1.0f / sqrtf(tot / (float)d + eps);
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int i4 = tid + k * ROWK_THREADS;
        if (i4 >= n4) continue;
        *reinterpret_cast<float4 *>(out32 + frag_index(blockIdx.x, 4 * i4, d, rsh)) = make_float4(v[k].x * (inv * bf16_lo(gv[k].x)), v[k].y * (inv * bf16_hi(gv[k].x)),
                                                             v[k].z * (inv * bf16_lo(gv[k].y)), v[k].w * (inv * bf16_hi(gv[k].y)));
    }
}

// Rotary embedding of q and k, KV-cache write: grid (n_rows, rope_blocks), block ROPE_THREADS; a thread has four consecutive rotary
// pairs or four values of V (head_dim / 2 is a multiple of 4).  A row's partial sums are pulled by several CUs: one workgroup of 1024
// threads per row took 6.4 in place of 5.7 us (7B shape, 128 rows), 6.2 in place of 5.3 (14B, 61).
struct RopeArgs {
    const float *qkv;              // [rows, (n_q+2 n_kv) hd] fp32, or `ksplit` partial sums of it, part_stride elements apart
    int ksplit; size_t part_stride;
    float *qbuf; uint16_t *kcache, *vcache;
    const float *rope_cos, *rope_sin;
    const int *row_pos, *row_slot, *row_bad;
    int n_q, n_kv, head_dim, max_ctx, max_seqs, layer;
};
inline int rope_blocks(int n_q, int n_kv, int hd) { return ((n_q + n_kv) * (hd / 8) + n_kv * (hd / 4) + ROPE_THREADS - 1) / ROPE_THREADS; }

__global__ void __launch_bounds__(ROPE_THREADS) k_rope_kv_rows(RopeArgs a) {
    const int r = blockIdx.x, hd = a.head_dim, half = hd >> 1, quads = half >> 2;
    const int n_rot = (a.n_q + a.n_kv) * quads, p4 = blockIdx.y * ROPE_THREADS + threadIdx.x;
    const int bad = a.row_bad[r], pos = a.row_pos[r], slot = a.row_slot[r];
    const size_t xo = (size_t)r * (a.n_q + 2 * a.n_kv) * hd;
    const int ks_n = a.ksplit > 1 ? a.ksplit : 1;
    if (p4 < n_rot) {
        const int head = p4 / quads, i = (p4 - head * quads) * 4;
        float *q = a.qbuf + ((size_t)r * a.n_q + head) * hd;
        if (bad) {
            if (head < a.n_q) { const float4 z = make_float4(0.f, 0.f, 0.f, 0.f); *reinterpret_cast<float4 *>(q + i) = z; *reinterpret_cast<float4 *>(q + i + half) = z; }
            return;
        }
        const float4 c = *reinterpret_cast<const float4 *>(a.rope_cos + (size_t)pos * half + i), s = *reinterpret_cast<const float4 *>(a.rope_sin + (size_t)pos * half + i);
        const size_t e0 = xo + head * hd + i;
        const float4 x0 = sum_splits4(a.qkv, e0, ks_n, a.part_stride, *reinterpret_cast<const float4 *>(a.qkv + e0));
        const float4 x1 = sum_splits4(a.qkv, e0 + half, ks_n, a.part_stride, *reinterpret_cast<const float4 *>(a.qkv + e0 + half));
        // (which product is rounded by itself is said here: which of two the compiler fuses depends on the order of the loads above, and K is rounded next)
        const float4 y0 = make_float4(fmaf(x0.x, c.x, -(x1.x * s.x)), fmaf(x0.y, c.y, -(x1.y * s.y)), fmaf(x0.z, c.z, -(x1.z * s.z)), fmaf(x0.w, c.w, -(x1.w * s.w)));
        const float4 y1 = make_float4(fmaf(x1.x, c.x, x0.x * s.x), fmaf(x1.y, c.y, x0.y * s.y), fmaf(x1.z, c.z, x0.z * s.z), fmaf(x1.w, c.w, x0.w * s.w));
        if (head < a.n_q) {
            *reinterpret_cast<float4 *>(q + i) = y0; *reinterpret_cast<float4 *>(q + i + half) = y1;
        } else {
            const size_t base = ((((size_t)a.layer * a.max_seqs + slot) * a.n_kv + (head - a.n_q)) * a.max_ctx + pos) * hd;
            *reinterpret_cast<uint2 *>(a.kcache + base + i) = make_uint2(pack_bf16x2(y0.x, y0.y), pack_bf16x2(y0.z, y0.w));
            *reinterpret_cast<uint2 *>(a.kcache + base + i + half) = make_uint2(pack_bf16x2(y1.x, y1.y), pack_bf16x2(y1.z, y1.w));
        }
    } else if (p4 - n_rot < (a.n_kv * hd) >> 2 && !bad) {
        const int p = (p4 - n_rot) * 4, vh = p / hd, e = p - vh * hd;
        const size_t e0 = xo + (a.n_q + a.n_kv) * hd + p;
        const float4 x = sum_splits4(a.qkv, e0, ks_n, a.part_stride, *reinterpret_cast<const float4 *>(a.qkv + e0));
        const size_t base = (((size_t)a.layer * a.max_seqs + slot) * a.n_kv + vh) * (size_t)a.max_ctx * hd;
        uint16_t *vp = a.vcache + base + (size_t)e * a.max_ctx + pos;          // V is stored [hd][position]
        vp[0] = f32_to_bf16(x.x); vp[a.max_ctx] = f32_to_bf16(x.y); vp[2 * (size_t)a.max_ctx] = f32_to_bf16(x.z); vp[3 * (size_t)a.max_ctx] = f32_to_bf16(x.w);
    }
}

// ------------------------------------------------------------------------------------------------
// out[m, n] = sum_k X[m, k] W[n, k] for M <= 16*NB token rows.
// A workgroup of GEMM_NW waves owns R consecutive tiles of 16 output columns (for gate/up a tile is 16
// gate rows plus the 16 matching up rows of W) and ALL of K; wave w takes the k windows w, w+GEMM_NW,
// ... of 64 elements (more waves where a matrix has few tiles, so that enough requests are in flight).  Per window a wave requests
//   * its piece of X once: fp32, 16 tokens x 64 k per 16-token block, four contiguous kilobytes (see frag_index), each lane
//     the values of its place in the B-operand layout of v_mfma_f32_16x16x32_bf16 (lane (i = lane % 16, g = lane / 16)
//     supplies the 8 consecutive k at 32 s + 8 g of token i), split into the three planes in
//     registers; the piece serves all R tiles, so X costs 2/R of the W bytes in L2 traffic (stored
//     planes cost 3/R: a 7B-shape call of 16 rows 4.84 -> 4.4 ms);
//   * the 16 x 64 piece of W of every tile it owns with coalesced 16-byte loads, eight lanes per
//     128-byte row piece (whole cache lines: on this chip 64-byte pieces, which the operand layout
//     would give directly, stream at 4.5 TB/s, 128-byte pieces at 6.2), parked in the wave's private
//     LDS area and read back in the A-operand layout.
// The requests of the next window are in flight while the current one is multiplied.  The per-wave
// 16x16 accumulators (lane holds D[4 g + r][token = lane % 16]) of a group meet in LDS; wave p sums
// and finishes tile-and-token-block pair p.  The launch makes every group resident at once, with the
// groups spread evenly over the CUs, because a CU draws at most ~30 GB/s (see launch_gemm).
// ------------------------------------------------------------------------------------------------
struct GemmArgs {
    const uint16_t *W; int N, K, M;       // M = valid token rows
    int rsh;                              // rows per block of the activation buffers: 1 << rsh (frag_index); 4 for more than 16 rows
    const float *X32;                     // activations: fp32 rows of K in operand order (split into three bf16 planes in registers)
    float *act32;                         // gate/up: SwiGLU output rows of d_ffn, fp32 in operand order
    float *out_f32; int ld_out;           // raw fp32 output [M, ld_out] (QKV)
    int yblocks;                          // > 1: the token rows are cut into yblocks blocks of 16*NB rows, each taken by its own
                                          //      workgroups (same weights; ids arranged so that they meet in one XCD's L2)
    int ksplit; size_t part_stride;       // > 1: K is split over workgroups too; split ks writes its partial sums to
    float *part;                          //      part[ks * part_stride + m * N + n] (QKV, O-proj, down) and the consumer adds them up
    float *h_out; int ld_h;               // residual accumulate
    int d_ffn;
    const float *seq_scale; SoftPartial *parts; float *logits; int n_parts;   // LM head
    int sample_on; unsigned long long sample_key;         // LM head: also track the arg max of logit + Gumbel noise
    const int *row_pos, *out_row;                         // sampling: position of the row that feeds output row m is row_pos[out_row[m]]
};

constexpr int GEMM_PITCH = GEMM_KW * 2 + 16;      // bytes per parked row (padded against LDS bank conflicts)

template <int MODE, int NB, int R, int GEMM_NW>
__host__ __device__ constexpr size_t gemm_lds_bytes() {
    constexpr size_t nt = (MODE == G_GATEUP) ? 2 : 1;
    constexpr size_t park = (size_t)GEMM_NW * R * nt * 16 * GEMM_PITCH, meet = (size_t)GEMM_NW * R * nt * NB * 1024;
    return park > meet ? (park > 2048 ? park : 2048) : (meet > 2048 ? meet : 2048);   // 2 KB: the LM head's state exchange
}

template <int MODE, int NB, int R, int GEMM_NW>
__global__ void __launch_bounds__(GEMM_NW * 64) k_gemm_rows(GemmArgs a) {
    constexpr bool TWO_IN_FLIGHT = NB == 1;                               // larger token blocks have no registers to spare
    constexpr int NT = (MODE == G_GATEUP) ? 2 : 1;
    constexpr int NS = GEMM_KW / 32;
    constexpr int NQ = (16 * GEMM_KW * 2) / 1024;                         // load instructions per 16-row piece (2)
    constexpr int SLOTS = R * NT * NB;
    static_assert(MODE != G_LMHEAD || NB == 1, "the router state of a lane follows one token");
    extern __shared__ __align__(16) unsigned char smem[];
    float4 *red = reinterpret_cast<float4 *>(smem);                       // [GEMM_NW][SLOTS][64], after the last window
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i16 = lane & 15, g = lane >> 4;
    unsigned char *park = smem + (size_t)wave * R * NT * 16 * GEMM_PITCH;   // this wave's [R*NT][16 rows][GEMM_PITCH]
    const int lrow = lane >> 3, lchunk = lane & 7;                        // load role: row 8 q + lrow, bytes 16 lchunk ..
    const int K = a.K;
    const int n_out = (MODE == G_GATEUP) ? a.d_ffn : a.N;                 // distinct output columns
    const int n_tiles = (n_out + 15) / 16, n_groups = (n_tiles + R - 1) / R;
    const int n_win = K / GEMM_KW;
    const int KSP = a.ksplit > 1 ? a.ksplit : 1;

    // Workgroup id -> (work unit, token-row block).  The hardware deals consecutive workgroup ids round
    // robin over the 8 XCDs; the row blocks of one unit stream the same weights, so they get ids that are
    // congruent modulo 8: one of them fetches a weight line from HBM, the others find it in that XCD's L2.
    const int Y = a.yblocks > 1 ? a.yblocks : 1;
    const int n_units = n_groups * KSP;
    int unit_first, unit_step, yb;
    if (Y == 1) { unit_first = blockIdx.x; unit_step = gridDim.x; yb = 0; }
    else {
        // the launch has 8 * Y * n_cs workgroups: column slot cs (of n_cs) on XCD x walks the units cs * 8 + x, + n_cs * 8, ...
        const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
        yb = slot % Y;
        unit_first = (slot / Y) * 8 + xcd;
        unit_step = (int)(gridDim.x / (8 * Y)) * 8;
    }
    const int m_base = yb * 16 * NB;

    // token side: rows past M (inside the padding of the buffer) hold anything; their products fill matrix-core columns
    // that belong to no row and are never stored
    const float *xp[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) xp[nb] = a.X32 + (size_t)(m_base + nb * 16) * K + ((g << a.rsh) + min(i16, (1 << a.rsh) - 1)) * 4;
    SoftState st; st.init();
    const int lm_row = i16;                               // LM head (one block of rows): the output row this lane's state follows
    const float lm_scale = (MODE == G_LMHEAD && lm_row < a.M) ? a.seq_scale[lm_row] : 1.f;
    unsigned long long noise_base = 0;                    // sampling: (position of the token being predicted) * V
    if (MODE == G_LMHEAD && a.sample_on && lm_row < a.M) noise_base = (unsigned long long)(a.row_pos[a.out_row[lm_row]] + 1) * (unsigned long long)a.N;

    for (int unit = unit_first; unit < n_units; unit += unit_step) {
        const int grp = unit / KSP, ksp = unit - grp * KSP;
        const int w_lo = (int)(((long long)n_win * ksp) / KSP), w_hi = (int)(((long long)n_win * (ksp + 1)) / KSP);
        f32x4_t acc[R][NT][NB];
        const uint16_t *wp[R][NT][NQ];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    const int row = min((grp * R + r) * 16 + 8 * q + lrow, n_out - 1) + (nt == 1 ? a.d_ffn : 0);
                    wp[r][nt][q] = a.W + (size_t)row * K + lchunk * 8;
                }
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) acc[r][nt][nb] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
            }
        // two windows in flight per wave: the requests of the next window are issued before the
        // products of the current one.  Requests are unconditional (the window index is clamped;
        // a duplicate is fetched but never multiplied) so that the compiler can count them and wait
        // for exactly the older set.
        auto request = [&](int win, float4 (&xb)[NB][NS][2], uint4 (&wr)[R][NT][NQ]) {
            const int k0 = min(win, w_hi - 1) * GEMM_KW;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    const float *q = xp[nb] + ((size_t)(k0 + 32 * s) << a.rsh);
                    xb[nb][s][0] = *reinterpret_cast<const float4 *>(q); xb[nb][s][1] = *reinterpret_cast<const float4 *>(q + (16 << a.rsh));
                }
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int q = 0; q < NQ; ++q)
                        wr[r][nt][q] = load_stream(reinterpret_cast<const uint4 *>(wp[r][nt][q] + k0));
        };
        auto multiply = [&](const float4 (&xb)[NB][NS][2], const uint4 (&wr)[R][NT][NQ]) {
            // this lane's 8 consecutive k of token i16 per k step, as three bf16 planes whose sum is the fp32 value
            bf16x8_t B[NB][NS][3];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    const float4 x0 = xb[nb][s][0], x1 = xb[nb][s][1];
                    const float xv[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
                    split3(xv, B[nb][s]);
                }
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    unsigned char *pk = park + (size_t)(r * NT + nt) * 16 * GEMM_PITCH;
#pragma unroll
                    for (int q = 0; q < NQ; ++q)
                        *reinterpret_cast<uint4 *>(pk + (size_t)(8 * q + lrow) * GEMM_PITCH + lchunk * 16) = wr[r][nt][q];
                }
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    const unsigned char *pk = park + (size_t)(r * NT + nt) * 16 * GEMM_PITCH;
#pragma unroll
                    for (int s = 0; s < NS; ++s) {
                        const bf16x8_t A = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4 *>(pk + (size_t)i16 * GEMM_PITCH + (4 * s + g) * 16));
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                            for (int pl = 2; pl >= 0; --pl)           // smallest plane first
                                acc[r][nt][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, B[nb][s][pl], acc[r][nt][nb], 0, 0, 0);
                    }
                }
        };
        if constexpr (TWO_IN_FLIGHT) {
            float4 xb0[NB][NS][2], xb1[NB][NS][2];
            uint4 wr0[R][NT][NQ], wr1[R][NT][NQ];
            int win = w_lo + wave;
            if (win < w_hi) {
                request(win, xb0, wr0);
                while (true) {
                    request(win + GEMM_NW, xb1, wr1);
                    multiply(xb0, wr0);
                    win += GEMM_NW;
                    if (win >= w_hi) break;
                    request(win + GEMM_NW, xb0, wr0);
                    multiply(xb1, wr1);
                    win += GEMM_NW;
                    if (win >= w_hi) break;
                }
            }
        } else {
            float4 xb0[NB][NS][2];
            uint4 wr0[R][NT][NQ];
            for (int win = w_lo + wave; win < w_hi; win += GEMM_NW) {
                request(win, xb0, wr0);
                multiply(xb0, wr0);
            }
        }
        __syncthreads();      // every wave is done with its parking area, which the accumulators now overwrite
        // ---- the waves' accumulators meet in LDS
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    red[(wave * SLOTS + (r * NT + nt) * NB + nb) * 64 + lane] =
                        make_float4(acc[r][nt][nb][0], acc[r][nt][nb][1], acc[r][nt][nb][2], acc[r][nt][nb][3]);
        __syncthreads();
        // ---- wave p finishes pair p = (tile r, token block nb): this lane holds output columns
        // n0 + 4 g + rr (rr = 0..3) of token nb*16 + i16
        for (int p = wave; p < R * NB; p += GEMM_NW) {
            const int r = p / NB, nb = p - r * NB;
            const int tile = grp * R + r, n0 = tile * 16, m = m_base + nb * 16 + i16;
            float4 v[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                v[nt] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (int w = 0; w < GEMM_NW; ++w) {
                    const float4 u = red[(w * SLOTS + (r * NT + nt) * NB + nb) * 64 + lane];
                    v[nt].x += u.x; v[nt].y += u.y; v[nt].z += u.z; v[nt].w += u.w;
                }
            }
            if (tile >= n_tiles || m >= a.M) continue;
            if constexpr (MODE != G_LMHEAD) {
                // (n_out is a multiple of 16: whole tiles, one 16-byte store per lane)
                const int n = n0 + 4 * g;
                float *dst;
                if constexpr (MODE == G_GATEUP) {
                    dst = a.act32 + frag_index(m, n, a.d_ffn, a.rsh);
                    v[0].x = v[0].x / (1.0f + expf(-v[0].x)) * v[NT - 1].x; v[0].y = v[0].y / (1.0f + expf(-v[0].y)) * v[NT - 1].y;
                    v[0].z = v[0].z / (1.0f + expf(-v[0].z)) * v[NT - 1].z; v[0].w = v[0].w / (1.0f + expf(-v[0].w)) * v[NT - 1].w;
                } else if (KSP > 1) dst = a.part + ksp * a.part_stride + (size_t)m * n_out + n;
                else if (MODE == G_QKV) dst = a.out_f32 + (size_t)m * a.ld_out + n;
                else {
                    dst = a.h_out + (size_t)m * a.ld_h + n;
                    const float4 h = *reinterpret_cast<const float4 *>(dst);
                    v[0] = make_float4(h.x + v[0].x, h.y + v[0].y, h.z + v[0].z, h.w + v[0].w);
                }
                *reinterpret_cast<float4 *>(dst) = v[0];
            } else {
                const float o0[4] = {v[0].x, v[0].y, v[0].z, v[0].w};
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) {
                    const int n = n0 + 4 * g + rr;
                    if (n >= n_out) continue;
                    const float lg = o0[rr] * lm_scale;
                    st.push(lg, n);
                    if (a.sample_on) st.push_noisy(lg, n, a.sample_key, noise_base);
                    if (a.logits) a.logits[(size_t)m * a.N + n] = lg;
                }
            }
        }
        __syncthreads();      // red[] is reused by the next group
    }
    if (MODE == G_LMHEAD) {
        // merge the four row groups of each wave (lanes 0..15 end up with the state of token i16), then the waves
        for (int o = 32; o >= 16; o >>= 1) {
            SoftState b = shfl_xor_state(st, o);
            if ((lane & o) == 0) st.merge(b); else { b.merge(st); st = b; }
        }
        SoftPartial *sp = reinterpret_cast<SoftPartial *>(smem);          // [GEMM_NW][16]
        if (g == 0) sp[wave * 16 + i16] = to_partial(st);
        __syncthreads();
        if (wave == 0 && g == 0 && lm_row < a.M) {
            SoftState s0 = from_partial(sp[i16]);
            for (int w = 1; w < GEMM_NW; ++w) s0.merge(from_partial(sp[w * 16 + i16]));
            a.parts[(size_t)lm_row * a.n_parts + blockIdx.x] = to_partial(s0);
        }
    }
}

}  // namespace rs
