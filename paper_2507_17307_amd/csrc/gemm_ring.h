// k_gemm_ring: out[m, n] = sum_k X[m, k] W[n, k] for 3 .. 128 token rows, one workgroup per block of output columns and all rows, so
// that W is read from HBM once per call.  The products are those of k_gemm_rows (three exact bf16 planes of X, smallest first).
//
// A workgroup fills a CU: NCW waves multiply (four, or eight), two waves fetch X and two fetch W, window by window (64 elements of K), with
// loads that go straight to LDS.  Before, every wave fetched its share of W and its own X into registers, parked W in LDS and
// multiplied: its requests held up its products, and because loads return in order the wait for a piece of X (L2) was a wait
// for all the W (HBM) requested before it.  Now X and W have rings of their own (XS and WS windows), each filled as far ahead as the
// 160 KB allow; the multiplying waves issue nothing but LDS reads, matrix instructions and the splits of X.
//   W  whole 128-byte row pieces, eight rows a load; lane (row r, piece c) fetches piece c ^ (r % 8), so that the A operands
//      (16 rows, one piece) are read back without bank conflicts although a direct load cannot pad the rows.
//   X  in operand order (frag_index): a window of 16 rows is four contiguous kilobytes, read back as it lies.
//   One barrier a window hands over W of the window and X of the next: the split of X into planes has a whole window's
//   matrix instructions to hide behind, two vector instructions between two of them (a third would cost issue slots).
// Rows: a multiplying wave takes RBW blocks of 16 rows (two above 64 rows, so that a tile of W read from LDS serves 32 rows), or
// up to 32 / 16 rows two / four waves share a block and split the columns (CS).  A wave whose second block lies past the
// call's rows leaves its products out.  Above 64 rows narrow groups (ring_eight_waves) and the LM head have eight waves of one
// block: beside the softmax state the sums of two blocks and 13 tiles do not fit the registers (57 spilled), and twice the
// waves share the softmax of a group.  With two blocks and ten tiles at most a vocabulary of 50257 took two rounds of 8 tiles
// in place of one of 13.
// Columns: CT tiles of 16; for gate/up a tile is 8 gate and the 8 matching up columns, which come closer to equal shares of the
// CUs than 16 + 16 (14B: 247 workgroups of 7 instead of 216 of 4; 32B at 33 .. 64 and from 81 rows on one round of 247 of 14 instead of 432 of 4; at other
// row counts the estimates of 14 and of 7 tie and it takes 494 of 7 in two rounds).
//
// What bounds it: up to 64 rows W, streamed at 5.3 .. 6.1 TB/s; at 128 rows the matrix cores, which run at 1.7 .. 1.8 GHz under this
// load (2330 cycles a window of 120 instructions, 2230 of them matrix-core time: 73 of the 88 us of 7B gate/up on that card, 93 and 102
// on others; where it took 93, activations of zeros, the same instructions at less power, took 80).  Kernel times in decode calls, us, k_gemm_rows or the kernel of 17 rows and more before this one (k_gemm_tile) -> now:
//   7B gate/up (272 MB)   5 / 16 / 24 / 48 / 72 / 128 rows   52 / 53 / 59 / 64 / 80 / 98 -> 46 / 44 / 45 / 50 / 72 / 88
//   14B gate/up (283 MB)  8 / 61 / 128 rows  56 / 85 / 108 -> 47 / 68 / 99
//   32B gate/up (566 MB)  16 / 29 / 61 / 128 rows  110 / 123 / 141 / 220 -> 95 / 104 / 107 / 170 (29 rows of ragged spans on
//                         long contexts 128 -> 112 .. 115)
//   14B, 61 rows  down (142 MB) 41 -> 34, O (52 MB) 21 -> 18;  7B QKV (33 MB) 48 / 128 rows 13.6 / 20.7 -> 13.3 / 20.9
//   LM head of the 7B shape (1090 MB)  5 / 16 / 24 / 65 / 128 sequences  179 / 202 / 213 / 378 / 428 -> 170 / 175 / 193 / 304 / 348
//   LM head of more than 64 sequences, before / two blocks a wave / eight waves: 50257 entries, 65 / 128 sequences, 1.5B width 71 / 80 / 55 and
//   76 / 89 / 65, 7B 127 / 146 / 105 and 147 / 165 / 130, 14B 178 / 196 / 148 and 203 / 222 / 177; 8192 entries, 7B 47 / 43 / 39 and 55 / 52 / 50
//
// Modes: G_GATEUP (SwiGLU epilogue into operand order), G_PART (K split over workgroups, raw partial sums part[ks][row][n] that the next
// kernel adds up in a fixed order), G_LMHEAD (scaled logits feed each row's softmax state, one partial per row and wave column).
#pragma once

#include <type_traits>

#include "device_utils.h"
#include "model_kernels.h"
#include "mrow_kernels.h"

namespace rs {

constexpr int G_PART = 5;
constexpr int RING_LDS = 160 * 1024;                           // of a CU

// LDS of a workgroup with CT column tiles and RB row blocks: XS buffers of X windows, then WS buffers of W windows
constexpr int RING_X = 4096, RING_W = 2048;                   // bytes of a window of one row block / one column tile
// (X two windows ahead where that leaves W three buffers: 100 rows, LM head of 8192 entries 59 -> 50 us, 7B down 55 -> 49; three where it leaves
// that of five tiles three: 1.5B down 65 rows 19.2 -> 18.6, gate/up 128 rows 30.2 -> 29.7)
template <int CT, int RB>
__host__ __device__ constexpr int ring_x_stages() { return RB <= 4 ? 3 : CT > 10 ? 2 : CT > 5 ? 3 : 4; }
template <int CT, int RB>
__host__ __device__ constexpr int ring_w_stages() {
    const int n = (RING_LDS - ring_x_stages<CT, RB>() * RB * RING_X) / (CT * RING_W);
    const int most = 1 + 63 / CT < 8 ? 1 + 63 / CT : 8;       // (the wait counter has six bits)
    return n < most ? n : most;
}
template <int CT, int RB>
__host__ __device__ constexpr int ring_lds_bytes() { return ring_x_stages<CT, RB>() * RB * RING_X + ring_w_stages<CT, RB>() * CT * RING_W; }

template <int N>
__device__ __forceinline__ void wait_loads_const() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
// at most n (uniform, below 64) of the wave's loads still on their way
__device__ __forceinline__ void wait_loads(int n) {
#define RS_W(k) case k: wait_loads_const<k>(); break;
#define RS_W8(k) RS_W(k) RS_W(k + 1) RS_W(k + 2) RS_W(k + 3) RS_W(k + 4) RS_W(k + 5) RS_W(k + 6) RS_W(k + 7)
    switch (n) {
        RS_W8(0) RS_W8(8) RS_W8(16) RS_W8(24) RS_W8(32) RS_W8(40) RS_W8(48) RS_W8(56)
        default: wait_loads_const<0>();
    }
#undef RS_W8
#undef RS_W
}

typedef __attribute__((address_space(3))) unsigned char lds_byte;
typedef __attribute__((address_space(1))) const unsigned char global_byte;

template <int MODE, int CT, int RBW, int CS, int NCW>
__global__ void __launch_bounds__(NCW * 64 + 256, 1) k_gemm_ring(GemmArgs a) {
    constexpr int NS = GEMM_KW / 32;                          // NCW waves multiply, two fetch X, two fetch W
    static_assert(MODE != G_LMHEAD || RBW == 1, "the router state of a lane follows one token");
    constexpr int RBK = NCW / CS, RB = RBK * RBW;             // multiplying waves that differ in their rows; row blocks
    constexpr int XS = ring_x_stages<CT, RB>(), WS = ring_w_stages<CT, RB>(), XB = RB * RING_X, WB = CT * RING_W;
    static_assert(WS >= 3, "W of two windows in flight at least");
    static_assert(ring_lds_bytes<CT, RB>() <= RING_LDS, "fits a CU");
    static_assert((WS - 2) * CT < 64 && (XS - 2) * 2 * RB < 64, "the wait counter has six bits");
    constexpr int CTH = (CT + CS - 1) / CS;                   // column tiles of a wave
    constexpr int NCH = (CTH + 4) / 5, CH = (CTH + NCH - 1) / NCH, NGR = NS * NCH;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, g = lane >> 4;
    const int K = a.K, n_out = (MODE == G_GATEUP) ? a.d_ffn : a.N;
    constexpr int TC = MODE == G_GATEUP ? 8 : 16;             // output columns of a tile (gate/up: 8 gate rows, 8 up rows of W)
    const int n_tiles = (n_out + TC - 1) / TC, n_groups = (n_tiles + CT - 1) / CT;
    // G_PART: grid (splits of K, groups of tiles), so that with eight splits every XCD reads one piece of X; else whole K and
    // a workgroup takes the groups blockIdx.y, + gridDim.y ..
    const int n_win = K / GEMM_KW, ksp = MODE == G_PART ? blockIdx.x : 0;
    const int w_first = MODE == G_PART ? n_win * ksp / a.ksplit : 0;
    const int w_count = MODE == G_PART ? n_win * (ksp + 1) / a.ksplit - w_first : n_win;
    const int nrb = min((a.M + 15) >> 4, RB);

    if (wave >= NCW) {
        // ---------------- fetching waves
        const bool is_x = wave < NCW + 2;
        const int which = wave & 1;
        const unsigned char *src[CT > 2 * RB ? CT : 2 * RB];
        int grp = blockIdx.y, left = 0, buf = 0;
        // (up to 16 rows: one block of 1 << rsh rows, a window of it is 1 << (rsh - 2) kilobytes)
        const int x_kb = RB == 1 ? 1 << (a.rsh - 2) : 4;
        const int n_ld = !is_x ? CT : RB == 1 ? min(max(x_kb - 2 * which, 0), 2) : 2 * nrb, depth = is_x ? XS : WS - 1;
        // X: quarters 2 which, 2 which + 1 of every row block's window; W: eight rows a load, every other eight
        const int lrow = lane >> 3, lchunk = (lane & 7) ^ lrow;
        auto start_unit = [&]() {
            left = w_count;
            if (is_x) {
#pragma unroll
                for (int i = 0; i < 2 * RB; ++i)
                    src[i] = reinterpret_cast<const unsigned char *>(a.X32 + (size_t)min(i >> 1, nrb - 1) * 16 * K + (size_t)w_first * (256 * x_kb) + (2 * which + (i & 1)) * 256 + lane * 4);
            } else {
#pragma unroll
                for (int i = 0; i < CT; ++i) {
                    const int j = 8 * (2 * i + which) + lrow;                 // row of W in the workgroup's tiles
                    const int row = MODE == G_GATEUP ? min(grp * CT * 8 + 8 * i + lrow, n_out - 1) + (which ? a.d_ffn : 0)
                                                     : min(grp * CT * 16 + j, n_out - 1);
                    src[i] = reinterpret_cast<const unsigned char *>(a.W + (size_t)row * K + (size_t)w_first * GEMM_KW + lchunk * 8);
                }
            }
        };
        auto issue = [&]() -> int {
            if (grp >= n_groups) return 0;
            if (is_x) {
                lds_byte *base = (lds_byte *)smem + buf * XB + which * 2048;
#pragma unroll
                for (int i = 0; i < 2 * RB; ++i)
                    if (i < n_ld) { __builtin_amdgcn_global_load_lds((global_byte *)src[i], base + (i >> 1) * RING_X + (i & 1) * 1024, 16, 0, 0); src[i] += 1024 * x_kb; }
                buf = buf + 1 == XS ? 0 : buf + 1;
            } else {
                lds_byte *base = (lds_byte *)smem + XS * XB + buf * WB + which * 1024;
#pragma unroll
                for (int i = 0; i < CT; ++i) { __builtin_amdgcn_global_load_lds((global_byte *)src[i], base + i * RING_W, 16, 0, 2); src[i] += GEMM_KW * 2; }
                buf = buf + 1 == WS ? 0 : buf + 1;
            }
            if (--left == 0) { grp += gridDim.y; if (grp < n_groups) start_unit(); }
            return 1;
        };
        int total = 0;                                        // windows of this workgroup
        for (int g_ = blockIdx.y; g_ < n_groups; g_ += gridDim.y) total += w_count;
        start_unit();
        int issued = 0;
        auto arrived = [&](int window) { wait_loads(max(issued - 1 - window, 0) * n_ld); };       // up to and with this one
        for (int i = 0; i < depth; ++i) issued += issue();
        if (is_x) arrived(0);
        asm volatile("s_barrier" ::: "memory");               // the first window of X is read before the first stage
        for (int s = 0; s < total; ++s) {
            arrived(is_x ? s + 1 : s);
            asm volatile("s_barrier" ::: "memory");           // stage s: W of window s and X of window s + 1 are there; W of s - 1 and X of s are free
            issued += issue();
        }
        asm volatile("s_barrier" ::: "memory");               // the barrier of the multiplying waves behind their last stage
        return;
    }

    // ---------------- multiplying waves
    const int rb0 = wave % RBK, ct0 = (wave / RBK) * CTH;     // row blocks rb0, rb0 + RBK ..; first column tile
    const bool rows = rb0 < nrb;
    // logits of a whole quad of columns in one store (64 bytes of a row in the place of four times 16 dwords)
    const bool wide = MODE == G_LMHEAD && a.logits && (a.N & 3) == 0 && (reinterpret_cast<size_t>(a.logits) & 15) == 0;
    const int a_off[NS] = {i16 * 128 + ((g ^ (i16 & 7)) << 4), i16 * 128 + (((4 + g) ^ (i16 & 7)) << 4)};
    // Up to 16 rows there is room for four sums in the place of one, of every fourth window each: the sums of k_gemm_rows' four waves,
    // in their order, so that it does not matter to a result which of the two kernels a matrix takes.
    constexpr int NA = CS == 4 ? 4 : 1;
    f32x4_t acc[RBW][CTH], part[NA][RBW][CTH];
    SoftState state; state.init();
    float lm_scale = 1.f;
    unsigned long long noise_base = 0;                        // sampling: (position of the token being predicted) * V
    if (MODE == G_LMHEAD && rb0 * 16 + i16 < a.M) {
        lm_scale = a.seq_scale[rb0 * 16 + i16];
        if (a.sample_on) noise_base = (unsigned long long)(a.row_pos[a.out_row[rb0 * 16 + i16]] + 1) * (unsigned long long)a.N;
    }
    // group q of a window: tiles CH (q % NCH) .. of k step q / NCH (a tile past the workgroup's last repeats it; its products are dropped)
    auto read_a = [&](const unsigned char *w, int q, bf16x8_t (&A)[CH]) {
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int t = (q % NCH) * CH + i;
            if (t < CTH) A[i] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4 *>(w + a_off[q / NCH] + (CS == 1 ? t : min(ct0 + t, CT - 1)) * RING_W));
        }
    };
    const int x_off = ((g << a.rsh) + min(i16, (1 << a.rsh) - 1)) * 16, x_step = 64 << a.rsh;      // up to 16 rows
    auto read_x = [&](const unsigned char *x, int s, float4 (&v)[RBW][2]) {
#pragma unroll
        for (int r = 0; r < RBW; ++r)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                v[r][h] = *reinterpret_cast<const float4 *>(x + (RB == 1 ? x_off + (2 * s + h) * x_step : (rb0 + r * RBK) * RING_X + (2 * s + h) * 1024 + lane * 16));
    };
    auto planes = [&](const float4 (&x)[2], bf16x8_t (&B)[3]) {
        const float xv[8] = {x[0].x, x[0].y, x[0].z, x[0].w, x[1].x, x[1].y, x[1].z, x[1].w};
        split3(xv, B);
    };
    bf16x8_t A[2][CH], B[NS][RBW][3];
    float4 x0[RBW][2], x1[RBW][2];
    int xb = 0, wb = 0;
    // a window of a group of tiles, added to sums `which`, for a wave with R row blocks
    auto window = [&](auto blocks, auto which) {
        constexpr int R = decltype(blocks)::value, WHICH = decltype(which)::value;
        const unsigned char *w = smem + XS * XB + wb * WB;
        wb = wb + 1 == WS ? 0 : wb + 1; xb = xb + 1 == XS ? 0 : xb + 1;
        const unsigned char *w_next = smem + XS * XB + wb * WB, *x_next = smem + xb * XB;
#pragma unroll
        for (int q = 0; q < NGR; ++q) {
            __builtin_amdgcn_sched_barrier(0);
            if (q + 1 < NGR) read_a(w, q + 1, A[(q + 1) & 1]);
            else {
                if (NCH == 1) read_x(x_next, 1, x1);
                lds_barrier();
                read_a(w_next, 0, A[0]);
            }
            if (q == NCH - 1) read_x(x_next, 0, x0);
            if (NCH > 1 && q == NGR - 2) read_x(x_next, 1, x1);
#pragma unroll
            for (int pl = 2; pl >= 0; --pl)
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int i = 0; i < CH; ++i) {
                        const int t = (q % NCH) * CH + i;
                        if (t < CTH) part[WHICH][r][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[q & 1][i], B[q / NCH][r][pl], part[WHICH][r][t], 0, 0, 0);
                    }
            // the planes of the next k step, spread over the groups of this one
            bool split = false;
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (r * NCH / R == q % NCH) {
                    if (q < NCH) planes(x1[r], B[1][r]); else planes(x0[r], B[0][r]);
                    split = true;
                }
            if (split) {
#pragma unroll
                for (int i = 0; i < 3 * R * CH; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
                }
            }
        }
    };
    auto walk = [&](auto blocks) {
        if constexpr (NA == 1) {
            for (int st = 0; st < w_count; ++st) window(blocks, std::integral_constant<int, 0>{});
        } else {
            for (int st = 0; st < w_count; st += 4) {
                window(blocks, std::integral_constant<int, 0>{});
                if (st + 1 < w_count) window(blocks, std::integral_constant<int, 1>{});
                if (st + 2 < w_count) window(blocks, std::integral_constant<int, 2>{});
                if (st + 3 < w_count) window(blocks, std::integral_constant<int, 3>{});
            }
        }
    };
    lds_barrier();
    if (rows) { read_x(smem, 0, x0); read_x(smem, 1, x1); }
    lds_barrier();
    if (rows) {
        read_a(smem + XS * XB, 0, A[0]);
#pragma unroll
        for (int r = 0; r < RBW; ++r) planes(x0[r], B[0][r]);
    }
    for (int grp = blockIdx.y; grp < n_groups; grp += gridDim.y) {
#pragma unroll
        for (int n = 0; n < NA; ++n)
#pragma unroll
            for (int r = 0; r < RBW; ++r)
#pragma unroll
                for (int t = 0; t < CTH; ++t) part[n][r][t] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
        if (!rows) {
            for (int st = 0; st < w_count; ++st) lds_barrier();
            continue;
        }
        if (RBW == 1 || rb0 + RBK < nrb) walk(std::integral_constant<int, RBW>{}); else walk(std::integral_constant<int, 1>{});
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < RBW; ++r)
#pragma unroll
            for (int t = 0; t < CTH; ++t) acc[r][t] = NA == 4 ? ((part[0][r][t] + part[NA / 4][r][t]) + part[NA / 2][r][t]) + part[NA - 1][r][t] : part[0][r][t];
        // ---- epilogue: this lane holds output columns 16 tile + 4 g + e of token 16 rb + i16
#pragma unroll
        for (int r = 0; r < RBW; ++r) {
            const int m = (rb0 + r * RBK) * 16 + i16;
            if (MODE == G_LMHEAD) {
                // (lanes past the call's rows follow along; their state and logits are not stored)
#pragma unroll
                for (int c = 0; c < CTH; ++c) {
                    const int n0 = (grp * CT + ct0 + c) * 16, n = n0 + 4 * g;
                    if (ct0 + c >= CT || n0 >= n_out) continue;
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = acc[r][c][e] * lm_scale;
                    const int idx[4] = {n, n + 1, n + 2, n + 3};
                    if (n0 + 16 <= n_out) state.push4(v, idx, {true, true, true, true});
                    else state.push4(v, idx, {n < n_out, n + 1 < n_out, n + 2 < n_out, n + 3 < n_out});
                    if (m >= a.M || (!a.sample_on && !a.logits)) continue;
                    if (wide && n < n_out) *reinterpret_cast<float4 *>(a.logits + (size_t)m * a.N + n) = make_float4(v[0], v[1], v[2], v[3]);
                    if (!a.sample_on && wide) continue;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (n + e >= n_out) continue;
                        if (a.sample_on) state.push_noisy(v[e], n + e, a.sample_key, noise_base);
                        if (a.logits && !wide) a.logits[(size_t)m * a.N + n + e] = v[e];
                    }
                }
                continue;
            }
            if (MODE == G_GATEUP) {
                // gate columns lie in the lanes below 32, the matching up columns in those above: two tiles trade halves, so that
                // the lanes below 32 finish the first and the others the second
#pragma unroll
                for (int c = 0; c < CTH; c += 2) {
                    f32x4_t gate = acc[r][c], up = c + 1 < CTH ? acc[r][c + 1] : acc[r][c];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(gate[e]), __float_as_uint(up[e]), false, false);
                        gate[e] = __uint_as_float(t[0]); up[e] = __uint_as_float(t[1]);
                    }
                    const int ct = c + (g >> 1), tile = grp * CT + ct0 + ct;
                    if (m >= a.M || ct >= CTH || ct0 + ct >= CT || tile >= n_tiles) continue;
                    float o[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = gate[e] / (1.0f + expf(-gate[e])) * up[e];
                    *reinterpret_cast<float4 *>(a.act32 + frag_index(m, tile * 8 + 4 * (g & 1), a.d_ffn, RB == 1 ? a.rsh : 4)) = make_float4(o[0], o[1], o[2], o[3]);
                }
                continue;
            }
            if (m >= a.M) continue;
#pragma unroll
            for (int c = 0; c < CTH; ++c) {
                const int tile = grp * CT + ct0 + c;
                if (ct0 + c >= CT || tile >= n_tiles) continue;
                *reinterpret_cast<float4 *>(a.part + ksp * a.part_stride + (size_t)m * n_out + tile * 16 + 4 * g) =
                    make_float4(acc[r][c][0], acc[r][c][1], acc[r][c][2], acc[r][c][3]);      // (n_out is a multiple of 16: whole tiles)
            }
        }
    }
    if (MODE == G_LMHEAD && rows) {
        const int m = rb0 * 16 + i16;
        for (int o = 32; o >= 16; o >>= 1) {
            SoftState b = shfl_xor_state(state, o);
            if ((lane & o) == 0) state.merge(b); else { b.merge(state); state = b; }
        }
        if (g == 0 && m < a.M) a.parts[(size_t)m * a.n_parts + blockIdx.y * CS + wave / RBK] = to_partial(state);
    }
}

}  // namespace rs
