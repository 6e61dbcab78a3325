// Decode-step kernels: row table + embedding, bandwidth-bound GEMV phases with
// fused prologues/epilogues for one token row, split-context GQA decode
// attention on the matrix cores (a partial kernel for one row, one for spans of
// rows, and the merge of the slices).  Wave64, 256-thread workgroups.
#pragma once

#include "attn_plan.h"
#include "device_utils.h"
#include "router.h"

#include <limits.h>

namespace rs {

// ------------------------------------------------------------------------------------------------
// Row table.  One block per token row.  Turns the caller's per-sequence arrays into per-row
// (slot, position, token, bad) entries, validates everything that lives in device memory, and
// gathers the embedding row into the fp32 residual stream.
//   decode:  n_seqs rows, row b = sequence b (span_off == nullptr)
//   catchup: n_rows rows; row r belongs to the sequence b with off[b] <= r < off[b+1]
// ------------------------------------------------------------------------------------------------
struct PrepArgs {
    int n_seqs, n_rows, d_model, vocab, max_ctx, max_seqs;
    const int *seq_slot, *tokens, *span_off, *pos0;
    const float *scale;
    const uint16_t *embed;
    int *row_slot, *row_pos, *row_bad, *out_row, *seq_bad;
    int4 *seq_info;                // per sequence {first row, end row, cache slot, first row's position}; first row = -1 for an invalid one
    float *seq_scale;
    // walked attention (attn_plan.h); all null or zero in calls that do not take it
    int *slice_len;                // [0] positions per context slice of this call, [1] list: slices of the longest context
    int slices;                    // fixed split: slices that divide the longest context of the call
    int4 *pieces;                  // list: two entries per piece, {first row, end row, cache slot, first row's position} of its sequence
                                   // (first row < 0: no piece) and {group of row slots, slice, positions per slice, slices of the longest context}
    int n_pieces, list_slots, list_slices, slot_rows;      // entries, see WalkPlan; rows per row slot
    float *h;
};

constexpr int MAX_SEQS = 128;     // sequences one call may carry
constexpr int MAX_ROWS = 128;     // token rows one call may carry
constexpr int PREP_LDS_INTS = 8 + 5 * MAX_SEQS;

// The call's control values in LDS (sh: PREP_LDS_INTS ints, the first four left free).  They may live in pinned host memory,
// where every dependent read costs a bus round trip: each one is requested by its own thread, all at once,
// and the validation then runs out of LDS.
struct PrepTable { int *off, *slot, *pos, *tok; float *scale; int ns, nr; };       // off: [MAX_SEQS + 1], the others [MAX_SEQS]
__device__ __forceinline__ PrepTable prepare_table(const PrepArgs &a, int *sh) {
    static_assert(MAX_ROWS <= MAX_SEQS && 2 * MAX_SEQS <= 256, "one thread per control value");
    const int tid = threadIdx.x;
    const PrepTable t{sh + 4, sh + 8 + MAX_SEQS, sh + 8 + 2 * MAX_SEQS, sh + 8 + 4 * MAX_SEQS, reinterpret_cast<float *>(sh + 8 + 3 * MAX_SEQS),
                      min(a.n_seqs, MAX_SEQS), min(a.n_rows, MAX_ROWS)};            // the host enforces both bounds
    if (a.span_off != nullptr && tid <= t.ns) t.off[tid] = a.span_off[tid];
    if (tid < t.nr) t.tok[tid] = a.tokens[tid];
    if (tid >= 128 && tid < 128 + t.ns) {
        const int i = tid - 128;
        t.slot[i] = a.seq_slot[i]; t.pos[i] = a.pos0[i]; t.scale[i] = a.scale ? a.scale[i] : 1.f;
    }
    __syncthreads();
    return t;
}

// sh: PREP_LDS_INTS ints of LDS
__device__ __forceinline__ void prepare_row(const PrepArgs &a, int r, int *sh) {
    const int tid = threadIdx.x;
    const PrepTable tb = prepare_table(a, sh);
    int *s_off = tb.off, *s_slot = tb.slot, *s_pos = tb.pos, *s_tok = tb.tok;
    float *s_scale = tb.scale;
    const int ns = tb.ns;
    // Every check is one comparison per thread (one thread walking the table of 128 sequences took 18 us):
    // first the span table, then the row's own sequence.  sh[0]: this row's sequence; sh[1]: longest context of the call
    int lo = r, hi = r + 1, bad = 0;
    if (tid == 0) { sh[0] = a.span_off == nullptr ? r : INT_MAX; sh[1] = 1; }
    __syncthreads();
    if (tid < ns) {
        int len = 1;
        if (a.span_off != nullptr) {
            const int o0 = s_off[tid], o1 = s_off[tid + 1];
            if (o1 <= o0 || o0 < 0 || o1 > a.n_rows) bad = 1;            // empty or malformed span
            if (r >= o0 && r < o1) atomicMin(&sh[0], tid);
            len = o1 - o0;
        }
        if (r == 0 && len > 0 && len <= a.n_rows && s_pos[tid] >= 0 && s_pos[tid] <= a.max_ctx - len) atomicMax(&sh[1], s_pos[tid] + len);
    }
    if (tid == 0 && a.span_off != nullptr && (s_off[0] != 0 || s_off[ns] != a.n_rows)) bad = 1;
    bad = __syncthreads_or(bad);
    const bool table_bad = bad;
    int b = sh[0];
    const int top = sh[1];
    if (b == INT_MAX) { b = -1; bad = 1; lo = 0; hi = 0; }
    else if (a.span_off != nullptr) { lo = s_off[b]; hi = s_off[b + 1]; }
    int bad2 = 0;
    if (!bad) {
        const int slot = s_slot[b], p0 = s_pos[b];
        if (slot < 0 || slot >= a.max_seqs || p0 < 0 || p0 > a.max_ctx - (hi - lo)) bad2 = 1;
        if (tid < ns && tid != b && s_slot[tid] == slot) bad2 = 1;       // slots must be distinct
        if (tid >= lo && tid < hi && (s_tok[tid] < 0 || s_tok[tid] >= a.vocab)) bad2 = 1;
    }
    bad |= __syncthreads_or(bad2);
    if (tid == 0) {
        a.row_bad[r] = bad;
        a.row_slot[r] = bad ? 0 : s_slot[b];
        a.row_pos[r] = bad ? 0 : s_pos[b] + (r - lo);
        if (b >= 0 && r == hi - 1 && b < ns) {
            a.out_row[b] = r; a.seq_bad[b] = bad;
            a.seq_scale[b] = s_scale[b];
            a.seq_info[b] = bad ? make_int4(-1, 0, 0, 0) : make_int4(lo, hi, s_slot[b], s_pos[b]);
        }
        if (r == 0 && a.slices > 0) *a.slice_len = attn_slice_len(top, a.slices);
        // a malformed offset table can leave sequences without any row: flag them all (and only then: the rows of the other
        // sequences write these entries too)
        if (table_bad && r == 0)
            for (int i = 0; i < ns; ++i) { a.seq_bad[i] = 1; a.out_row[i] = 0; a.seq_scale[i] = 1.f; a.seq_info[i] = make_int4(-1, 0, 0, 0); }
    }
    // (d_model is a multiple of 128: four values per thread and round)
    float4 *h = reinterpret_cast<float4 *>(a.h + (size_t)r * a.d_model);
    if (bad) { for (int i = tid; i < (a.d_model >> 2); i += 256) h[i] = make_float4(0.f, 0.f, 0.f, 0.f); return; }
    const uint2 *e = reinterpret_cast<const uint2 *>(a.embed + (size_t)s_tok[r] * a.d_model);
    for (int i = tid; i < (a.d_model >> 2); i += 256) {
        const uint2 v = e[i];
        h[i] = make_float4(bf16_lo(v.x), bf16_hi(v.x), bf16_lo(v.y), bf16_hi(v.y));
    }
}

// The pieces of the walked attention of this call (attn_plan.h), by one workgroup beside those of the rows.  Every sequence of
// a well-formed table whose slot and positions are in range has pieces, also where its rows turn out invalid for another reason
// (token, slot named twice): what such pieces read is in range, and the merge clears the rows' outputs.
// It has to end before the rows' workgroups do, which wait for their embedding rows (5 us a call): one thread per row, which is
// a group's if it is the first row of one, each wave tries slice lengths of its own, no loops over the sequences.
// sh: PREP_LDS_INTS ints of LDS.
__device__ __forceinline__ void prepare_pieces(const PrepArgs &a, int *sh) {
    static_assert(WALK_GROUPS_MAX == MAX_ROWS && MAX_ROWS == 2 * RS_WAVE, "one thread per row, two waves of them");
    __shared__ int g_seq[MAX_ROWS], g_passes[MAX_ROWS], g_end[MAX_ROWS], tried[WALK_TRIES];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, group_rows = 4 * a.slot_rows;
    if (tid < MAX_ROWS) g_seq[tid] = -1;
    const PrepTable tb = prepare_table(a, sh);
    int lo = tid, hi = tid + 1, bad = 0;
    if (tid < tb.ns && a.span_off) {
        lo = tb.off[tid]; hi = tb.off[tid + 1];
        bad = hi <= lo || lo < 0 || hi > a.n_rows || (tid == 0 && (lo != 0 || tb.off[tb.ns] != a.n_rows));
    }
    const bool table_bad = __syncthreads_or(bad);
    if (tid < tb.ns && !table_bad) {
        const int slot = tb.slot[tid], p0 = tb.pos[tid];
        if (slot >= 0 && slot < a.max_seqs && p0 >= 0 && p0 <= a.max_ctx - (hi - lo))
            for (int r = lo; r < hi; r += group_rows) g_seq[r] = tid;
    }
    __syncthreads();
    // thread r: the passes over the longest context of the group that starts at row r
    int passes = 0;
    if (tid < MAX_ROWS) {
        const int seq = g_seq[tid];
        if (seq >= 0) {
            const int first_row = a.span_off ? tb.off[seq] : seq, end_row = a.span_off ? tb.off[seq + 1] : seq + 1;
            passes = (tb.pos[seq] + min(tid + group_rows, end_row) - first_row + ATT_BT - 1) / ATT_BT;
        }
        g_passes[tid] = passes;
    }
    __syncthreads();
    const int p0 = g_passes[lane], p1 = g_passes[64 + lane];
    // (a row's passes stay below 2^20: its K rows fit 31 bits)
    const int longest = (int)wave_max((float)max(p0, p1));
    const int first = walk_first_len(wave_sum_i32(p0 + p1), longest, a.list_slots, a.list_slices);
    for (int k = wave; k < WALK_TRIES; k += 4) {
        const int len = walk_try_len(first, k), n = wave_sum_i32((p0 + len - 1) / len + (p1 + len - 1) / len);
        if (lane == 0) tried[k] = n;
    }
    __syncthreads();
    int len = first;
    for (int k = WALK_TRIES - 1; k >= 0; --k)
        if (tried[k] <= a.list_slots) len = walk_try_len(first, k);
    // place of the group's first piece: the pieces of the groups before it
    const int n_own = (passes + len - 1) / len;
    int end = n_own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) { const int u = __shfl_up(end, o, RS_WAVE); if (lane >= o) end += u; }
    if (tid < MAX_ROWS) g_end[tid] = end;
    __syncthreads();
    const int half = g_end[63], n_all = half + g_end[127], most = (longest + len - 1) / len;
    // the entries: 256 threads over the rows, a power of two each
    int per = 256 / MAX_ROWS;
    while (2 * per * tb.nr <= 256) per *= 2;
    const int r = tid / per;
    if (r < tb.nr && g_seq[r] >= 0) {
        const int seq = g_seq[r], n = (g_passes[r] + len - 1) / len, at = g_end[r] + (r >= 64 ? half : 0) - n;
        const int4 of = a.span_off ? make_int4(tb.off[seq], tb.off[seq + 1], tb.slot[seq], tb.pos[seq]) : make_int4(seq, seq + 1, tb.slot[seq], tb.pos[seq]);
        for (int s = tid % per; s < n; s += per) {
            const int i = min(at + s, a.n_pieces - 1);                             // (there are at most slots + groups: see attn_plan.h)
            a.pieces[2 * i] = of;
            a.pieces[2 * i + 1] = make_int4((r - of.x) / group_rows, s, len * ATT_BT, most);
        }
    }
    for (int i = n_all + tid; i < a.n_pieces; i += 256) a.pieces[2 * i] = make_int4(-1, 0, 0, 0);
    if (tid == 0) { a.slice_len[0] = len * ATT_BT; a.slice_len[1] = most; }
}

// grid n_rows, LIST: and one more workgroup for the list of attention pieces
template <bool LIST>
__global__ void __launch_bounds__(256) k_prepare(PrepArgs a) {
    __shared__ int sh[PREP_LDS_INTS];
    if (LIST && (int)blockIdx.x == a.n_rows) prepare_pieces(a, sh);
    else prepare_row(a, blockIdx.x, sh);
}

// ------------------------------------------------------------------------------------------------
// GEMV phases for 1..8 token rows.  y[m][n] = sum_k W[n,k] x[m][k]: W is bf16, row-major, streamed
// once from HBM with 16-byte non-temporal loads whatever the number of rows; x is fp32 and staged in
// LDS; accumulation is fp32.  A wave owns RT rows of W at a time and its lanes stride over K
// (KS = 1); with KS = 4 the four waves of a workgroup split K of the same rows (short, wide
// matrices).  MP is the number of token rows the kernel is compiled for (1, 2, 4, 8); a call with
// fewer rows leaves the spare ones zero.  When MP * K floats exceed the LDS segment the workgroup
// walks K in segments, restaging x (KS = 4 only).
// Prologue and epilogue depend on the phase:
//   G_QKV     x = RMSNorm(h);  rows come in rotary pairs (i, i + hd/2); epilogue rotates q and k,
//             writes q (fp32) and the bf16 K/V rows of each token's position into the cache
//   G_OPROJ   x = attention output;  h += y
//   G_GATEUP  x = RMSNorm(h);  rows come in (gate i, up i) pairs; act[i] = silu(gate) * up
//   G_DOWN    x = act;  h += y
//   G_LMHEAD  x = RMSNorm(h[gather]);  logit = y * scale feeds the single-pass softmax state of
//             the wave; the workgroup's four states are merged into one partial per token row
// ------------------------------------------------------------------------------------------------
enum { G_QKV = 0, G_OPROJ = 1, G_GATEUP = 2, G_DOWN = 3, G_LMHEAD = 4 };

constexpr int GEMV_LDS_FLOATS = 38912;   // fp32 elements of x held in LDS at a time (152 KB of the CU's 160 KB)

struct GemvArgs {
    const uint16_t *W; int N, K;
    int m_rows;                                           // token rows in this call (<= MP)
    const float *h_in; int ld_h; const uint16_t *gain; float eps;   // RMSNorm input rows (norm phases), row stride ld_h
    const int *gather;                                    // LM head: h row of output row m, or null (= m)
    const float *x_in;                                    // ready fp32 rows [m][K] (other phases)
    float *h_out;                                         // residual stream rows, stride ld_h (O-proj, down)
    float *act;                                           // SwiGLU output rows [m][d_ffn] (gate/up)
    float *qbuf; uint16_t *kcache, *vcache;               // QKV outputs (q rows [m][n_q*hd])
    const float *rope_cos, *rope_sin;                     // [max_ctx, head_dim/2]
    int n_q, n_kv, head_dim, max_ctx, max_seqs, layer, d_ffn;
    const int *row_pos, *row_slot, *row_bad;
    const float *seq_scale; SoftPartial *parts; int n_parts; float *logits;   // LM head
    int sample_on; unsigned long long sample_key;         // LM head: also track the arg max of logit + Gumbel noise (needs row_pos)
};

// elements of K one LDS segment holds for MP rows
template <int MP>
__host__ __device__ constexpr int gemv_seg(int K) { return K * MP <= GEMV_LDS_FLOATS ? K : (GEMV_LDS_FLOATS / MP) / 2048 * 2048; }
template <int MP>
__host__ __device__ constexpr size_t gemv_lds_bytes(int K) { return (size_t)gemv_seg<MP>(K) * MP * 4 + 4096; }

template <int MODE, int RT, int KS, int UNR, int MP, int PRE = 0>
__device__ __forceinline__ void gemv_phase(const GemvArgs &a, unsigned char *smem, int wg, int nwg) {
    static_assert(PRE == 0 || MP == 1, "the early weight request exists for single-row calls only");
    float4 *xs = reinterpret_cast<float4 *>(smem);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int K = a.K, M = a.m_rows;
    const int seg = gemv_seg<MP>(K);                      // elements of K per LDS segment
    const int plane_len = seg >> 3;                       // float4 per plane; row m uses planes 2m and 2m+1
    float *red = reinterpret_cast<float *>(smem + (size_t)seg * MP * 4);   // [2][4][RT*MP]
    float *red_ss = red + 2 * 4 * RT * MP;                                  // [4][MP]
    const bool resident = KS != 4 || seg == K;            // only the split-K launch may walk K in segments (the host checks)
    constexpr bool NORM = (MODE == G_QKV || MODE == G_GATEUP || MODE == G_LMHEAD);

    // ---- tiles
    constexpr int P = RT / 2;
    const int half = a.head_dim >> 1;
    int n_tiles, n_rot_tiles = 0;
    if (MODE == G_QKV) {
        n_rot_tiles = (a.n_q + a.n_kv) * (half / P);
        n_tiles = n_rot_tiles + (a.n_kv * a.head_dim) / RT;
    } else if (MODE == G_GATEUP) {
        n_tiles = a.d_ffn / P;
    } else {
        n_tiles = (a.N + RT - 1) / RT;
    }
    // each workgroup owns a contiguous range of tiles (a contiguous stretch of W); with KS == 1 its
    // four waves interleave inside that range
    // n_tiles * nwg stays far below 2^31 (at most ~2e4 tiles, a few thousand workgroups)
    const int t_lo = (int)(((unsigned)n_tiles * (unsigned)wg) / (unsigned)nwg), t_hi = (int)(((unsigned)n_tiles * (unsigned)(wg + 1)) / (unsigned)nwg);
    const int unit0 = (KS == 1) ? t_lo + wave : t_lo;
    const int ustride = (KS == 1) ? 4 : 1;
    const int c0 = (KS == 1) ? lane : wave * 64 + lane;
    const int cstride = 64 * KS;

    auto tile_rows = [&](int t, int (&rows)[RT], int &head, int &pair0, bool &rot) {
        head = 0; pair0 = 0; rot = false;
        if (MODE == G_QKV) {
            if (t < n_rot_tiles) {
                rot = true; head = t / (half / P); pair0 = (t % (half / P)) * P;
#pragma unroll
                for (int j = 0; j < P; ++j) { rows[2 * j] = head * a.head_dim + pair0 + j; rows[2 * j + 1] = rows[2 * j] + half; }
            } else {
#pragma unroll
                for (int j = 0; j < RT; ++j) rows[j] = (a.n_q + a.n_kv) * a.head_dim + (t - n_rot_tiles) * RT + j;
            }
        } else if (MODE == G_GATEUP) {
#pragma unroll
            for (int j = 0; j < P; ++j) { rows[2 * j] = t * P + j; rows[2 * j + 1] = a.d_ffn + t * P + j; }
        } else {
#pragma unroll
            for (int j = 0; j < RT; ++j) rows[j] = min(t * RT + j, a.N - 1);
        }
    };

    // PRE > 0: the first PRE chunks of this wave's first tile are requested before the prologue
    // touches x, so the weight stream's first round trip overlaps the prologue's instead of
    // following it.  It costs PRE * RT * 4 registers, so it is compiled in only where the sweep
    // showed a gain.  Chunk indices are clamped, not guarded; a clamped chunk is cancelled later by
    // zeroing its x operand.
    uint4 pre[PRE > 0 ? PRE : 1][RT];
    const bool have0 = PRE > 0 && resident && unit0 < t_hi;
    if (have0) {
        int rows0[RT], head0, pair00; bool rot0;
        tile_rows(unit0, rows0, head0, pair00, rot0);
#pragma unroll
        for (int u = 0; u < PRE; ++u) {
            const int c = min(c0 + u * cstride, (K >> 3) - 1);
#pragma unroll
            for (int r = 0; r < RT; ++r) pre[u][r] = load_stream(reinterpret_cast<const uint4 *>(a.W + (size_t)rows0[r] * K) + c);
        }
    }

    // row position / slot (QKV only), read once up front so that no epilogue waits on it
    int row_bad[MP], row_pos[MP], row_slot[MP];
#pragma unroll
    for (int m = 0; m < MP; ++m) {
        row_bad[m] = 1; row_pos[m] = 0; row_slot[m] = 0;
        if (MODE == G_QKV && m < M) { row_bad[m] = a.row_bad[m]; row_pos[m] = a.row_pos[m]; row_slot[m] = a.row_slot[m]; }
    }

    // ---- prologue: x (fp32) into LDS.  Norm phases: K = d_model fits one segment for every MP.
    float inv[MP];
    constexpr int HCACHE = (MP == 1) ? 6 : 0;            // float4 per thread kept between the two passes over h
    float4 hreg[HCACHE > 0 ? HCACHE : 1];
    uint2 greg[HCACHE > 0 ? HCACHE : 1];
    if (NORM) {
        const uint2 *g2 = reinterpret_cast<const uint2 *>(a.gain);
#pragma unroll
        for (int m = 0; m < MP; ++m) {
            float ss = 0.f;
            if (m < M) {
                const int src = (MODE == G_LMHEAD && a.gather) ? a.gather[m] : m;
                const float4 *h4 = reinterpret_cast<const float4 *>(a.h_in + (size_t)src * a.ld_h);
                if (HCACHE > 0) {
#pragma unroll
                    for (int j = 0; j < HCACHE; ++j) {
                        const int i = tid + j * 256;
                        hreg[j] = make_float4(0.f, 0.f, 0.f, 0.f); greg[j] = make_uint2(0, 0);
                        if (i < (K >> 2)) { hreg[j] = h4[i]; greg[j] = g2[i]; }
                    }
#pragma unroll
                    for (int j = 0; j < HCACHE; ++j) {
                        ss = fmaf(hreg[j].x, hreg[j].x, ss); ss = fmaf(hreg[j].y, hreg[j].y, ss);
                        ss = fmaf(hreg[j].z, hreg[j].z, ss); ss = fmaf(hreg[j].w, hreg[j].w, ss);
                    }
                }
                for (int i = tid + HCACHE * 256; i < (K >> 2); i += 256) {
                    const float4 v = h4[i];
                    ss = fmaf(v.x, v.x, ss); ss = fmaf(v.y, v.y, ss); ss = fmaf(v.z, v.z, ss); ss = fmaf(v.w, v.w, ss);
                }
            }
            ss = wave_sum(ss);
            if (lane == 0) red_ss[wave * MP + m] = ss;
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < MP; ++m)
            inv[m] = 1.0f / sqrtf((red_ss[0 * MP + m] + red_ss[1 * MP + m] + red_ss[2 * MP + m] + red_ss[3 * MP + m]) / (float)K + a.eps);
    }
    // stage the K-range [k0, k0+len) of every row: float4 index i covers elements 4i..4i+3; even i -> plane A, odd i -> plane B
    auto stage = [&](int k0, int len) {
#pragma unroll
        for (int m = 0; m < MP; ++m) {
            float4 *xm = xs + (size_t)2 * m * plane_len;
            if (m >= M) {
                for (int i = tid; i < (len >> 2); i += 256) xm[(i & 1) * plane_len + (i >> 1)] = make_float4(0.f, 0.f, 0.f, 0.f);
            } else if (NORM) {
                const int src = (MODE == G_LMHEAD && a.gather) ? a.gather[m] : m;
                const float4 *h4 = reinterpret_cast<const float4 *>(a.h_in + (size_t)src * a.ld_h + k0);
                const uint2 *g2 = reinterpret_cast<const uint2 *>(a.gain + k0);
                const float iv = inv[m];
                if (HCACHE > 0) {
#pragma unroll
                    for (int j = 0; j < HCACHE; ++j) {
                        const int i = tid + j * 256;
                        if (i < (len >> 2)) {
                            float4 v = hreg[j]; const uint2 g = greg[j];
                            v.x *= iv * bf16_lo(g.x); v.y *= iv * bf16_hi(g.x); v.z *= iv * bf16_lo(g.y); v.w *= iv * bf16_hi(g.y);
                            xm[(i & 1) * plane_len + (i >> 1)] = v;
                        }
                    }
                }
                for (int i = tid + HCACHE * 256; i < (len >> 2); i += 256) {
                    float4 v = h4[i]; const uint2 g = g2[i];
                    v.x *= iv * bf16_lo(g.x); v.y *= iv * bf16_hi(g.x); v.z *= iv * bf16_lo(g.y); v.w *= iv * bf16_hi(g.y);
                    xm[(i & 1) * plane_len + (i >> 1)] = v;
                }
            } else {
                // batches of SB loads per thread, all requested before the first is stored
                const float4 *x4 = reinterpret_cast<const float4 *>(a.x_in + (size_t)m * K + k0);
                constexpr int SB = 10;
                const int n4 = len >> 2;
                for (int i0 = tid; i0 < n4; i0 += 256 * SB) {
                    float4 v[SB];
#pragma unroll
                    for (int j = 0; j < SB; ++j) v[j] = x4[min(i0 + j * 256, n4 - 1)];
#pragma unroll
                    for (int j = 0; j < SB; ++j) {
                        const int i = i0 + j * 256;
                        if (i < n4) xm[(i & 1) * plane_len + (i >> 1)] = v[j];
                    }
                }
            }
        }
    };
    if (resident) { stage(0, K); __syncthreads(); }

    SoftState st[MP];
    float lm_scale[MP];
    unsigned long long noise_base[MP];                   // sampling: (position of the token being predicted) * V
#pragma unroll
    for (int m = 0; m < MP; ++m) {
        st[m].init(); lm_scale[m] = (MODE == G_LMHEAD && m < M) ? a.seq_scale[m] : 1.f;
        noise_base[m] = 0;
        if (MODE == G_LMHEAD && a.sample_on && m < M)
            noise_base[m] = (unsigned long long)(a.row_pos[a.gather ? a.gather[m] : m] + 1) * (unsigned long long)a.N;
    }
    int parity = 0;

    // accumulate chunks [c_begin, c_end) of the tile; the LDS segment starts at chunk seg_c0
    auto accumulate = [&](const uint4 *const (&wp)[RT], int seg_c0, int c_begin, int c_end, int c_step, float (&acc)[RT][MP]) {
#pragma unroll UNR
        for (int c = c_begin; c < c_end; c += c_step) {
            uint4 wv[RT];
#pragma unroll
            for (int r = 0; r < RT; ++r) wv[r] = load_stream(wp[r] + c);
            float4 xa[MP], xb[MP];
#pragma unroll
            for (int m = 0; m < MP; ++m) { xa[m] = xs[(2 * m) * plane_len + c - seg_c0]; xb[m] = xs[(2 * m + 1) * plane_len + c - seg_c0]; }
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                const float w0 = bf16_lo(wv[r].x), w1 = bf16_hi(wv[r].x), w2 = bf16_lo(wv[r].y), w3 = bf16_hi(wv[r].y);
                const float w4 = bf16_lo(wv[r].z), w5 = bf16_hi(wv[r].z), w6 = bf16_lo(wv[r].w), w7 = bf16_hi(wv[r].w);
#pragma unroll
                for (int m = 0; m < MP; ++m) {
                    float v = acc[r][m];
                    v = fmaf(w0, xa[m].x, v); v = fmaf(w1, xa[m].y, v); v = fmaf(w2, xa[m].z, v); v = fmaf(w3, xa[m].w, v);
                    v = fmaf(w4, xb[m].x, v); v = fmaf(w5, xb[m].y, v); v = fmaf(w6, xb[m].z, v); v = fmaf(w7, xb[m].w, v);
                    acc[r][m] = v;
                }
            }
        }
    };

    for (int t = unit0; t < t_hi; t += ustride) {
        int rows[RT];
        int head, pair0; bool rot;
        tile_rows(t, rows, head, pair0, rot);
        const uint4 *wp[RT];
        float acc[RT][MP];
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            wp[r] = reinterpret_cast<const uint4 *>(a.W + (size_t)rows[r] * K);
#pragma unroll
            for (int m = 0; m < MP; ++m) acc[r][m] = 0.f;
        }
        // what the epilogue will need from memory is requested now, ahead of the weight stream
        float epi[RT][MP];
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int m = 0; m < MP; ++m) epi[r][m] = 0.f;
        if (MODE == G_QKV) {
            if (rot) {
#pragma unroll
                for (int m = 0; m < MP; ++m) if (!row_bad[m]) {
#pragma unroll
                    for (int j = 0; j < P; ++j) {
                        epi[2 * j][m] = a.rope_cos[(size_t)row_pos[m] * half + pair0 + j];
                        epi[2 * j + 1][m] = a.rope_sin[(size_t)row_pos[m] * half + pair0 + j];
                    }
                }
            }
        } else if (MODE == G_OPROJ || MODE == G_DOWN) {
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int m = 0; m < MP; ++m) if (m < M) epi[r][m] = a.h_out[(size_t)m * a.ld_h + rows[r]];
        }
        if (resident) {
            int cb = c0;
            if (PRE > 0 && t == unit0) {
#pragma unroll
                for (int u = 0; u < PRE; ++u) {
                    const int c = c0 + u * cstride;
                    const bool valid = c < (K >> 3);
                    const int cc = valid ? c : 0;
                    float4 xa = xs[cc], xb = xs[plane_len + cc];
                    if (!valid) { xa = make_float4(0.f, 0.f, 0.f, 0.f); xb = xa; }
#pragma unroll
                    for (int r = 0; r < RT; ++r) {
                        const uint4 w = pre[u][r];
                        float v = acc[r][0];
                        v = fmaf(bf16_lo(w.x), xa.x, v); v = fmaf(bf16_hi(w.x), xa.y, v); v = fmaf(bf16_lo(w.y), xa.z, v); v = fmaf(bf16_hi(w.y), xa.w, v);
                        v = fmaf(bf16_lo(w.z), xb.x, v); v = fmaf(bf16_hi(w.z), xb.y, v); v = fmaf(bf16_lo(w.w), xb.z, v); v = fmaf(bf16_hi(w.w), xb.w, v);
                        acc[r][0] = v;
                    }
                }
                cb = c0 + PRE * cstride;
            }
            accumulate(wp, 0, cb, K >> 3, cstride, acc);
        } else {
            for (int k0 = 0; k0 < K; k0 += seg) {              // KS == 4 only: the tile loop is workgroup-uniform
                const int len = min(seg, K - k0);
                __syncthreads();
                stage(k0, len);
                __syncthreads();
                accumulate(wp, k0 >> 3, (k0 >> 3) + c0, (k0 + len) >> 3, cstride, acc);
            }
        }
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int m = 0; m < MP; ++m) acc[r][m] = wave_sum(acc[r][m]);
        if (KS > 1) {
            if (lane == 0) {
#pragma unroll
                for (int r = 0; r < RT; ++r)
#pragma unroll
                    for (int m = 0; m < MP; ++m) red[(parity * 4 + wave) * RT * MP + r * MP + m] = acc[r][m];
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int m = 0; m < MP; ++m)
                    acc[r][m] = red[(parity * 4 + 0) * RT * MP + r * MP + m] + red[(parity * 4 + 1) * RT * MP + r * MP + m] +
                                red[(parity * 4 + 2) * RT * MP + r * MP + m] + red[(parity * 4 + 3) * RT * MP + r * MP + m];
            parity ^= 1;
        }
        const bool writer = (KS == 1) ? (lane == 0) : (tid == 0);
        if (!writer) continue;

        // ---- epilogue (one lane)
#pragma unroll
        for (int m = 0; m < MP; ++m) {
            if (m >= M) continue;
            if (MODE == G_QKV) {
                if (row_bad[m]) continue;
                const int pos = row_pos[m], slot = row_slot[m];
                if (rot) {
#pragma unroll
                    for (int j = 0; j < P; ++j) {
                        const int i = pair0 + j;
                        const float c = epi[2 * j][m], s = epi[2 * j + 1][m], x0 = acc[2 * j][m], x1 = acc[2 * j + 1][m];
                        const float y0 = x0 * c - x1 * s, y1 = x1 * c + x0 * s;
                        if (head < a.n_q) {
                            float *q = a.qbuf + (size_t)m * a.n_q * a.head_dim + head * a.head_dim;
                            q[i] = y0; q[i + half] = y1;
                        } else {
                            const size_t base = ((((size_t)a.layer * a.max_seqs + slot) * a.n_kv + (head - a.n_q)) * a.max_ctx + pos) * a.head_dim;
                            a.kcache[base + i] = f32_to_bf16(y0); a.kcache[base + i + half] = f32_to_bf16(y1);
                        }
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < RT; ++j) {
                        const int vr = rows[j] - (a.n_q + a.n_kv) * a.head_dim;      // index inside the V section
                        const int vh = vr / a.head_dim, e = vr % a.head_dim;
                        const size_t base = (((size_t)a.layer * a.max_seqs + slot) * a.n_kv + vh) * (size_t)a.max_ctx * a.head_dim;
                        a.vcache[base + (size_t)e * a.max_ctx + pos] = f32_to_bf16(acc[j][m]);     // V is stored [hd][position]
                    }
                }
            } else if (MODE == G_GATEUP) {
#pragma unroll
                for (int j = 0; j < P; ++j) {
                    const float g = acc[2 * j][m], u = acc[2 * j + 1][m];
                    a.act[(size_t)m * a.d_ffn + t * P + j] = g / (1.0f + expf(-g)) * u;
                }
            } else if (MODE == G_OPROJ || MODE == G_DOWN) {
#pragma unroll
                for (int j = 0; j < RT; ++j) if (t * RT + j < a.N) a.h_out[(size_t)m * a.ld_h + t * RT + j] = epi[j][m] + acc[j][m];
            } else {   // G_LMHEAD
#pragma unroll
                for (int j = 0; j < RT; ++j) if (t * RT + j < a.N) {
                    const float lg = acc[j][m] * lm_scale[m];
                    st[m].push(lg, t * RT + j);
                    if (a.sample_on) st[m].push_noisy(lg, t * RT + j, a.sample_key, noise_base[m]);
                    if (a.logits) a.logits[(size_t)m * a.N + t * RT + j] = lg;
                }
            }
        }
    }
    if (MODE == G_LMHEAD) {
        // one partial per workgroup and token row: the four waves' states meet in LDS
        SoftPartial *sp = reinterpret_cast<SoftPartial *>(red);           // [4][MP], inside the 4 KB tail of the segment
        if (KS == 1) {
            if (lane == 0) {
#pragma unroll
                for (int m = 0; m < MP; ++m) sp[wave * MP + m] = to_partial(st[m]);
            }
            __syncthreads();
            if (tid < MP && tid < M) {
                SoftState s0 = from_partial(sp[tid]);
                for (int w = 1; w < 4; ++w) s0.merge(from_partial(sp[w * MP + tid]));
                a.parts[(size_t)tid * a.n_parts + wg] = to_partial(s0);
            }
        } else if (tid == 0) {
#pragma unroll
            for (int m = 0; m < MP; ++m)
                if (m < M) a.parts[(size_t)m * a.n_parts + wg] = to_partial(st[m]);
        }
    }
}

template <int MODE, int RT, int KS, int UNR, int MP, int PRE = 0>
__global__ void __launch_bounds__(256) k_gemv(GemvArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    gemv_phase<MODE, RT, KS, UNR, MP, PRE>(a, smem, blockIdx.x, gridDim.x);
}

// ------------------------------------------------------------------------------------------------
// Single-row GEMV phases with the activation vector in REGISTERS.  K = 512 * NCH: a row of W is NCH
// chunks of 16 bytes per lane, and lane l of every wave holds exactly the x values those chunks
// meet (elements 8 (l + 64 u) .. + 7, u < NCH), K / 64 floats.  A wave is then self-contained: it
// loads its own copy of h (or of the ready activation), reduces the sum of squares of an RMSNorm
// across its lanes with DPP adds, scales, and streams its weight tiles against registers.  No LDS
// staging, no workgroup barrier, no LDS reads in the stream; the only LDS is the LM head's
// exchange of four softmax states.  The first UG chunks of a wave's first tile are requested
// before the activation loads, so the weight stream's first round trip overlaps the prologue.
// Tiles and epilogues are those of gemv_phase (KS = 1).  MP token rows (a call of a few rows: short catch-up
// spans, small batches) share every weight chunk: each row's x lives in its own registers.
// ------------------------------------------------------------------------------------------------
template <int MODE, int RT, int NCH, int UG, int MP = 1>
__global__ void __launch_bounds__(256) k_gemv_reg(GemvArgs a) {
    static_assert(MODE != G_DOWN, "the down projection splits K over the waves");
    static_assert(UG >= 1 && UG <= NCH, "group size");
    static_assert(MODE != G_LMHEAD || MP == 1, "the LM head runs on one row per sequence; batches take the LDS-staged kernel");
    constexpr bool NORM = (MODE == G_QKV || MODE == G_GATEUP || MODE == G_LMHEAD);
    constexpr int P = RT / 2;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wg = blockIdx.x, nwg = gridDim.x;
    const int K = a.K, M = a.m_rows;                      // K == 512 * NCH (the host checks); M <= MP token rows
    const int half = a.head_dim >> 1;
    int n_tiles, n_rot_tiles = 0;
    if (MODE == G_QKV) {
        n_rot_tiles = (a.n_q + a.n_kv) * (half / P);
        n_tiles = n_rot_tiles + (a.n_kv * a.head_dim) / RT;
    } else if (MODE == G_GATEUP) {
        n_tiles = a.d_ffn / P;
    } else {
        n_tiles = (a.N + RT - 1) / RT;
    }
    const int t_lo = (int)(((unsigned)n_tiles * (unsigned)wg) / (unsigned)nwg), t_hi = (int)(((unsigned)n_tiles * (unsigned)(wg + 1)) / (unsigned)nwg);
    const int unit0 = t_lo + wave;

    auto tile_rows = [&](int t, int (&rows)[RT], int &head, int &pair0, bool &rot) {
        head = 0; pair0 = 0; rot = false;
        if (MODE == G_QKV) {
            if (t < n_rot_tiles) {
                rot = true; head = t / (half / P); pair0 = (t % (half / P)) * P;
#pragma unroll
                for (int j = 0; j < P; ++j) { rows[2 * j] = head * a.head_dim + pair0 + j; rows[2 * j + 1] = rows[2 * j] + half; }
            } else {
#pragma unroll
                for (int j = 0; j < RT; ++j) rows[j] = (a.n_q + a.n_kv) * a.head_dim + (t - n_rot_tiles) * RT + j;
            }
        } else if (MODE == G_GATEUP) {
#pragma unroll
            for (int j = 0; j < P; ++j) { rows[2 * j] = t * P + j; rows[2 * j + 1] = a.d_ffn + t * P + j; }
        } else {
#pragma unroll
            for (int j = 0; j < RT; ++j) rows[j] = min(t * RT + j, a.N - 1);
        }
    };

    // ---- first weight requests of the wave's first tile (a wave without a tile requests the last tile's, unused)
    uint4 pre[UG][RT];
    {
        int rows0[RT], head0, pair00; bool rot0;
        tile_rows(min(unit0, n_tiles - 1), rows0, head0, pair00, rot0);
#pragma unroll
        for (int u = 0; u < UG; ++u)
#pragma unroll
            for (int r = 0; r < RT; ++r) pre[u][r] = load_stream(reinterpret_cast<const uint4 *>(a.W + (size_t)rows0[r] * K) + lane + 64 * u);
    }
    int row_bad[MP], row_pos[MP], row_slot[MP];
#pragma unroll
    for (int m = 0; m < MP; ++m) {
        row_bad[m] = 1; row_pos[m] = 0; row_slot[m] = 0;
        if (MODE == G_QKV && m < M) { row_bad[m] = a.row_bad[m]; row_pos[m] = a.row_pos[m]; row_slot[m] = a.row_slot[m]; }
    }

    // ---- x into registers: token row m, chunk u of this lane (a row past the call's count is a copy of row 0, never written)
    float xr[MP][NCH][8];
#pragma unroll
    for (int m = 0; m < MP; ++m) {
        const int src = (MODE == G_LMHEAD && a.gather) ? a.gather[0] : (m < M ? m : 0);
        const float4 *x4 = reinterpret_cast<const float4 *>(NORM ? a.h_in + (size_t)src * a.ld_h : a.x_in + (size_t)src * K);
        float4 xa[NCH], xb[NCH];
#pragma unroll
        for (int u = 0; u < NCH; ++u) { xa[u] = x4[2 * (lane + 64 * u)]; xb[u] = x4[2 * (lane + 64 * u) + 1]; }
        if (NORM) {
            const uint4 *g4 = reinterpret_cast<const uint4 *>(a.gain);
            uint4 gg[NCH];
#pragma unroll
            for (int u = 0; u < NCH; ++u) gg[u] = g4[lane + 64 * u];
            float ss = 0.f;
#pragma unroll
            for (int u = 0; u < NCH; ++u) {
                ss = fmaf(xa[u].x, xa[u].x, ss); ss = fmaf(xa[u].y, xa[u].y, ss); ss = fmaf(xa[u].z, xa[u].z, ss); ss = fmaf(xa[u].w, xa[u].w, ss);
                ss = fmaf(xb[u].x, xb[u].x, ss); ss = fmaf(xb[u].y, xb[u].y, ss); ss = fmaf(xb[u].z, xb[u].z, ss); ss = fmaf(xb[u].w, xb[u].w, ss);
            }
            const float inv = 1.0f / sqrtf(wave_sum(ss) / (float)K + a.eps);
#pragma unroll
            for (int u = 0; u < NCH; ++u) {
                xr[m][u][0] = xa[u].x * (inv * bf16_lo(gg[u].x)); xr[m][u][1] = xa[u].y * (inv * bf16_hi(gg[u].x));
                xr[m][u][2] = xa[u].z * (inv * bf16_lo(gg[u].y)); xr[m][u][3] = xa[u].w * (inv * bf16_hi(gg[u].y));
                xr[m][u][4] = xb[u].x * (inv * bf16_lo(gg[u].z)); xr[m][u][5] = xb[u].y * (inv * bf16_hi(gg[u].z));
                xr[m][u][6] = xb[u].z * (inv * bf16_lo(gg[u].w)); xr[m][u][7] = xb[u].w * (inv * bf16_hi(gg[u].w));
            }
        } else {
#pragma unroll
            for (int u = 0; u < NCH; ++u) {
                xr[m][u][0] = xa[u].x; xr[m][u][1] = xa[u].y; xr[m][u][2] = xa[u].z; xr[m][u][3] = xa[u].w;
                xr[m][u][4] = xb[u].x; xr[m][u][5] = xb[u].y; xr[m][u][6] = xb[u].z; xr[m][u][7] = xb[u].w;
            }
        }
    }

    SoftState st; st.init();
    const float lm_scale = MODE == G_LMHEAD ? a.seq_scale[0] : 1.f;

    for (int t = unit0; t < t_hi; t += 4) {
        int rows[RT];
        int head, pair0; bool rot;
        tile_rows(t, rows, head, pair0, rot);
        const uint4 *wp[RT];
        float acc[RT][MP], epi[RT][MP];
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            wp[r] = reinterpret_cast<const uint4 *>(a.W + (size_t)rows[r] * K) + lane;
#pragma unroll
            for (int m = 0; m < MP; ++m) { acc[r][m] = 0.f; epi[r][m] = 0.f; }
        }
        // what the epilogue needs from memory is requested ahead of the weight stream
        if (MODE == G_QKV) {
            if (rot) {
#pragma unroll
                for (int m = 0; m < MP; ++m) if (!row_bad[m]) {
#pragma unroll
                    for (int j = 0; j < P; ++j) {
                        epi[2 * j][m] = a.rope_cos[(size_t)row_pos[m] * half + pair0 + j];
                        epi[2 * j + 1][m] = a.rope_sin[(size_t)row_pos[m] * half + pair0 + j];
                    }
                }
            }
        } else if (MODE == G_OPROJ) {
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int m = 0; m < MP; ++m) if (m < M) epi[r][m] = a.h_out[(size_t)m * a.ld_h + rows[r]];
        }
        // groups of UG chunks; the first group of the first tile is already on its way
#pragma unroll
        for (int u0 = 0; u0 < NCH; u0 += UG) {
            uint4 wv[UG][RT];
            if (u0 == 0 && t == unit0) {
#pragma unroll
                for (int u = 0; u < UG; ++u)
#pragma unroll
                    for (int r = 0; r < RT; ++r) wv[u][r] = pre[u][r];
            } else {
#pragma unroll
                for (int u = 0; u < UG; ++u)
#pragma unroll
                    for (int r = 0; r < RT; ++r)
                        if (u0 + u < NCH) wv[u][r] = load_stream(wp[r] + 64 * (u0 + u));
            }
#pragma unroll
            for (int u = 0; u < UG; ++u)
#pragma unroll
                for (int r = 0; r < RT; ++r)
                    if (u0 + u < NCH) {
                        const uint4 w = wv[u][r];
                        const float w0 = bf16_lo(w.x), w1 = bf16_hi(w.x), w2 = bf16_lo(w.y), w3 = bf16_hi(w.y);
                        const float w4 = bf16_lo(w.z), w5 = bf16_hi(w.z), w6 = bf16_lo(w.w), w7 = bf16_hi(w.w);
#pragma unroll
                        for (int m = 0; m < MP; ++m) {
                            const float (&x)[8] = xr[m][u0 + u];
                            float v = acc[r][m];
                            v = fmaf(w0, x[0], v); v = fmaf(w1, x[1], v); v = fmaf(w2, x[2], v); v = fmaf(w3, x[3], v);
                            v = fmaf(w4, x[4], v); v = fmaf(w5, x[5], v); v = fmaf(w6, x[6], v); v = fmaf(w7, x[7], v);
                            acc[r][m] = v;
                        }
                    }
        }
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int m = 0; m < MP; ++m) acc[r][m] = wave_sum(acc[r][m]);
        if (lane != 0) continue;

        // ---- epilogue (one lane)
#pragma unroll
        for (int m = 0; m < MP; ++m) {
            if (m >= M) continue;
            if (MODE == G_QKV) {
                if (row_bad[m]) continue;
                const int pos = row_pos[m], slot = row_slot[m];
                if (rot) {
#pragma unroll
                    for (int j = 0; j < P; ++j) {
                        const int i = pair0 + j;
                        const float c = epi[2 * j][m], sn = epi[2 * j + 1][m], x0 = acc[2 * j][m], x1 = acc[2 * j + 1][m];
                        const float y0 = x0 * c - x1 * sn, y1 = x1 * c + x0 * sn;
                        if (head < a.n_q) {
                            float *q = a.qbuf + (size_t)m * a.n_q * a.head_dim + head * a.head_dim;
                            q[i] = y0; q[i + half] = y1;
                        } else {
                            const size_t base = ((((size_t)a.layer * a.max_seqs + slot) * a.n_kv + (head - a.n_q)) * a.max_ctx + pos) * a.head_dim;
                            a.kcache[base + i] = f32_to_bf16(y0); a.kcache[base + i + half] = f32_to_bf16(y1);
                        }
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < RT; ++j) {
                        const int vr = rows[j] - (a.n_q + a.n_kv) * a.head_dim;      // index inside the V section
                        const int vh = vr / a.head_dim, e = vr % a.head_dim;
                        const size_t base = (((size_t)a.layer * a.max_seqs + slot) * a.n_kv + vh) * (size_t)a.max_ctx * a.head_dim;
                        a.vcache[base + (size_t)e * a.max_ctx + pos] = f32_to_bf16(acc[j][m]);     // V is stored [hd][position]
                    }
                }
            } else if (MODE == G_GATEUP) {
#pragma unroll
                for (int j = 0; j < P; ++j) {
                    const float g = acc[2 * j][m], up = acc[2 * j + 1][m];
                    a.act[(size_t)m * a.d_ffn + t * P + j] = g / (1.0f + expf(-g)) * up;
                }
            } else if (MODE == G_OPROJ) {
#pragma unroll
                for (int j = 0; j < RT; ++j) if (t * RT + j < a.N) a.h_out[(size_t)m * a.ld_h + t * RT + j] = epi[j][m] + acc[j][m];
            } else {   // G_LMHEAD (MP == 1)
#pragma unroll
                for (int j = 0; j < RT; ++j) if (t * RT + j < a.N) {
                    const float lg = acc[j][m] * lm_scale;
                    st.push(lg, t * RT + j);
                    if (a.logits) a.logits[t * RT + j] = lg;
                }
            }
        }
    }
    if (MODE == G_LMHEAD) {
        __shared__ SoftPartial sp[4];
        if (lane == 0) sp[wave] = to_partial(st);
        __syncthreads();
        if (tid == 0) {
            SoftState s0 = from_partial(sp[0]);
            for (int w = 1; w < 4; ++w) s0.merge(from_partial(sp[w]));
            a.parts[wg] = to_partial(s0);
        }
    }
}

// ------------------------------------------------------------------------------------------------
// Single-row down projection (h += W_down . act) without any staging: the four waves of a workgroup
// split K (wave w takes the chunks w * 64 + lane, + 256, ...), and every lane reads the eight activation values of a chunk straight from
// global memory next to the RT weight rows of that chunk.  The activation vector (tens of KB) is
// the same for every workgroup, so those reads are served by the CU's cache and the L2; they cost
// 32 bytes per lane and chunk against RT x 16 bytes of weights, but there is no copy into LDS, no
// barrier before the weight stream starts and no LDS footprint that limits the workgroups per CU.
// grid: workgroups share the ceil(N / RT) row tiles in contiguous ranges.
// ------------------------------------------------------------------------------------------------
template <int RT, int UNR, int MP = 1>
__global__ void __launch_bounds__(256) k_down_direct(GemvArgs a) {
    __shared__ float red[2][4][RT * MP];
    const int K = a.K, n_chunks = K >> 3, M = a.m_rows;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wg = blockIdx.x, nwg = gridDim.x;
    const int n_tiles = (a.N + RT - 1) / RT;
    const int t_lo = (int)(((unsigned)n_tiles * (unsigned)wg) / (unsigned)nwg), t_hi = (int)(((unsigned)n_tiles * (unsigned)(wg + 1)) / (unsigned)nwg);
    const int c0 = wave * 64 + lane, cstride = 256;
    // token row m reads its own activation row; a row past the call's count reads row 0 again and is never written
    const float4 *x4[MP];
#pragma unroll
    for (int m = 0; m < MP; ++m) x4[m] = reinterpret_cast<const float4 *>(a.x_in + (size_t)(m < M ? m : 0) * K);
    int parity = 0;
    for (int t = t_lo; t < t_hi; ++t) {
        float acc[RT][MP], epi[RT][MP];
        const uint4 *wp[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            const int row = min(t * RT + r, a.N - 1);
            wp[r] = reinterpret_cast<const uint4 *>(a.W + (size_t)row * K);
#pragma unroll
            for (int m = 0; m < MP; ++m) {
                acc[r][m] = 0.f;
                epi[r][m] = a.h_out[(size_t)(m < M ? m : 0) * a.ld_h + row];   // requested ahead of the weight stream
            }
        }
#pragma unroll UNR
        for (int c = c0; c < n_chunks; c += cstride) {
            uint4 wv[RT];
#pragma unroll
            for (int r = 0; r < RT; ++r) wv[r] = load_stream(wp[r] + c);
            float4 xa[MP], xb[MP];
#pragma unroll
            for (int m = 0; m < MP; ++m) { xa[m] = x4[m][2 * c]; xb[m] = x4[m][2 * c + 1]; }
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                const uint4 w = wv[r];
                const float w0 = bf16_lo(w.x), w1 = bf16_hi(w.x), w2 = bf16_lo(w.y), w3 = bf16_hi(w.y);
                const float w4 = bf16_lo(w.z), w5 = bf16_hi(w.z), w6 = bf16_lo(w.w), w7 = bf16_hi(w.w);
#pragma unroll
                for (int m = 0; m < MP; ++m) {
                    float v = acc[r][m];
                    v = fmaf(w0, xa[m].x, v); v = fmaf(w1, xa[m].y, v); v = fmaf(w2, xa[m].z, v); v = fmaf(w3, xa[m].w, v);
                    v = fmaf(w4, xb[m].x, v); v = fmaf(w5, xb[m].y, v); v = fmaf(w6, xb[m].z, v); v = fmaf(w7, xb[m].w, v);
                    acc[r][m] = v;
                }
            }
        }
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int m = 0; m < MP; ++m) acc[r][m] = wave_sum(acc[r][m]);
        if (lane == 0) {
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int m = 0; m < MP; ++m) red[parity][wave][r * MP + m] = acc[r][m];
        }
        __syncthreads();
        if (tid == 0) {
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                const int row = t * RT + r;
#pragma unroll
                for (int m = 0; m < MP; ++m)
                    if (row < a.N && m < M)
                        a.h_out[(size_t)m * a.ld_h + row] = epi[r][m] + (red[parity][0][r * MP + m] + red[parity][1][r * MP + m] +
                                                                        red[parity][2][r * MP + m] + red[parity][3][r * MP + m]);
            }
        }
        parity ^= 1;
    }
}

// ------------------------------------------------------------------------------------------------
// Split-K grouped-query decode attention in two kernels.
//
// k_attn_partial: grid (n_slices, n_kv_heads, n_rows), block 256.  A workgroup owns one KV head,
// one slice of the context and ALL query heads of that KV head's group, so every K/V byte is read
// once per row.  Both contractions run on the matrix cores (v_mfma_f32_16x16x32_bf16):
//   scores[token, head] = sum_d K[token, d] q[head, d]     A = K rows (16 tokens x 32 d, 16-byte
//                                                           loads straight from the cache),
//                                                           B = q as three bf16 planes (exact fp32)
//   out[d, head]        = sum_t V[t, d] p[head, t]          A = V, which the cache stores TRANSPOSED
//                                                           ([head_dim][position]) so that a lane's
//                                                           8 tokens are contiguous, B = p as three
//                                                           bf16 planes taken directly from the score
//                                                           accumulator registers (the token <-> k
//                                                           slot assignment is free as long as both
//                                                           operands agree)
// The softmax weights use the hardware exponential (__expf: v_exp_f32 after a multiply; relative error
// ~1e-6 for the arguments that matter, far inside the tolerance, an order of magnitude fewer instructions).
// A wave handles 16 tokens per pass with an online softmax; the four waves are merged through LDS
// and the workgroup writes one partial record per query head: [m, l, 0, 0, acc[HD]] fp32.
//
// k_attn_combine: grid (n_q_heads, n_rows), block 256: merges the slices of one head.
// ------------------------------------------------------------------------------------------------
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

struct AttnArgs {
    const float *qbuf;             // [rows, n_q*hd] fp32, rotated
    const uint16_t *kcache;        // [layer][slot][kv_head][position][hd] bf16
    const uint16_t *vcache;        // [layer][slot][kv_head][hd][position] bf16
    float *partials;               // [rows, n_q, n_slices, hd+4]; behind a list of pieces slice_len[1] in the place of n_slices
    float *out;                    // [rows, n_q*hd] fp32, or the same in operand order (out_frag)
    int out_frag, rsh;             // a matrix-core kernel reads `out`: rows in the order of frag_index with blocks of 1 << rsh
    const int *row_pos, *row_slot, *row_bad;
    int n_q, n_kv, max_ctx, max_seqs, layer, n_slices;
    int slot_split;                // k_attn_span, k_attn_walk with a fixed split: workgroups per sequence, slice and KV head
    int walked;                    // k_attn_walk and the merge after it: the records' maxima are in units of ln 2, rows of one slice have no record
    const int *slice_len;          // walked: positions per slice
    const int4 *pieces;            // walked: list of pieces (PrepArgs), or null for a fixed split
    int direct;                    // k_attn_walk: one slice for every row, no merge follows
    const int4 *seq_info;          // per sequence {first row, end row, cache slot, first row's position}, first row < 0: invalid (k_attn_span)
};

// Place of element k of token row m in an activation buffer of rows of K fp32 values (K a multiple of 32) that a matrix-core
// kernel reads: [block of R rows][32 k][half of 8][g][row of the block][4], g = (k % 32) / 8, half = (k % 8) / 4, R = 1 << rsh: the
// 16 bytes that the lanes (row, g) need for one half of their B operand lie in one contiguous piece of 64 R bytes per request.
// Row by row, a request touches R cache lines that neighbouring lanes take in turn, and the CU's cache looks one up per lane
// (7B shape: QKV / down of 128 rows 32.6 / 51 -> 23.0 / 41.1 us, gate/up of 16 rows 57.0 -> 54.2; of 5 rows the same).
// R is 16 for more than 16 rows, else the smallest power of two that holds the rows: one row's worth of requests for the
// one-row LM head of a long span (1.5B shape: 97 us with blocks of 16, 84 with its own row).
// Four consecutive k (from a multiple of four) stay contiguous.  Buffers hold whole blocks: rows up to the next multiple of 32.
__host__ __device__ __forceinline__ size_t frag_index(int m, int k, int K, int rsh) {
    return ((((size_t)(m >> rsh) * (K >> 5) + (k >> 5)) * 8 + ((k >> 2) & 1) * 4 + ((k >> 3) & 3)) << (rsh + 2)) + ((m & ((1 << rsh) - 1)) << 2) + (k & 3);
}
inline int frag_shift(int rows) { int s = 0; while (s < 4 && (1 << s) < rows) ++s; return s; }

constexpr int ATT_GMAX = 8;       // query heads per kv head, at most
constexpr int ATT_WT = 16;        // tokens per wave and pass

// split 8 fp32 values into three bf16x8 planes whose sum is exact
__device__ __forceinline__ void split3(const float (&x)[8], bf16x8_t (&pl)[3]) {
    uint32_t w0[4], w1[4], w2[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float a = x[2 * i], b = x[2 * i + 1];
        w0[i] = pack_bf16x2(a, b);
        const float ra = a - bf16_lo(w0[i]), rb = b - bf16_hi(w0[i]);
        w1[i] = pack_bf16x2(ra, rb);
        w2[i] = pack_bf16x2(ra - bf16_lo(w1[i]), rb - bf16_hi(w1[i]));
    }
    pl[0] = __builtin_bit_cast(bf16x8_t, make_uint4(w0[0], w0[1], w0[2], w0[3]));
    pl[1] = __builtin_bit_cast(bf16x8_t, make_uint4(w1[0], w1[1], w1[2], w1[3]));
    pl[2] = __builtin_bit_cast(bf16x8_t, make_uint4(w2[0], w2[1], w2[2], w2[3]));
}

template <int HD>
__host__ __device__ constexpr size_t attn_lds_bytes(int G = ATT_GMAX) { return (size_t)(4 * G * (HD + 4) + 2 * 4 * 16) * 4; }

// Cache operands of one wave pass (ATT_WT = 16 tokens from t0): K rows as the A operand of the score
// contraction, V^T rows as the A operand of the output contraction.  The loads are unconditional:
// positions are clamped into the cache row (max_ctx is a multiple of 8, so a group of 4 positions
// that starts at or before max_ctx - 4 ends inside it) and a clamped lane just fetches a duplicate.
// Which tokens count is decided later by masks, once the row's context length has arrived; without
// branches around them the compiler issues all loads back to back and waits once.
template <int HD>
struct AttnTile {
    uint4 k[HD / 32];
    uint2 v[HD / 16];
    __device__ __forceinline__ void load(const uint16_t *Kp, const uint16_t *Vp, int t0, int max_ctx, int j, int kg) {
        const int tok = min(t0 + j, max_ctx - 1);
#pragma unroll
        for (int ds = 0; ds < HD / 32; ++ds)
            k[ds] = *reinterpret_cast<const uint4 *>(Kp + (size_t)tok * HD + 32 * ds + 8 * kg);
        const int tv = min(t0 + 4 * kg, max_ctx - 4);
#pragma unroll
        for (int db = 0; db < HD / 16; ++db)
            v[db] = *reinterpret_cast<const uint2 *>(Vp + (size_t)(16 * db + j) * max_ctx + tv);
    }
};

// One (context slice, kv head, token row) unit.  Slice s covers positions [s*C, (s+1)*C) with C fixed
// by max_ctx and the slice count, NOT by the row's context length: the addresses of the first pass
// are known at launch, so the row table, q, K and V are all requested at once and the unit pays one
// memory round trip instead of three dependent ones.  Slices at or past the context length write
// nothing; attn_combine_unit derives the same slice length and reads only the slices before it.
// UPFRONT = false gives that up: the unit first waits for the row's position and leaves before
// requesting anything when its slice lies past the context.  With UPFRONT every launch reads K and V
// of ALL slices up to max_ctx, whatever the context is; that is the better trade while a layer's cache
// is a few MB (the 1.5B and 7B shapes at 4608 positions: 4.7 and 9.4 MB), and a poor one for a large
// cache (eight KV heads at 9216 positions: 37.7 MB per layer, 12.7 us at a context of 1000).
// ONEPASS: the host promises that a slice is one 64-position pass (C == ATT_BT); the unit then keeps no
// second tile and builds q's bf16 planes d step by d step, which brings it under a third of a SIMD's
// registers (more resident workgroups: a long cache is a throughput problem, not a latency one).
template <int HD, bool UPFRONT = true, bool ONEPASS = false>
__device__ __forceinline__ void attn_partial_unit(const AttnArgs &a, unsigned char *smem, int split, int S, int kvh, int row) {
    constexpr int NDS = HD / 32;       // 32-wide d steps of the score contraction
    constexpr int NDB = HD / 16;       // 16-wide d blocks of the output
    constexpr int PS = HD + 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int j = lane & 15, kg = lane >> 4;
    const int G = a.n_q / a.n_kv;

    // a small footprint matters: eight KV heads at 9216 positions are 1152 workgroups, one round only if a CU
    // holds five of them
    float (*m_lds)[16] = reinterpret_cast<float (*)[16]>(smem);                         // [4 waves][16 columns]
    float (*l_lds)[16] = m_lds + 4;
    float *acc_lds = reinterpret_cast<float *>(smem + (size_t)2 * 4 * 16 * 4);          // [4 waves][G heads][HD+4]

    int C = (a.max_ctx + S - 1) / S;
    C = ((C + ATT_BT - 1) / ATT_BT) * ATT_BT;
    const int t_begin = split * C;
    // with one cache slot the slot index needs no load; otherwise clamp it so that a row the
    // validation rejected (its slot is then stored as 0 anyway) can never address outside the cache
    int slot = 0;
    if (a.max_seqs > 1) slot = min(max(a.row_slot[row], 0), a.max_seqs - 1);
    const int bad = a.row_bad[row];
    const int pos = a.row_pos[row];
    const size_t kv_base = (((size_t)a.layer * a.max_seqs + slot) * a.n_kv + kvh) * (size_t)a.max_ctx * HD;
    const uint16_t *Kp = a.kcache + kv_base;      // [position][hd]
    const uint16_t *Vp = a.vcache + kv_base;      // [hd][position]
    const float scale = 1.0f / sqrtf((float)HD);
    if (!UPFRONT) {
        if (t_begin >= (bad ? 0 : pos + 1)) return;
    }

    // lanes j >= G have no head: they fetch head G-1 again and are cleared after the wait
    float4 qraw[NDS][2];
    {
        const float4 *qp = reinterpret_cast<const float4 *>(a.qbuf + ((size_t)row * a.n_q + kvh * G + min(j, G - 1)) * HD + 8 * kg);
#pragma unroll
        for (int ds = 0; ds < NDS; ++ds) { qraw[ds][0] = qp[8 * ds]; qraw[ds][1] = qp[8 * ds + 1]; }
    }
    AttnTile<HD> cur;
    cur.load(Kp, Vp, t_begin + wave * ATT_WT, a.max_ctx, j, kg);
    __builtin_amdgcn_sched_barrier(0);             // every request is in flight before anything waits

    const int ctx = bad ? 0 : pos + 1;
    const int t_end = min(ctx, t_begin + C);
    if (t_begin >= t_end) return;                  // nothing of this slice is in the context: the merge skips it too

    // q of head j as the B operand of the score contraction: three exact bf16 planes per d step
    auto q_planes = [&](int ds, bf16x8_t (&out)[3]) {
        const float4 x0 = qraw[ds][0], x1 = qraw[ds][1];
        float qv[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
        if (j >= G) {
#pragma unroll
            for (int e = 0; e < 8; ++e) qv[e] = 0.f;
        }
        split3(qv, out);
    };
    bf16x8_t qB[ONEPASS ? 1 : NDS][3];
    if (!ONEPASS) {
#pragma unroll
        for (int ds = 0; ds < NDS; ++ds) q_planes(ds, qB[ds]);
    }

    float m_run = -INFINITY, l_run = 0.f;          // head j (replicated over the four kg groups)
    f32x4_t acc[NDB];                              // out[d = 16 db + 4 kg + r][head j]
#pragma unroll
    for (int db = 0; db < NDB; ++db) acc[db] = (f32x4_t){0.f, 0.f, 0.f, 0.f};

    for (int t0 = t_begin + wave * ATT_WT; t0 < t_end; t0 += ATT_BT) {
        AttnTile<HD> nxt;
        const bool more = !ONEPASS && t0 + ATT_BT < t_end;
        if (more) nxt.load(Kp, Vp, t0 + ATT_BT, a.max_ctx, j, kg);
        // ---- scores of 16 tokens; lane holds tokens t0 + 4 kg + r of head j.
        // Positions at or past t_end may hold anything (a rejected step's rows, never-written memory):
        // their scores are replaced, not scaled.
        f32x4_t sc = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ds = 0; ds < NDS; ++ds) {
            const bf16x8_t A = __builtin_bit_cast(bf16x8_t, cur.k[ds]);
            if (ONEPASS) {
                bf16x8_t qb[3];
                q_planes(ds, qb);
#pragma unroll
                for (int pl = 2; pl >= 0; --pl) sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, qb[pl], sc, 0, 0, 0);
            } else {
#pragma unroll
                for (int pl = 2; pl >= 0; --pl) sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, qB[ds][pl], sc, 0, 0, 0);
            }
        }
        float mx = -INFINITY;
        const int tok_lo = t0 + 4 * kg;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float v = tok_lo + r < t_end ? sc[r] * scale : -INFINITY;
            sc[r] = v;
            mx = fmaxf(mx, v);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16, RS_WAVE));
        mx = fmaxf(mx, __shfl_xor(mx, 32, RS_WAVE));
        const float m_new = fmaxf(m_run, mx);                         // finite: the pass has at least one valid token
        const float alpha = (m_run == -INFINITY) ? 0.f : __expf(m_run - m_new);
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < NDB; ++db) { acc[db][0] *= alpha; acc[db][1] *= alpha; acc[db][2] *= alpha; acc[db][3] *= alpha; }
        // ---- P V: k slot (kg, r) is token t0 + 4 kg + r; slots (kg, 4..7) are unused (zero on both sides)
        float pv[8];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float p = (sc[r] == -INFINITY) ? 0.f : __expf(sc[r] - m_new);
            pv[r] = p; pv[4 + r] = 0.f;
            l_run += p;
        }
        bf16x8_t pB[3];
        split3(pv, pB);
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
            // clear the V columns of positions at or past t_end (0 * NaN would poison the sum)
            uint2 lo = cur.v[db];
            if (tok_lo + 3 >= t_end) {
                if (tok_lo + 1 >= t_end) lo.x &= 0x0000ffffu;
                if (tok_lo + 2 >= t_end) lo.y = 0; else if (tok_lo + 3 >= t_end) lo.y &= 0x0000ffffu;
                if (tok_lo >= t_end) lo.x = 0;
            }
            const bf16x8_t A = __builtin_bit_cast(bf16x8_t, make_uint4(lo.x, lo.y, 0u, 0u));
#pragma unroll
            for (int pl = 2; pl >= 0; --pl) acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, pB[pl], acc[db], 0, 0, 0);
        }
        if (more) cur = nxt;
    }
    // l_run so far covers this lane's own tokens: add the other three kg groups
    l_run += __shfl_xor(l_run, 16, RS_WAVE);
    l_run += __shfl_xor(l_run, 32, RS_WAVE);

    // ---- merge the four waves
    if (j < G) {
#pragma unroll
        for (int db = 0; db < NDB; ++db)
            *reinterpret_cast<float4 *>(&acc_lds[(size_t)(wave * G + j) * PS + 16 * db + 4 * kg]) = make_float4(acc[db][0], acc[db][1], acc[db][2], acc[db][3]);
    }
    if (kg == 0) { m_lds[wave][j] = m_run; l_lds[wave][j] = l_run; }
    __syncthreads();
    // one float4 of one head per thread: G * HD / 4 items (224 for seven heads of 128 channels)
    for (int i = tid; i < G * (HD / 4); i += 256) {
        const int g = i / (HD / 4), d = 4 * (i - g * (HD / 4));
        const float m0 = m_lds[0][g], m1 = m_lds[1][g], m2 = m_lds[2][g], m3 = m_lds[3][g];
        const float M = fmaxf(fmaxf(m0, m1), fmaxf(m2, m3));
        float L = 0.f;
        float4 O = make_float4(0.f, 0.f, 0.f, 0.f);
        if (M > -INFINITY) {
            const float w0 = m0 > -INFINITY ? __expf(m0 - M) : 0.f, w1 = m1 > -INFINITY ? __expf(m1 - M) : 0.f;
            const float w2 = m2 > -INFINITY ? __expf(m2 - M) : 0.f, w3 = m3 > -INFINITY ? __expf(m3 - M) : 0.f;
            L = l_lds[0][g] * w0 + l_lds[1][g] * w1 + l_lds[2][g] * w2 + l_lds[3][g] * w3;
            const float4 a0 = *reinterpret_cast<const float4 *>(&acc_lds[(size_t)(0 * G + g) * PS + d]);
            const float4 a1 = *reinterpret_cast<const float4 *>(&acc_lds[(size_t)(1 * G + g) * PS + d]);
            const float4 a2 = *reinterpret_cast<const float4 *>(&acc_lds[(size_t)(2 * G + g) * PS + d]);
            const float4 a3 = *reinterpret_cast<const float4 *>(&acc_lds[(size_t)(3 * G + g) * PS + d]);
            O.x = a0.x * w0 + a1.x * w1 + a2.x * w2 + a3.x * w3;
            O.y = a0.y * w0 + a1.y * w1 + a2.y * w2 + a3.y * w3;
            O.z = a0.z * w0 + a1.z * w1 + a2.z * w2 + a3.z * w3;
            O.w = a0.w * w0 + a1.w * w1 + a2.w * w2 + a3.w * w3;
        }
        float *p = a.partials + (((size_t)row * a.n_q + kvh * G + g) * S + split) * PS;
        *reinterpret_cast<float4 *>(p + 4 + d) = O;
        if (d == 0) { p[0] = M; p[1] = L; }
    }
}

template <int HD, bool UPFRONT, bool ONEPASS>
__global__ void __launch_bounds__(256, ONEPASS ? 3 : 1) k_attn_partial(AttnArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    attn_partial_unit<HD, UPFRONT, ONEPASS>(a, smem, blockIdx.x, gridDim.x, blockIdx.y, blockIdx.z);
}

// ------------------------------------------------------------------------------------------------
// k_attn_span: partial records for a call with several token rows per sequence (catch-up spans) whose slices are one
// 64-position pass.  The 16 columns of the matrix-core tiles carry RP = 16 / G token rows at once (G = query heads per
// KV head; RP consecutive rows are a row slot): column rr * G + gh is head gh of the rr-th row of the slot, so one K/V
// tile serves RP rows.  Causality is per column: row r attends to positions 0..pos[r].  grid (n_slices, n_kv_heads,
// n_seqs * ZS), block 256
// (ZS = a.slot_split workgroups share a sequence's row slots: workgroup zs takes the slots w + 4 zs, + 4 ZS, ...
// of wave w; long spans are spread over more CUs that way).
// A workgroup owns one context slice of one KV head of one SEQUENCE of the call and all of that
// sequence's rows: the four waves fetch the slice's K rows (64 x HD, contiguous in the cache) and V^T
// rows (HD pieces of 128 bytes) once, with whole-line 16-byte loads, into LDS; then wave w takes the row
// slots w, w + 4, ... and reads its operands from LDS (waves that fetched their operands themselves, one 16-byte (K) or
// 8-byte (V) piece per lane and row, were bound by the CU's vector-memory request rate: 7B shape, 8 rows 17.5 us
// against 13.8, 3 rows 11.0 against 6.8).
// V positions at or past the sequence's last row may hold anything (never written): they are cleared
// when the tile is written to LDS; K rows there only feed scores that the causal mask discards.
// ------------------------------------------------------------------------------------------------
template <int HD>
__host__ __device__ constexpr size_t attn_span_lds_bytes() { return (size_t)64 * (HD * 2 + 16) + (size_t)HD * (64 * 2 + 16); }

// MINW: workgroups per CU that the registers must allow, see span_pairs (attn_plan.h)
template <int HD, int MINW>
__global__ void __launch_bounds__(256, MINW) k_attn_span(AttnArgs a) {
    constexpr int NDS = HD / 32, NDB = HD / 16, PS = HD + 4;
    constexpr int KP = HD * 2 + 16, VP = 64 * 2 + 16;           // LDS row pitches in bytes (padded against bank conflicts)
    constexpr int KQ = 64 * HD * 2 / 4096, VQ = HD * 128 / 4096; // 16-byte loads per thread for each tile
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char *sK = smem, *sV = smem + (size_t)64 * KP;
    const int split = blockIdx.x, S = gridDim.x, kvh = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int j = lane & 15, kg = lane >> 4;
    const int G = a.n_q / a.n_kv, RP = 16 / G;
    const int rr = j / G, gh = j - rr * G;                     // this lane's column: row rr of the slot, head gh
    const int ZS = a.slot_split > 1 ? a.slot_split : 1, zs = blockIdx.z % ZS;
    const int4 info = a.seq_info[blockIdx.z / ZS];             // {first row, end row, cache slot, position of the first row}, first row < 0: skip
    if (info.x < 0) return;
    const int r_lo = info.x, r_hi = info.y, t_begin = split * 64;
    const int ctx_max = info.w + (r_hi - r_lo);                // positions the last row attends to
    const int n_slots = (r_hi - r_lo + RP - 1) / RP;
    if (t_begin >= ctx_max || 4 * zs >= n_slots) return;
    const int kv_slot = min(max(info.z, 0), a.max_seqs - 1);
    const size_t kv_base = (((size_t)a.layer * a.max_seqs + kv_slot) * a.n_kv + kvh) * (size_t)a.max_ctx * HD;
    const float scale = 1.0f / sqrtf((float)HD);

    // the tile: requests first, the first slot's q next, then the LDS writes
    uint4 kq[KQ], vq[VQ];
#pragma unroll
    for (int i = 0; i < KQ; ++i) {
        const int off = (tid + 256 * i) * 16, row = off / (HD * 2), col = off - row * (HD * 2);
        const int tok = min(t_begin + row, a.max_ctx - 1);
        kq[i] = *reinterpret_cast<const uint4 *>(reinterpret_cast<const unsigned char *>(a.kcache + kv_base + (size_t)tok * HD) + col);
    }
#pragma unroll
    for (int i = 0; i < VQ; ++i) {
        const int off = (tid + 256 * i) * 16, d = off >> 7, c8 = (off & 127) >> 4;
        const int tv = min(t_begin + 8 * c8, a.max_ctx - 8);
        vq[i] = *reinterpret_cast<const uint4 *>(a.vcache + kv_base + (size_t)d * a.max_ctx + tv);
    }
    auto load_q = [&](int slot, float4 (&q)[NDS][2]) {
        const int r0 = r_lo + slot * RP, my_row = r0 + rr;
        const bool ok = rr < RP && my_row < r_hi;
        const float4 *qp = reinterpret_cast<const float4 *>(a.qbuf + ((size_t)(ok ? my_row : r_lo) * a.n_q + kvh * G + (ok ? gh : 0)) * HD + 8 * kg);
#pragma unroll
        for (int ds = 0; ds < NDS; ++ds) { q[ds][0] = qp[8 * ds]; q[ds][1] = qp[8 * ds + 1]; }
    };
    float4 qn[NDS][2];
    if (wave + 4 * zs < n_slots) load_q(wave + 4 * zs, qn);
#pragma unroll
    for (int i = 0; i < KQ; ++i) {
        const int off = (tid + 256 * i) * 16, row = off / (HD * 2), col = off - row * (HD * 2);
        *reinterpret_cast<uint4 *>(sK + (size_t)row * KP + col) = kq[i];
    }
#pragma unroll
    for (int i = 0; i < VQ; ++i) {
        const int off = (tid + 256 * i) * 16, d = off >> 7, c8 = (off & 127) >> 4;
        const int t0 = t_begin + 8 * c8;                       // position of the first of this piece's 8 values
        uint4 v = vq[i];
        if (t0 + 7 >= ctx_max) {
            uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (t0 + 2 * e >= ctx_max) w[e] = 0;
                else if (t0 + 2 * e + 1 >= ctx_max) w[e] &= 0x0000ffffu;
            }
            v = make_uint4(w[0], w[1], w[2], w[3]);
        }
        *reinterpret_cast<uint4 *>(sV + (size_t)d * VP + c8 * 16) = v;
    }
    __syncthreads();

    for (int slot = wave + 4 * zs; slot < n_slots; slot += 4 * ZS) {
        const int r0 = r_lo + slot * RP, my_row = r0 + rr;
        const bool col_ok = rr < RP && my_row < r_hi;
        const int ctx_col = col_ok ? info.w + (my_row - r_lo) + 1 : 0;
        const int t_end_col = min(ctx_col, t_begin + 64);
        bf16x8_t qB[NDS][3];
#pragma unroll
        for (int ds = 0; ds < NDS; ++ds) {
            float qv[8] = {qn[ds][0].x, qn[ds][0].y, qn[ds][0].z, qn[ds][0].w, qn[ds][1].x, qn[ds][1].y, qn[ds][1].z, qn[ds][1].w};
            if (!col_ok) {
#pragma unroll
                for (int e = 0; e < 8; ++e) qv[e] = 0.f;
            }
            split3(qv, qB[ds]);
        }
        if (slot + 4 * ZS < n_slots) load_q(slot + 4 * ZS, qn);   // the next slot's q is in flight during this slot's products
        // scores: lane holds positions t_begin + 16 tb + 4 kg + r of its column
        f32x4_t sc[4];
        float mx = -INFINITY;
#pragma unroll
        for (int tb = 0; tb < 4; ++tb) {
            sc[tb] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ds = 0; ds < NDS; ++ds) {
                const bf16x8_t A = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4 *>(sK + (size_t)(16 * tb + j) * KP + 64 * ds + 16 * kg));
#pragma unroll
                for (int pl = 2; pl >= 0; --pl) sc[tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, qB[ds][pl], sc[tb], 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float v = (t_begin + 16 * tb + 4 * kg + r) < t_end_col ? sc[tb][r] * scale : -INFINITY;
                sc[tb][r] = v;
                mx = fmaxf(mx, v);
            }
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16, RS_WAVE));
        mx = fmaxf(mx, __shfl_xor(mx, 32, RS_WAVE));            // -inf for a column without positions in this slice
        float l_run = 0.f;
        f32x4_t acc[NDB];
#pragma unroll
        for (int db = 0; db < NDB; ++db) acc[db] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            float pv[8];
#pragma unroll
            for (int hf = 0; hf < 2; ++hf)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float s_ = sc[2 * ks + hf][r];
                    const float p = (s_ == -INFINITY) ? 0.f : __expf(s_ - mx);
                    pv[4 * hf + r] = p;
                    l_run += p;
                }
            bf16x8_t pB[3];
            split3(pv, pB);
#pragma unroll
            for (int db = 0; db < NDB; ++db) {
                const unsigned char *vr = sV + (size_t)(16 * db + j) * VP + 64 * ks + 8 * kg;
                const uint2 lo = *reinterpret_cast<const uint2 *>(vr), hi = *reinterpret_cast<const uint2 *>(vr + 32);
                const bf16x8_t A = __builtin_bit_cast(bf16x8_t, make_uint4(lo.x, lo.y, hi.x, hi.y));
#pragma unroll
                for (int pl = 2; pl >= 0; --pl) acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, pB[pl], acc[db], 0, 0, 0);
            }
        }
        l_run += __shfl_xor(l_run, 16, RS_WAVE);
        l_run += __shfl_xor(l_run, 32, RS_WAVE);
        if (col_ok && t_begin < t_end_col) {
            float *p = a.partials + (((size_t)my_row * a.n_q + kvh * G + gh) * S + split) * PS;
#pragma unroll
            for (int db = 0; db < NDB; ++db)
                *reinterpret_cast<float4 *>(p + 4 + 16 * db + 4 * kg) = make_float4(acc[db][0], acc[db][1], acc[db][2], acc[db][3]);
            if (kg == 0) { p[0] = mx; p[1] = l_run; }
        }
    }
}

// ------------------------------------------------------------------------------------------------
// k_attn_walk: attention of calls with several rows or several sequences where one 64-position pass per
// workgroup would be many rounds of the machine.  Block 256; grid (n_slices, n_kv_heads, n_seqs * ZS) where the split is fixed,
// (n_kv_heads, pieces) where the row table lists the pieces (attn_plan.h; heads fastest: with eight KV heads every XCD has
// one, so that the groups of a long span meet its K/V rows in one L2).
// A workgroup walks one slice of one group of row slots in passes of 64 positions: the four waves fetch the pass's K rows and V^T pieces with whole-line loads one pass ahead into registers and
// park them in one of two LDS buffers (one bare barrier per pass: the loads of the next pass stay in flight across
// it).  Online softmax per matrix-core column as in the kernels above.
//   SHARE = false: wave w owns row slot 4 group + w of the sequence and takes all 64 positions of a pass
//   SHARE = true:  the sequence has one row slot (decode steps, very short spans); wave w takes the 16 positions
//                  16 w .. of every pass and the four states are merged at the end
// The records' maxima are in units of ln 2 (see q_scale).  A row whose context is one slice leaves no record: it is
// normalised here, and the merge passes it by (or is not launched, where that holds for every row: a.direct).
// What bounds it: long spans the vector work beside the matrix cores (14B, 61 rows at 9000 positions: 53 us a layer against
// 159 for waves that fetched their own tiles; the matrix cores are busy a third of that), decode steps the one pass a
// workgroup has in flight (7B, 128 sequences of 520 .. 1000 positions, 195 MB: 47 us = 4.1 TB/s, 77 + 12 us for one pass per
// workgroup plus the merge; 16 sequences, 42 MB: 11.8 us against 20.6; 32B, 8 ragged sequences: 53 against 104).
// ------------------------------------------------------------------------------------------------
template <int HD>
__host__ __device__ constexpr size_t attn_walk_lds_bytes() { return 2 * attn_span_lds_bytes<HD>(); }

// workgroup barrier for LDS hand-over that leaves global loads in flight: the LDS accesses issued so far complete
// (lgkmcnt(0); expcnt and vmcnt are left alone), then the barrier; the compiler moves no memory access across it
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// largest of the four lanes j, j + 16, j + 32, j + 48 (the position groups of one matrix-core column), in all of them
__device__ __forceinline__ float max_over_kg(float v) {
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

template <int HD, bool SHARE>
__global__ void __launch_bounds__(256, 2) k_attn_walk(AttnArgs a) {
    constexpr int NDS = HD / 32, NDB = HD / 16, PS = HD + 4;
    constexpr int KP = HD * 2 + 16, VP = 64 * 2 + 16;           // LDS row pitches in bytes (padded against bank conflicts)
    constexpr int KQ = 64 * HD * 2 / 4096, VQ = HD * 128 / 4096; // 16-byte loads per thread for each tile
    constexpr int NTB = SHARE ? 1 : 4;                           // 16-position score blocks per wave and pass
    constexpr int SLOTS = SHARE ? 1 : 4;                         // row slots of a group
    constexpr size_t BUF = attn_span_lds_bytes<HD>();
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int j = lane & 15, kg = lane >> 4;
    const int G = a.n_q / a.n_kv, RP = 16 / G;
    const int rr = j / G, gh = j - rr * G;                      // this lane's column: row rr of the slot, head gh
    int kvh, split, group, C, S = a.n_slices;
    int4 info;                                                  // {first row, end row, cache slot, position of the first row}, first row < 0: skip
    if (a.pieces) {
        kvh = blockIdx.x;
        info = a.pieces[2 * blockIdx.y];
        const int4 piece = a.pieces[2 * blockIdx.y + 1];
        group = piece.x; split = piece.y; C = piece.z; S = piece.w;
        if (info.x < 0) return;
    } else {
        split = blockIdx.x; kvh = blockIdx.y;
        const int ZS = a.slot_split, seq = blockIdx.z / ZS;
        group = blockIdx.z % ZS;
        info = a.seq_info[seq];
        C = *a.slice_len;
        if (info.x < 0) {
            // no merge kernel follows a decode step of one slice: the rejected row's output is cleared here
            if (SHARE && a.direct)
                for (int i = tid; i < G * HD; i += 256)
                    a.out[a.out_frag ? frag_index(seq, kvh * G * HD + i, a.n_q * HD, a.rsh) : ((size_t)seq * a.n_q + kvh * G) * HD + i] = 0.f;
            return;
        }
    }
    const int r_lo = info.x, r_hi = info.y;
    const int ctx_max = info.w + (r_hi - r_lo);                 // positions the last row attends to
    const int n_slots = (r_hi - r_lo + RP - 1) / RP, slot0 = SLOTS * group;
    const int t_begin = split * C;
    const int last = min(r_lo + (slot0 + SLOTS) * RP, r_hi) - 1;                     // last row of the group
    const int t_end = min(t_begin + C, info.w + (last - r_lo) + 1);
    if (slot0 >= n_slots || t_begin >= t_end) return;           // no such group, or all of it lies before this slice
    const int kv_slot = min(max(info.z, 0), a.max_seqs - 1);
    const size_t kv_base = (((size_t)a.layer * a.max_seqs + kv_slot) * a.n_kv + kvh) * (size_t)a.max_ctx * HD;
    // one head's K or V rows stay below 2^31 bytes (the launch checks), so a piece is a uniform base and a 32-bit offset
    const unsigned char *Kp = reinterpret_cast<const unsigned char *>(a.kcache + kv_base), *Vp = reinterpret_cast<const unsigned char *>(a.vcache + kv_base);
    // scores in units of ln 2: the factor goes into q before it is split (one rounding per element of q in the place of
    // one per score), and a softmax weight is one subtraction and one v_exp_f32
    const float q_scale = 1.44269504088896341f / sqrtf((float)HD);

    // (vector types, not structs: a struct array that the lambdas capture is left in scratch memory)
    u32x4_t kq[KQ], vq[VQ];
    auto fetch = [&](int t0) {                                   // positions clamped into the cache row
#pragma unroll
        for (int i = 0; i < KQ; ++i) {
            const int off = (tid + 256 * i) * 16, row = off / (HD * 2), col = off - row * (HD * 2);
            kq[i] = *reinterpret_cast<const u32x4_t *>(Kp + (uint32_t)(min(t0 + row, a.max_ctx - 1) * (HD * 2) + col));
        }
#pragma unroll
        for (int i = 0; i < VQ; ++i) {
            const int off = (tid + 256 * i) * 16, d = off >> 7, c8 = (off & 127) >> 4;
            vq[i] = *reinterpret_cast<const u32x4_t *>(Vp + (uint32_t)((d * a.max_ctx + min(t0 + 8 * c8, a.max_ctx - 8)) * 2));
        }
    };
    auto park = [&](unsigned char *buf, int t0) {
        unsigned char *sK = buf, *sV = buf + (size_t)64 * KP;
#pragma unroll
        for (int i = 0; i < KQ; ++i) {
            const int off = (tid + 256 * i) * 16, row = off / (HD * 2), col = off - row * (HD * 2);
            *reinterpret_cast<u32x4_t *>(sK + (size_t)row * KP + col) = kq[i];
        }
        if (t0 + 64 > ctx_max) {
            // positions past the sequence's last row may hold anything (never written): their V columns are cleared
            // (n_ok of a piece's 8 positions are inside)
#pragma unroll
            for (int i = 0; i < VQ; ++i) {
                const int n_ok = ctx_max - (t0 + 8 * (((tid + 256 * i) & 7)));
                auto keep = [&](uint32_t x, int e) { return n_ok >= 2 * e + 2 ? x : (n_ok == 2 * e + 1 ? x & 0x0000ffffu : 0u); };
                vq[i] = (u32x4_t){keep(vq[i].x, 0), keep(vq[i].y, 1), keep(vq[i].z, 2), keep(vq[i].w, 3)};
            }
        }
#pragma unroll
        for (int i = 0; i < VQ; ++i) {
            const int off = (tid + 256 * i) * 16, d = off >> 7, c8 = (off & 127) >> 4;
            *reinterpret_cast<u32x4_t *>(sV + (size_t)d * VP + c8 * 16) = vq[i];
        }
    };

    int parity = 0;
    const int slot = slot0 + (SHARE ? 0 : wave);
    const int my_row = r_lo + slot * RP + rr;
    const bool active = slot < n_slots, col_ok = active && rr < RP && my_row < r_hi;
    // positions this lane's row attends to; a column that belongs to no row (q = 0, never written) takes part in everything
    const int ctx_col = col_ok ? info.w + (my_row - r_lo) + 1 : ctx_max;
    const int ctx_lo = info.w + slot * RP + 1;               // ... and the slot's first row
    const int ctx_hi = min(info.w + (slot + 1) * RP, ctx_max);
    fetch(t_begin);
    bf16x8_t qB[NDS][3];
    {
        const float4 *qp = reinterpret_cast<const float4 *>(a.qbuf + ((size_t)(col_ok ? my_row : r_lo) * a.n_q + kvh * G + (col_ok ? gh : 0)) * HD + 8 * kg);
#pragma unroll
        for (int ds = 0; ds < NDS; ++ds) {
            const float4 x0 = qp[8 * ds], x1 = qp[8 * ds + 1];
            float qv[8] = {x0.x * q_scale, x0.y * q_scale, x0.z * q_scale, x0.w * q_scale, x1.x * q_scale, x1.y * q_scale, x1.z * q_scale, x1.w * q_scale};
            if (!col_ok) {
#pragma unroll
                for (int e = 0; e < 8; ++e) qv[e] = 0.f;
            }
            split3(qv, qB[ds]);
        }
    }
    float m_run = -INFINITY, l_run = 0.f;
    f32x4_t acc[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db) acc[db] = (f32x4_t){0.f, 0.f, 0.f, 0.f};

    for (int t0 = t_begin; t0 < t_end; t0 += 64) {
        unsigned char *buf = smem + parity * BUF;
        parity ^= 1;
        park(buf, t0);
        lds_barrier();                                       // the pass is in LDS; everybody is done with the other buffer's last use
        fetch(walk_next_pass(t0, t_end));
        const int w0 = t0 + (SHARE ? 16 * wave : 0);         // first position this wave looks at
        if (!active || w0 >= ctx_hi) continue;
        const unsigned char *sK = buf, *sV = buf + (size_t)64 * KP;
        // scores: lane holds positions w0 + 16 tb + 4 kg + r of its column.  Consecutive products go to different
        // accumulators; per accumulator the order is d steps, smallest plane first.
        f32x4_t sc[NTB];
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) sc[tb] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ds = 0; ds < NDS; ++ds) {
            bf16x8_t A[NTB];
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb)
                A[tb] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4 *>(sK + (size_t)(w0 - t0 + 16 * tb + j) * KP + 64 * ds + 16 * kg));
#pragma unroll
            for (int pl = 2; pl >= 0; --pl)
#pragma unroll
                for (int tb = 0; tb < NTB; ++tb) sc[tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[tb], qB[ds][pl], sc[tb], 0, 0, 0);
        }
        if (w0 + 16 * NTB > ctx_lo) {                        // the causal edge of some row
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (w0 + 16 * tb + 4 * kg + r >= ctx_col) sc[tb][r] = -INFINITY;
        }
        float mx = -INFINITY;
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) mx = fmaxf(mx, fmaxf(fmaxf(sc[tb][0], sc[tb][1]), fmaxf(sc[tb][2], sc[tb][3])));
        mx = max_over_kg(mx);
        const float m_new = fmaxf(m_run, mx);                // -inf while the column has no position yet
        if (__any(m_new > m_run)) {                          // rescale only when some column's maximum moved
            const float alpha = (m_run == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < NDB; ++db) { acc[db][0] *= alpha; acc[db][1] *= alpha; acc[db][2] *= alpha; acc[db][3] *= alpha; }
            m_run = m_new;
        }
        const float m_sub = m_new == -INFINITY ? 0.f : m_new;                    // 2^-inf = 0 for a column without positions
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
            for (int r = 0; r < 4; ++r) { sc[tb][r] = __builtin_amdgcn_exp2f(sc[tb][r] - m_sub); l_run += sc[tb][r]; }
        // P V: k slot (kg, 4 hf + r) is position w0 + 32 ks + 16 hf + 4 kg + r; SHARE fills only hf = 0
#pragma unroll
        for (int ks = 0; ks < (SHARE ? 1 : 2); ++ks) {
            float pv[8];
#pragma unroll
            for (int r = 0; r < 4; ++r) { pv[r] = sc[SHARE ? 0 : 2 * ks][r]; pv[4 + r] = SHARE ? 0.f : sc[SHARE ? 0 : 2 * ks + 1][r]; }
            bf16x8_t pB[3];
            split3(pv, pB);
            bf16x8_t A[NDB];
#pragma unroll
            for (int db = 0; db < NDB; ++db) {
                const unsigned char *vr = sV + (size_t)(16 * db + j) * VP + 2 * (w0 - t0) + 64 * ks + 8 * kg;
                const uint2 lo = *reinterpret_cast<const uint2 *>(vr);
                uint2 hi = make_uint2(0u, 0u);
                if (!SHARE) hi = *reinterpret_cast<const uint2 *>(vr + 32);
                A[db] = __builtin_bit_cast(bf16x8_t, make_uint4(lo.x, lo.y, hi.x, hi.y));
            }
#pragma unroll
            for (int pl = 2; pl >= 0; --pl)
#pragma unroll
                for (int db = 0; db < NDB; ++db) acc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[db], pB[pl], acc[db], 0, 0, 0);
        }
    }
    l_run += __shfl_xor(l_run, 16, RS_WAVE);
    l_run += __shfl_xor(l_run, 32, RS_WAVE);
    if constexpr (!SHARE) {
        if (col_ok && ctx_col <= C && t_begin == 0) {             // (a later slice of the group holds nothing of this row)
            const float inv = l_run > 0.f ? 1.f / l_run : 0.f;
#pragma unroll
            for (int db = 0; db < NDB; ++db) {
                const int k = (kvh * G + gh) * HD + 16 * db + 4 * kg;
                *reinterpret_cast<float4 *>(a.out + (a.out_frag ? frag_index(my_row, k, a.n_q * HD, a.rsh) : (size_t)my_row * a.n_q * HD + k)) =
                    make_float4(acc[db][0] * inv, acc[db][1] * inv, acc[db][2] * inv, acc[db][3] * inv);
            }
        } else if (col_ok && t_begin < ctx_col) {
            float *p = a.partials + (((size_t)my_row * a.n_q + kvh * G + gh) * S + split) * PS;
#pragma unroll
            for (int db = 0; db < NDB; ++db)
                *reinterpret_cast<float4 *>(p + 4 + 16 * db + 4 * kg) = make_float4(acc[db][0], acc[db][1], acc[db][2], acc[db][3]);
            if (kg == 0) { p[0] = m_run; p[1] = l_run; }
        }
    } else {
        // merge the four waves' states of the slot's 16 columns; the tiles' LDS is free once everybody is here
        __syncthreads();
        float (*m_lds)[16] = reinterpret_cast<float (*)[16]>(smem);
        float (*l_lds)[16] = m_lds + 4;
        float *acc_lds = reinterpret_cast<float *>(smem + (size_t)2 * 4 * 16 * 4);                   // [4 waves][16 columns][HD + 4]
#pragma unroll
        for (int db = 0; db < NDB; ++db)
            *reinterpret_cast<float4 *>(&acc_lds[(size_t)(wave * 16 + j) * PS + 16 * db + 4 * kg]) = make_float4(acc[db][0], acc[db][1], acc[db][2], acc[db][3]);
        if (kg == 0) { m_lds[wave][j] = m_run; l_lds[wave][j] = l_run; }
        __syncthreads();
        for (int i = tid; i < RP * G * (HD / 4); i += 256) {
            const int c = i / (HD / 4), d = 4 * (i - c * (HD / 4)), row = r_lo + slot0 * RP + c / G;
            if (row >= r_hi || t_begin >= info.w + (row - r_lo) + 1) continue;
            const float m0 = m_lds[0][c], m1 = m_lds[1][c], m2 = m_lds[2][c], m3 = m_lds[3][c];
            const float M = fmaxf(fmaxf(m0, m1), fmaxf(m2, m3));                // -inf only if every score is -inf
            const float w0 = m0 > -INFINITY ? __builtin_amdgcn_exp2f(m0 - M) : 0.f, w1 = m1 > -INFINITY ? __builtin_amdgcn_exp2f(m1 - M) : 0.f;
            const float w2 = m2 > -INFINITY ? __builtin_amdgcn_exp2f(m2 - M) : 0.f, w3 = m3 > -INFINITY ? __builtin_amdgcn_exp2f(m3 - M) : 0.f;
            const float L = l_lds[0][c] * w0 + l_lds[1][c] * w1 + l_lds[2][c] * w2 + l_lds[3][c] * w3;
            const float4 a0 = *reinterpret_cast<const float4 *>(&acc_lds[(size_t)(0 * 16 + c) * PS + d]);
            const float4 a1 = *reinterpret_cast<const float4 *>(&acc_lds[(size_t)(1 * 16 + c) * PS + d]);
            const float4 a2 = *reinterpret_cast<const float4 *>(&acc_lds[(size_t)(2 * 16 + c) * PS + d]);
            const float4 a3 = *reinterpret_cast<const float4 *>(&acc_lds[(size_t)(3 * 16 + c) * PS + d]);
            float4 O;
            O.x = a0.x * w0 + a1.x * w1 + a2.x * w2 + a3.x * w3;
            O.y = a0.y * w0 + a1.y * w1 + a2.y * w2 + a3.y * w3;
            O.z = a0.z * w0 + a1.z * w1 + a2.z * w2 + a3.z * w3;
            O.w = a0.w * w0 + a1.w * w1 + a2.w * w2 + a3.w * w3;
            const size_t head = (size_t)row * a.n_q + kvh * G + c % G;
            if (info.w + (row - r_lo) + 1 <= C) {
                const float inv = L > 0.f ? 1.f / L : 0.f;
                const size_t oi = a.out_frag ? frag_index(row, (kvh * G + c % G) * HD + d, a.n_q * HD, a.rsh) : head * HD + d;
                *reinterpret_cast<float4 *>(a.out + oi) = make_float4(O.x * inv, O.y * inv, O.z * inv, O.w * inv);
            } else {
                float *p = a.partials + (head * S + split) * PS;
                *reinterpret_cast<float4 *>(p + 4 + d) = O;
                if (d == 0) { p[0] = M; p[1] = L; }
            }
        }
    }
}

// merge the context slices of one (row, query head); 256 threads = (float4 columns) x (slice groups).
// DQ workgroups share a head, each taking HD / DQ output columns: a head's records are S * (HD+4) floats
// (38 KB for 72 slices), and with one workgroup per head only n_q CUs pull them.
// smem: ATT_SMAX + 1024 floats
template <int HD>
__host__ __device__ constexpr size_t attn_combine_lds_bytes() { return (size_t)(ATT_SMAX + 1024) * 4; }

// SMAX: the slice count this instantiation is unrolled for (n_slices <= SMAX <= ATT_SMAX, a multiple of 64)
// LIST: behind a list of pieces.
template <int HD, int SMAX = ATT_SMAX, int DQ = 1, bool LIST = false>
__device__ __forceinline__ void attn_combine_unit(const AttnArgs &a, unsigned char *smem, int head, int row, int dq = 0) {
    static_assert(SMAX % 64 == 0 && SMAX <= ATT_SMAX, "whole slices per lane, inside the LDS weights array");
    static_assert(HD % (4 * DQ) == 0 && 256 % (HD / 4 / DQ) == 0, "whole float4 columns per workgroup");
    constexpr int PS = HD + 4, NQ = HD / 4 / DQ, NSG = 256 / NQ, NLD = (SMAX + NSG - 1) / NSG, HDB = HD / DQ;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int S = LIST ? a.slice_len[1] : a.n_slices;
    float *w_sh = reinterpret_cast<float *>(smem);                               // [ATT_SMAX]
    float (*red)[HDB] = reinterpret_cast<float (*)[HDB]>(w_sh + ATT_SMAX);       // [NSG][HDB]: 1024 floats
    const float *pbase = a.partials + ((size_t)row * a.n_q + head) * S * PS;
    const int qd = tid % NQ, sg = tid / NQ;
    // The records of all S slices are requested together with the row's position (one round trip instead of
    // two dependent ones); a slice past the context holds whatever an earlier call left there and is
    // replaced, never scaled, once the position has arrived.
    const int bad = a.row_bad[row], pos = a.row_pos[row], len = a.walked ? *a.slice_len : attn_slice_len(a.max_ctx, S);
    constexpr int NPL = SMAX / 64;                          // slices per lane (wave 0)
    float4 buf[NLD];
    float2 mlr[NPL];
#pragma unroll
    for (int k = 0; k < NLD; ++k) {
        const int s = sg + k * NSG;
        buf[k] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (s < S) buf[k] = *reinterpret_cast<const float4 *>(pbase + (size_t)s * PS + 4 + dq * HDB + 4 * qd);
    }
    if (wave == 0) {
#pragma unroll
        for (int k = 0; k < NPL; ++k) {
            const int s = lane + 64 * k;
            mlr[k] = make_float2(0.f, 0.f);
            if (s < S) mlr[k] = *reinterpret_cast<const float2 *>(pbase + (size_t)s * PS);
        }
    }
    __builtin_amdgcn_sched_barrier(0);                      // every request is in flight before anything waits
    // slices that hold context: same slice length as the kernel that wrote the records
    const int S_act = bad ? 0 : min(S, pos / len + 1);
    if (a.walked && S_act == 1) return;                     // k_attn_walk has written this row
#pragma unroll
    for (int k = 0; k < NLD; ++k)
        if (sg + k * NSG >= S_act) buf[k] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (wave == 0) {
        float ms[NPL], ls[NPL], w[NPL];
        float mx = -INFINITY;
#pragma unroll
        for (int k = 0; k < NPL; ++k) {
            const int s = lane + 64 * k;
            ms[k] = -INFINITY; ls[k] = 0.f;
            if (s < S_act) { ls[k] = mlr[k].y; ms[k] = ls[k] > 0.f ? mlr[k].x : -INFINITY; }
            mx = fmaxf(mx, ms[k]);
        }
        const float M = wave_max(mx);
        float lsum = 0.f;
#pragma unroll
        for (int k = 0; k < NPL; ++k) {
            w[k] = ls[k] > 0.f ? (a.walked ? __builtin_amdgcn_exp2f(ms[k] - M) : __expf(ms[k] - M)) : 0.f;
            lsum = fmaf(ls[k], w[k], lsum);
        }
        const float L = wave_sum(lsum);
#pragma unroll
        for (int k = 0; k < NPL; ++k) w_sh[lane + 64 * k] = L > 0.f ? w[k] / L : 0.f;
    }
    __syncthreads();
    float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int k = 0; k < NLD; ++k) {
        const int s = sg + k * NSG;
        const float w = s < S_act ? w_sh[s] : 0.f;
        sum.x = fmaf(w, buf[k].x, sum.x); sum.y = fmaf(w, buf[k].y, sum.y); sum.z = fmaf(w, buf[k].z, sum.z); sum.w = fmaf(w, buf[k].w, sum.w);
    }
    *reinterpret_cast<float4 *>(&red[sg][4 * qd]) = sum;
    __syncthreads();
    if (tid < HDB) {
        float o = 0.f;
#pragma unroll
        for (int g = 0; g < NSG; ++g) o += red[g][tid];
        const int k = head * HD + dq * HDB + tid;
        const size_t oi = a.out_frag ? frag_index(row, k, a.n_q * HD, a.rsh) : (size_t)row * a.n_q * HD + k;
        a.out[oi] = o;
    }
}

// The merge of a few slices (at most 64) for many rows: one wave per (row, head), no LDS.  Lane s holds slice s's weight, lane d the
// channels d, d + 64.  grid ceil(n_rows * n_q / 4), block 256.  LIST: behind a list of pieces, where most rows have one slice.
constexpr int ATT_SFEW = 32;       // slices of a fixed split up to which many rows take it
template <int HD, bool LIST>
__global__ void __launch_bounds__(256) k_attn_merge_few(AttnArgs a, int n_rows) {
    constexpr int PS = HD + 4, NC = (HD + 63) / 64, BATCH = 8;
    const int lane = threadIdx.x & 63, item = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (item >= n_rows * a.n_q) return;
    const int row = item / a.n_q, head = item - row * a.n_q, S = LIST ? a.slice_len[1] : a.n_slices;
    const float *p = a.partials + (size_t)item * S * PS;
    const int bad = a.row_bad[row], pos = a.row_pos[row], len = a.walked ? *a.slice_len : attn_slice_len(a.max_ctx, S);
    if (LIST && !bad && pos < len) return;                  // k_attn_walk has written this row: nothing is requested for it
    // (records of slices past the context hold whatever an earlier call left there and are replaced, never scaled)
    const float2 ml = *reinterpret_cast<const float2 *>(p + (size_t)min(lane, S - 1) * PS);
    float v[BATCH][NC];
    auto load = [&](int s0) {
#pragma unroll
        for (int k = 0; k < BATCH; ++k)
#pragma unroll
            for (int c = 0; c < NC; ++c) v[k][c] = p[(size_t)min(s0 + k, S - 1) * PS + 4 + min(lane + 64 * c, HD - 1)];
    };
    load(0);
    __builtin_amdgcn_sched_barrier(0);                      // every request is in flight before anything waits
    const int S_act = bad ? 0 : min(S, pos / len + 1);
    if (a.walked && S_act == 1) return;                     // k_attn_walk has written this row
    const float l = lane < S_act ? ml.y : 0.f, m = l > 0.f ? ml.x : -INFINITY;
    const float M = wave_max(m), e = l > 0.f ? (a.walked ? __builtin_amdgcn_exp2f(m - M) : __expf(m - M)) : 0.f;
    const float L = wave_sum(l * e), w = L > 0.f ? e / L : 0.f;
    float o[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) o[c] = 0.f;
    for (int s0 = 0; s0 < S_act; s0 += BATCH) {
        if (s0 > 0) load(s0);
#pragma unroll
        for (int k = 0; k < BATCH; ++k) {
            const float wk = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w), min(s0 + k, 63)));
#pragma unroll
            for (int c = 0; c < NC; ++c) o[c] = fmaf(s0 + k < S_act ? wk : 0.f, s0 + k < S_act ? v[k][c] : 0.f, o[c]);
        }
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int d = lane + 64 * c, k = head * HD + d;
        if (d < HD) a.out[a.out_frag ? frag_index(row, k, a.n_q * HD, a.rsh) : (size_t)row * a.n_q * HD + k] = o[c];
    }
}

// grid (n_q_heads, n_rows, DQ)
template <int HD, int SMAX, int DQ, bool LIST>
__global__ void __launch_bounds__(256) k_attn_combine(AttnArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    attn_combine_unit<HD, SMAX, DQ, LIST>(a, smem, blockIdx.x, blockIdx.y, blockIdx.z);
}

}  // namespace rs
