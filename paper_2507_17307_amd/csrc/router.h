// Router kernels: normalised entropy (Eq. 1), argmax and the switching flags
// (Eq. 2 / Algorithm 1) from partial single-pass softmax states.
#pragma once

#include "device_utils.h"
#include "../../include/rstitch.h"

namespace rs {

// One softmax state from the states of all threads of a workgroup of NW waves; valid in thread 0 only.  In place of a tree of
// pairwise merges (two exponentials and eight shuffles at each of its levels): the workgroup's maximum, one rescale of each
// thread's sums to it, then plain sums.  The largest logit of a state is its m; the sampled entry takes the same route.
// sh: NW SoftPartial of LDS, free when the workgroup enters.
template <int NW>
__device__ __forceinline__ SoftState block_merge(const SoftState &t, SoftPartial *sh, bool sample) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const float mw = wave_max(t.m);
    const int iw = wave_min_i32(t.m == mw ? t.idx : 0x7fffffff), bw = __any(t.bad);
    float gw = -INFINITY; int giw = 0x7fffffff;
    if (sample) { gw = wave_max(t.gbest); giw = wave_min_i32(t.gbest == gw ? t.gidx : 0x7fffffff); }
    if (lane == 0) { sh[wave].m = mw; sh[wave].idx = iw; sh[wave].bad = bw; sh[wave].gbest = gw; sh[wave].gidx = giw; }
    __syncthreads();
    SoftState o; o.init();
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const float m = sh[w].m, gb = sh[w].gbest;
        if (m > o.m || (m == o.m && sh[w].idx < o.idx)) o.idx = sh[w].idx;
        o.m = fmaxf(o.m, m);
        o.bad |= sh[w].bad;
        if (gb > o.gbest || (gb == o.gbest && sh[w].gidx < o.gidx)) { o.gbest = gb; o.gidx = sh[w].gidx; }
    }
    const float d = t.m - o.m, e = t.z > 0.f ? expf(d) : 0.f;
    // (a factor of zero takes no part: d * z may overflow where all of a thread's logits are masked with a huge negative value)
    const float z = wave_sum(t.z * e), s = wave_sum(e > 0.f ? e * (t.s + d * t.z) : 0.f);
    if (lane == 0) { sh[wave].z = z; sh[wave].s = s; }
    __syncthreads();
    o.z = sh[0].z; o.s = sh[0].s;
#pragma unroll
    for (int w = 1; w < NW; ++w) { o.z += sh[w].z; o.s += sh[w].s; }
    o.best = o.m;
    return o;
}

// State of the logits x[i] * sc of one thread: the values i = first, first + step, ... (vocab % 4 == 0 and x 16-byte aligned:
// in groups of four).
__device__ __forceinline__ SoftState row_state(const float *__restrict__ x, int vocab, float sc, int first, int step) {
    SoftState st; st.init();
    if ((vocab & 3) == 0) {
        const float4 *x4 = reinterpret_cast<const float4 *>(x);
#pragma unroll 2
        for (int i = first; i < (vocab >> 2); i += step) {
            const float4 q = x4[i];
            st.push4({q.x * sc, q.y * sc, q.z * sc, q.w * sc}, {4 * i, 4 * i + 1, 4 * i + 2, 4 * i + 3}, {true, true, true, true});
        }
    } else {
        for (int i = first; i < vocab; i += 4 * step) {
            const int j[4] = {i, i + step, i + 2 * step, i + 3 * step};
            const bool ok[4] = {true, j[1] < vocab, j[2] < vocab, j[3] < vocab};
            // all four requested before the first is looked at: left to itself the compiler of k_route_wide waits for the first one (3000 rows of
            // 40001 entries 124 -> 107 us, 32769 105 -> 89)
            const float q[4] = {x[i], x[ok[1] ? j[1] : i], x[ok[2] ? j[2] : i], x[ok[3] ? j[3] : i]};
            __builtin_amdgcn_sched_barrier(0);
            st.push4({q[0] * sc, q[1] * sc, q[2] * sc, q[3] * sc}, j, ok);
        }
    }
    return st;
}

// The record of a row from its merged state (one thread).
__device__ __forceinline__ rs_route_out route_record(const SoftState &st, int vocab, float tau, int active, bool bad, int sample) {
    rs_route_out r;
    uint32_t flags = 0;
    if (bad || st.bad || !(st.z > 0.f)) {
        const float qnan = __uint_as_float(0x7fc00000u);
        flags = (bad ? RS_FLAG_BADARG : RS_FLAG_NONFINITE) | RS_FLAG_HI | RS_FLAG_NEXT_LLM;
        if (active == RS_LLM) flags |= RS_FLAG_ACCEPT;
        r.token = -1; r.h_nats = qnan; r.h_norm = qnan; r.max_logit = qnan; r.log_z = qnan;
    } else {
        const float lz = logf(st.z);
        float h = lz - st.s / st.z;
        h = fmaxf(h, 0.f);
        const float hn = h / logf((float)vocab);
        const bool hi = hn > tau;
        flags = (hi ? (RS_FLAG_HI | RS_FLAG_NEXT_LLM) : 0u);
        if (!(active == RS_SLM && hi)) flags |= RS_FLAG_ACCEPT;
        r.token = sample ? st.gidx : st.idx; r.h_nats = h; r.h_norm = hn; r.max_logit = st.m; r.log_z = st.m + lz;
    }
    r.flags = flags;
    return r;
}

// The states that workgroups of one launch leave for each other: three words of eight bytes, past the L2s of the XCDs (which
// are not coherent with each other; a fence would write back and invalidate all of an L2).  The last eight bytes of a SoftPartial, the sampled entry, are
// not among them.
__device__ __forceinline__ void store_partial(SoftPartial *p, const SoftPartial &v) {
    unsigned long long w[4];
    __builtin_memcpy(w, &v, sizeof(v));
#pragma unroll
    for (int i = 0; i < 3; ++i) __hip_atomic_store(reinterpret_cast<unsigned long long *>(p) + i, w[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ SoftPartial load_partial(const SoftPartial *p) {
    unsigned long long w[4];
#pragma unroll
    for (int i = 0; i < 3; ++i) w[i] = __hip_atomic_load(reinterpret_cast<const unsigned long long *>(p) + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    w[3] = 0x7fffffffff800000ull;                             // (nothing sampled: -inf, no index)
    SoftPartial v;
    __builtin_memcpy(&v, w, sizeof(v));
    return v;
}

// Final merge and routing decision for one row by one 256-thread workgroup.
// row_bad: optional per-row flag (nonzero = the row's inputs were out of range); sh: 4 SoftPartial of LDS.
// HERE: the states were stored by other workgroups of this launch (k_route_wide): loaded past the L2s, without the sampled entry.
// sample: the record's token is the arg max of logit + Gumbel noise (a draw from the distribution) instead of the arg max
template <bool HERE = false>
__device__ __forceinline__ void route_merge_row(const SoftPartial *__restrict__ parts, int n_parts, int vocab, float tau,
                                                int active, const int *__restrict__ row_bad, rs_route_out *__restrict__ out,
                                                int row, SoftPartial *sh, int sample = 0) {
    const int tid = threadIdx.x;
    const SoftPartial *pr = parts + (size_t)row * n_parts;
    const bool bad = row_bad && row_bad[row];
    // a thread's partials, four requested at a time: their common maximum first, so that the sums wait for one exponential
    // each instead of a chain of merges
    SoftState st; st.init();
    for (int p0 = tid; p0 < n_parts; p0 += 1024) {
        SoftPartial q[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) q[k] = HERE ? load_partial(pr + min(p0 + 256 * k, n_parts - 1)) : pr[min(p0 + 256 * k, n_parts - 1)];
        float m = st.m;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (p0 + 256 * k >= n_parts) q[k].z = 0.f;
            else {
                st.bad |= q[k].bad;
                if (q[k].best > st.best || (q[k].best == st.best && q[k].idx < st.idx)) { st.best = q[k].best; st.idx = q[k].idx; }
                if (q[k].gbest > st.gbest || (q[k].gbest == st.gbest && q[k].gidx < st.gidx)) { st.gbest = q[k].gbest; st.gidx = q[k].gidx; }
            }
            if (q[k].z > 0.f) m = fmaxf(m, q[k].m);
        }
        if (st.z > 0.f && m > st.m) { const float d = st.m - m, e = expf(d); st.s = e > 0.f ? e * (st.s + d * st.z) : 0.f; st.z *= e; }
        st.m = m;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (q[k].z > 0.f) { const float d = q[k].m - m, e = expf(d); st.s += e > 0.f ? e * (q[k].s + d * q[k].z) : 0.f; st.z = fmaf(q[k].z, e, st.z); }
    }
    const SoftState o = block_merge<4>(st, sh, sample != 0);
    if (tid == 0) out[row] = route_record(o, vocab, tau, active, bad, sample);
}

// grid n_rows, block 256
__global__ void __launch_bounds__(256)
k_route_merge(const SoftPartial *__restrict__ parts, int n_parts, int vocab, float tau, int active,
              const int *__restrict__ row_bad, rs_route_out *__restrict__ out, int sample) {
    __shared__ SoftPartial sh[4];
    route_merge_row(parts, n_parts, vocab, tau, active, row_bad, out, blockIdx.x, sh, sample);
}

// The whole of rs_route for long rows: grid (n_parts, n_rows), block 256.  Each workgroup strides over its row and leaves its state; the one that
// finds all others of the row arrived merges them.  Arrivals are counted in the word behind the row's first state, {tag, count}: nobody has cleared
// the caller's scratch, so a word without this call's 56-bit tag counts as zero, and the last workgroup leaves zero (a captured call is replayed with
// its tag).  Nothing waits for another workgroup.
// What bounds it: a few rows the launch and the round trips (calls back to back, one row of 50257 / 152064 entries: 8.5 / 8.6 us with a second kernel for the
// merge, 5.6 / 6.2 now; 8 of 152064 8.9 -> 6.7), many the exponentials (64 of 152064 15.1 -> 12.8, 128 22.8 -> 19.8, both with exp_small and 1536 workgroups in the place of 2048).  The word is read before the logits and set while they
// are added up, so that a workgroup's last act is one addition: a loop of compare and exchange in its place took 102 us for 128 workgroups of a row.
__global__ void __launch_bounds__(256)
k_route_wide(const float *__restrict__ logits, int vocab, const float *__restrict__ scale, SoftPartial *parts, unsigned long long tag, float tau, int active,
             rs_route_out *__restrict__ out) {
    __shared__ SoftPartial sh[4];
    __shared__ int sh_last;
    const int row = blockIdx.y, n_parts = gridDim.x;
    SoftPartial *pr = parts + (size_t)row * n_parts;
    unsigned long long *word = reinterpret_cast<unsigned long long *>(pr) + 3, seen = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const SoftState st = row_state(logits + (size_t)row * vocab, vocab, scale ? scale[row] : 1.f, blockIdx.x * 256 + threadIdx.x, n_parts * 256);
    if (threadIdx.x == 0 && (seen >> 8) != tag)                // this call's first: no arrivals yet (fails where another workgroup was faster)
        __hip_atomic_compare_exchange_strong(word, &seen, tag << 8, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const SoftState a = block_merge<4>(st, sh, false);
    if (threadIdx.x == 0) {
        store_partial(pr + blockIdx.x, to_partial(a));
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // acknowledged where the other XCDs read it, before it counts as arrived
        const bool last = (__hip_atomic_fetch_add(word, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 255) + 1 == n_parts;
        if (last) __hip_atomic_store(word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sh_last = last;
    }
    __syncthreads();
    if (sh_last) route_merge_row<true>(parts, n_parts, vocab, tau, active, nullptr, out, row, sh);
}

// The whole of rs_route for a short row: grid n_rows, block 1024, no partial states in memory and no second launch.
__global__ void __launch_bounds__(1024)
k_route_row(const float *__restrict__ logits, int vocab, const float *__restrict__ scale, float tau, int active,
            rs_route_out *__restrict__ out) {
    __shared__ SoftPartial sh[16];
    const int row = blockIdx.x;
    const SoftState st = row_state(logits + (size_t)row * vocab, vocab, scale ? scale[row] : 1.f, threadIdx.x, 1024);
    const SoftState o = block_merge<16>(st, sh, false);
    if (threadIdx.x == 0) out[row] = route_record(o, vocab, tau, active, false, 0);
}

// ------------------------------------------------------------------------------------------------
// Router of R-Stitch+ (Section "Architecture and Overhead of Router"; Algorithm 1, R-Stitch+ branch):
// six residual feed-forward blocks x <- x + W2 gelu(W1 x + b1) + b2 with a bottleneck of r channels,
// a LayerNorm, a linear layer with two outputs (0 = stay on the small model, 1 = switch to the large
// one).  One workgroup of ROUTER_THREADS threads per sequence; x (fp32, d values) lives in LDS; weights are bf16,
// accumulation fp32.  The record of the sequence is updated in place: a small-model step above tau
// whose router output prefers "stay" keeps its token and stays (RS_FLAG_ROUTER_STAY); every other
// record is left as the entropy rule made it.
// What bounds it: one workgroup's chain of twelve phases, each a read of x or t from LDS, its sums and a barrier.  The weights do not depend on x,
// so each phase requests those of the next one before it starts on its own (one call, d 1536, r 8: 25.4 -> 10.1 us; 5120, 8: 65 -> 22; all six
// blocks' weights requested up front 10.8).
// With a wide bottleneck it is the megabytes that one CU draws (5120, 64: 562 -> 191 us for 7.9 MB).
// ------------------------------------------------------------------------------------------------
constexpr int ROUTER_BLOCKS = 6;
constexpr int ROUTER_RMAX = 64;

struct RouterPlusArgs {
    const uint16_t *w1[ROUTER_BLOCKS], *b1[ROUTER_BLOCKS], *w2[ROUTER_BLOCKS], *b2[ROUTER_BLOCKS];
    const uint16_t *ln_gain, *ln_bias, *w_head, *b_head;
    int d, r;
    float ln_eps;
    const float *hidden; int ld_hidden;       // rows of d floats, ld_hidden apart
    const int *gather;                         // row of sequence b inside `hidden`, or null (= b)
    int active;
    rs_route_out *out;                         // [n_seqs], updated in place
    float *logits;                             // [n_seqs, 2] or null
};

constexpr int ROUTER_THREADS = 512, ROUTER_WAVES = ROUTER_THREADS / 64;

__device__ __forceinline__ float2 block_sum2(float v, float w, float2 *sh) {        // sh: ROUTER_WAVES float2 of LDS
    v = wave_sum(v); w = wave_sum(w);
    __syncthreads();                                                      // sh may still be read from the last call
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = make_float2(v, w);
    __syncthreads();
    float2 t = sh[0];
#pragma unroll
    for (int i = 1; i < ROUTER_WAVES; ++i) { t.x += sh[i].x; t.y += sh[i].y; }
    return t;
}

__device__ __forceinline__ float dot8f(const uint4 &w, const float4 &xa, const float4 &xb, float acc) {
    acc = fmaf(bf16_lo(w.x), xa.x, acc); acc = fmaf(bf16_hi(w.x), xa.y, acc); acc = fmaf(bf16_lo(w.y), xa.z, acc); acc = fmaf(bf16_hi(w.y), xa.w, acc);
    acc = fmaf(bf16_lo(w.z), xb.x, acc); acc = fmaf(bf16_hi(w.z), xb.y, acc); acc = fmaf(bf16_lo(w.w), xb.z, acc); return fmaf(bf16_hi(w.w), xb.w, acc);
}

// the two outputs, and the decision in the record (one thread writes)
__device__ __forceinline__ void router_decide(const RouterPlusArgs &a, float o0, float o1) {
    const int b = blockIdx.x;
    if (threadIdx.x != 0) return;
    o0 += bf16_to_f32(a.b_head[0]);
    o1 += bf16_to_f32(a.b_head[1]);
    if (a.logits) { a.logits[2 * b] = o0; a.logits[2 * b + 1] = o1; }
    rs_route_out rec = a.out[b];
    const uint32_t untouchable = RS_FLAG_NONFINITE | RS_FLAG_BADARG | RS_FLAG_ABORTED;
    if (a.active == RS_SLM && (rec.flags & RS_FLAG_HI) && !(rec.flags & untouchable) && !(o1 > o0)) {
        rec.flags = (rec.flags | RS_FLAG_ACCEPT | RS_FLAG_ROUTER_STAY) & ~RS_FLAG_NEXT_LLM;
        a.out[b] = rec;
    }
}

// NU: pieces of a row of W1 per lane (8 channels each) and output channels per thread, at least d / 512: widths up to 5120.
// dynamic LDS: d floats
template <int NU>
__global__ void __launch_bounds__(ROUTER_THREADS) k_router_plus(RouterPlusArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    float *x = reinterpret_cast<float *>(smem);
    __shared__ __align__(16) float t_sh[ROUTER_RMAX];
    __shared__ float2 red[ROUTER_WAVES];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int d = a.d, r = a.r, n_ch = d >> 3;
    const float *src = a.hidden + (size_t)(a.gather ? a.gather[b] : b) * a.ld_hidden;
    // (vector types: arrays of structs that lambdas capture are left in scratch memory)
    auto load_w1 = [&](int blk, int row, u32x4_t (&w)[NU]) {
        const u32x4_t *wp = reinterpret_cast<const u32x4_t *>(a.w1[blk] + (size_t)row * d);
#pragma unroll
        for (int u = 0; u < NU; ++u) w[u] = wp[min(lane + 64 * u, n_ch - 1)];
    };
    u32x4_t w1[NU];
    float xin[NU];
#pragma unroll
    for (int k = 0; k < NU; ++k) xin[k] = src[min(tid + ROUTER_THREADS * k, d - 1)];
    load_w1(0, wave, w1);
#pragma unroll
    for (int k = 0; k < NU; ++k)
        if (tid + ROUTER_THREADS * k < d) x[tid + ROUTER_THREADS * k] = xin[k];
    __syncthreads();
    for (int blk = 0; blk < ROUTER_BLOCKS; ++blk) {
        // the first 8 of the r values of this thread's rows of W2, and their biases
        u32x4_t w2[NU];
        float b2[NU];
#pragma unroll
        for (int k = 0; k < NU; ++k) {
            const int i = min(tid + ROUTER_THREADS * k, d - 1);
            w2[k] = *reinterpret_cast<const u32x4_t *>(a.w2[blk] + (size_t)i * r);
            b2[k] = bf16_to_f32(a.b2[blk][i]);
        }
        // t = gelu(W1 x + b1): wave w takes the rows w, w + 8, ... (r is a multiple of 8); lanes stride over d in pieces of 8
        for (int row = wave; row < r; row += ROUTER_WAVES) {
            if (row != wave) load_w1(blk, row, w1);
            const float b1 = bf16_to_f32(a.b1[blk][row]);
            float acc = 0.f;
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const int c = lane + 64 * u;
                if (c < n_ch) acc = dot8f(make_uint4(w1[u].x, w1[u].y, w1[u].z, w1[u].w), *reinterpret_cast<const float4 *>(x + 8 * c), *reinterpret_cast<const float4 *>(x + 8 * c + 4), acc);
            }
            acc = wave_sum(acc);
            if (lane == 0) {
                const float z = acc + b1;
                t_sh[row] = 0.5f * z * (1.0f + erff(z * 0.70710678118654752f));
            }
        }
        load_w1(min(blk + 1, ROUTER_BLOCKS - 1), wave, w1);               // the next block's first rows (after the last: unused)
        __syncthreads();
        // x += W2 t + b2: output channels tid, tid + 512, ...; a row of W2 is r bf16 values
#pragma unroll
        for (int k = 0; k < NU; ++k) {
            const int i = tid + ROUTER_THREADS * k;
            if (i >= d) continue;
            float acc = dot8f(make_uint4(w2[k].x, w2[k].y, w2[k].z, w2[k].w), *reinterpret_cast<const float4 *>(t_sh), *reinterpret_cast<const float4 *>(t_sh + 4), b2[k]);
            const uint4 *wp = reinterpret_cast<const uint4 *>(a.w2[blk] + (size_t)i * r);
            for (int c = 1; c < (r >> 3); ++c) acc = dot8f(wp[c], *reinterpret_cast<const float4 *>(t_sh + 8 * c), *reinterpret_cast<const float4 *>(t_sh + 8 * c + 4), acc);
            x[i] += acc;
        }
        __syncthreads();
    }
    // LayerNorm (mean, then the mean of squared deviations), then the two outputs.  A thread's channels are in registers.
    float xv[NU], gain[NU], bias[NU], h0[NU], h1[NU], s = 0.f;
#pragma unroll
    for (int k = 0; k < NU; ++k) {
        const int i = tid + ROUTER_THREADS * k, j = min(i, d - 1);
        gain[k] = bf16_to_f32(a.ln_gain[j]); bias[k] = bf16_to_f32(a.ln_bias[j]);
        h0[k] = bf16_to_f32(a.w_head[j]); h1[k] = bf16_to_f32(a.w_head[d + j]);
        xv[k] = i < d ? x[i] : 0.f;
        s += xv[k];
    }
    const float mu = block_sum2(s, 0.f, red).x / (float)d;
    float q = 0.f;
#pragma unroll
    for (int k = 0; k < NU; ++k) { const float dv = tid + ROUTER_THREADS * k < d ? xv[k] - mu : 0.f; q = fmaf(dv, dv, q); }
    const float inv = 1.0f / sqrtf(block_sum2(q, 0.f, red).x / (float)d + a.ln_eps);
    float o0 = 0.f, o1 = 0.f;
#pragma unroll
    for (int k = 0; k < NU; ++k) {
        if (tid + ROUTER_THREADS * k >= d) continue;
        const float y = (xv[k] - mu) * inv * gain[k] + bias[k];
        o0 = fmaf(h0[k], y, o0);
        o1 = fmaf(h1[k], y, o1);
    }
    const float2 o = block_sum2(o0, o1, red);
    router_decide(a, o.x, o.y);
}

// Wider ones: the same phases over parts of ROUTER_PART pieces of 512 channels, of which only the first part's weights are requested a
// phase ahead.  (With one part of 24 pieces for every width the kernel above spilled 123 registers: d 5128, r 8, 1 / 128 sequences
// 53 / 74 us a call, now 30 / 32; 8192, 16: 86 / 118 -> 59 / 62; 12288, 64: 491 / 506 -> 445 / 478.)  dynamic LDS: d floats
constexpr int ROUTER_PART = 8;
__global__ void __launch_bounds__(ROUTER_THREADS) k_router_plus_wide(RouterPlusArgs a) {
    constexpr int NU = ROUTER_PART;
    extern __shared__ __align__(16) unsigned char smem[];
    float *x = reinterpret_cast<float *>(smem);
    __shared__ __align__(16) float t_sh[ROUTER_RMAX];
    __shared__ float2 red[ROUTER_WAVES];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int d = a.d, r = a.r, n_ch = d >> 3, parts = (d + ROUTER_THREADS * NU - 1) / (ROUTER_THREADS * NU);
    const float *src = a.hidden + (size_t)(a.gather ? a.gather[b] : b) * a.ld_hidden;
    auto channel = [&](int part, int k) { return tid + ROUTER_THREADS * (k + NU * part); };       // output channel k of this thread
    auto load_w1 = [&](int blk, int row, int part, u32x4_t (&w)[NU]) {
        const u32x4_t *wp = reinterpret_cast<const u32x4_t *>(a.w1[blk] + (size_t)row * d);
#pragma unroll
        for (int u = 0; u < NU; ++u) w[u] = wp[min(lane + 64 * (u + NU * part), n_ch - 1)];
    };
    auto load_w2 = [&](int blk, int part, u32x4_t (&w)[NU], float (&bias)[NU]) {
#pragma unroll
        for (int k = 0; k < NU; ++k) {
            const int i = min(channel(part, k), d - 1);
            w[k] = *reinterpret_cast<const u32x4_t *>(a.w2[blk] + (size_t)i * r);
            bias[k] = bf16_to_f32(a.b2[blk][i]);
        }
    };
    auto dot_w1 = [&](int part, const u32x4_t (&w)[NU], float acc) {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int c = lane + 64 * (u + NU * part);
            if (c < n_ch) acc = dot8f(make_uint4(w[u].x, w[u].y, w[u].z, w[u].w), *reinterpret_cast<const float4 *>(x + 8 * c), *reinterpret_cast<const float4 *>(x + 8 * c + 4), acc);
        }
        return acc;
    };
    auto add_w2 = [&](int blk, int part, const u32x4_t (&w)[NU], const float (&bias)[NU]) {
#pragma unroll
        for (int k = 0; k < NU; ++k) {
            const int i = channel(part, k);
            if (i >= d) continue;
            float acc = dot8f(make_uint4(w[k].x, w[k].y, w[k].z, w[k].w), *reinterpret_cast<const float4 *>(t_sh), *reinterpret_cast<const float4 *>(t_sh + 4), bias[k]);
            const uint4 *wp = reinterpret_cast<const uint4 *>(a.w2[blk] + (size_t)i * r);
            for (int c = 1; c < (r >> 3); ++c) acc = dot8f(wp[c], *reinterpret_cast<const float4 *>(t_sh + 8 * c), *reinterpret_cast<const float4 *>(t_sh + 8 * c + 4), acc);
            x[i] += acc;
        }
    };
    u32x4_t w1[NU];
    load_w1(0, wave, 0, w1);
    for (int i = tid; i < d; i += ROUTER_THREADS) x[i] = src[i];
    __syncthreads();
    for (int blk = 0; blk < ROUTER_BLOCKS; ++blk) {
        u32x4_t w2[NU];
        float b2[NU];
        load_w2(blk, 0, w2, b2);
        for (int row = wave; row < r; row += ROUTER_WAVES) {
            const float b1 = bf16_to_f32(a.b1[blk][row]);
            if (row != wave) load_w1(blk, row, 0, w1);
            float acc = dot_w1(0, w1, 0.f);
#pragma unroll 1
            for (int part = 1; part < parts; ++part) { load_w1(blk, row, part, w1); acc = dot_w1(part, w1, acc); }
            acc = wave_sum(acc);
            if (lane == 0) {
                const float z = acc + b1;
                t_sh[row] = 0.5f * z * (1.0f + erff(z * 0.70710678118654752f));
            }
        }
        load_w1(min(blk + 1, ROUTER_BLOCKS - 1), wave, 0, w1);
        __syncthreads();
        add_w2(blk, 0, w2, b2);
#pragma unroll 1
        for (int part = 1; part < parts; ++part) { load_w2(blk, part, w2, b2); add_w2(blk, part, w2, b2); }
        __syncthreads();
    }
    float s = 0.f, q = 0.f, o0 = 0.f, o1 = 0.f;
    for (int i = tid; i < d; i += ROUTER_THREADS) s += x[i];
    const float mu = block_sum2(s, 0.f, red).x / (float)d;
    for (int i = tid; i < d; i += ROUTER_THREADS) { const float dv = x[i] - mu; q = fmaf(dv, dv, q); }
    const float inv = 1.0f / sqrtf(block_sum2(q, 0.f, red).x / (float)d + a.ln_eps);
#pragma unroll 4
    for (int i = tid; i < d; i += ROUTER_THREADS) {
        const float y = (x[i] - mu) * inv * bf16_to_f32(a.ln_gain[i]) + bf16_to_f32(a.ln_bias[i]);
        o0 = fmaf(bf16_to_f32(a.w_head[i]), y, o0);
        o1 = fmaf(bf16_to_f32(a.w_head[d + i]), y, o1);
    }
    const float2 o = block_sum2(o0, o1, red);
    router_decide(a, o.x, o.y);
}

}  // namespace rs
