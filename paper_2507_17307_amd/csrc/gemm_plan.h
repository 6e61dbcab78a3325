// Arithmetic of the launches of the matrix-core products (k_gemm_rows, k_gemm_ring): which kernel takes a matrix, how K is split and how many
// column tiles a workgroup gets; and of the down projection of few rows (k_down_direct).  Plain C++ without HIP types, so that it can also be compiled and checked on a CPU.
#pragma once

#include <cstddef>
#include <initializer_list>

namespace rs {

constexpr int GEMM_KW = 64;                       // k elements per window: K must be a multiple
constexpr int KSPLIT_MAX = 8;                     // workgroup-level splits of K, at most

// ---- In which order a product's terms are added: a matter of its shape, kept apart from the kernels and their launch shapes.
// K and V are rounded to bf16, and a sum in another order now and then rounds the other way; with a context of a few hundred positions one
// such step moves a row's logits by up to 1e-4 of their size, fifty times what the order itself does.  So the splits of K below stay as
// they are whichever kernel takes a matrix.
// k_gemm_rows: tiles of a workgroup, and its split of K: further while the launch has fewer than 1.75 workgroups per CU (A/B of the
// whole stitched run: with a threshold of 2 the 7B O-proj went from 448 to 896 workgroups of 7 windows each and its calls
// were 0.04 ms slower)
inline int rows_tiles(bool one_block, int n_win) { return one_block && n_win < 128 ? 2 : 4; }      // short rows: smaller groups rather than thin K slices
inline int split_few(bool one_block, int n_tiles, int n_win, int n_cu) {
    const int r = rows_tiles(one_block, n_win), groups = (n_tiles + r - 1) / r;
    int ks = 1;
    while (ks < KSPLIT_MAX && groups * ks < 7 * n_cu / 4 && n_win / (2 * ks) >= 4) ks *= 2;
    return ks;
}
// k_gemm_rows, products over whole K (gate/up and LM head of up to 16 rows): tiles of a workgroup
inline int rows_tiles_whole(int n_tiles, int n_cu) { return (n_tiles + 1) / 2 >= 7 * n_cu / 4 ? 2 : 1; }
// More than 16 rows: the split with which groups of ten tiles or fewer (gate/up, which cannot be split: pairs of five or fewer) come
// closest to whole rounds of the machine, and how close that is.
struct SplitPlan { int ks; double eff; };
inline SplitPlan split_many(bool gateup, int n_tiles, int n_win, int n_cu) {
    static const int ct_gu[] = {5, 4, 3, 2, 0}, ct_part[] = {10, 8, 7, 6, 4, 0};
    SplitPlan best{1, -1.0};
    for (const int *c = gateup ? ct_gu : ct_part; *c; ++c) {
        const int groups = (n_tiles + *c - 1) / *c;
        for (int ks = 1; ks <= (gateup ? 1 : KSPLIT_MAX); ++ks) {
            if (ks > 1 && n_win / ks < 6) break;
            const int units = groups * ks, rounds = (units + n_cu - 1) / n_cu;
            const double eff = (double)units / ((double)rounds * n_cu) * ((double)n_tiles / ((double)groups * *c));
            if (eff > best.eff + 1e-9) best = SplitPlan{ks, eff};
        }
    }
    return best;
}

// k_gemm_ring: multiplying waves that share a block of 16 rows and split the workgroup's columns
inline int ring_column_splits(int M) { return M <= 16 ? 4 : M <= 32 ? 2 : 1; }
// More than 64 rows: whether eight waves of one block multiply and not four of two.  A wave splits its X into planes by itself, some 110
// vector instructions a block and window, which the matrix instructions of a few tiles do not hide; two waves of a SIMD hide each other's.
// 1.5B down (24 groups of 4 tiles, K split 8 ways), 65 / 128 rows: four waves 19.4 / 22.5 us, eight 18.1 / 20.3, with three tiles and X fetched
// four windows ahead 17.8 / 20.4 (the kernel before the ring 17.2 / 20.5).  Wider groups are better off with every W tile read once for 32 rows: 7B gate/up,
// ten tiles, 77.6 / 84.6 and 81.1 / 87.5.
inline bool ring_eight_waves(bool lm_head, int M, int ct) { return M > 64 && (lm_head || ct <= 5); }

// Column tiles per workgroup of a product of M rows with n_tiles tiles (gate/up 8 + 8 columns each, else 16) over n_win windows, K split
// ks ways: the least estimated time.  A window of a workgroup takes the longest of
//   its matrix instructions   60.5 ns for each column tile and row block of a SIMD (six of 16 cycles and what lies between them, at the 1.8 GHz that this
//                             load leaves; ten tiles at 128 rows are 20 of them, 1.21 us)
//   its loads                 45 bytes/ns into one CU, W at 24.5 of them (6.3 TB/s over 256 CUs); the kernels that fetch as much X as W (24 .. 61 rows)
//                             were seen at 31 .. 35
//   its dependent steps       0.45 us; above 64 rows 0.6, or 1.0 where X is requested only one window ahead
inline int plan_ring(bool lm_head, int M, int n_tiles, int n_win, int ks, int n_cu) {
    static const int ct_layer[] = {14, 13, 10, 9, 8, 7, 6, 5, 4, 3, 0}, ct_lm[] = {13, 10, 8, 6, 4, 2, 1, 0};
    const int simd_blocks = M > 64 ? 2 : 1, cs = ring_column_splits(M), blocks = (M + 15) / 16;
    int best = 0;
    double least = 1e30;
    for (const int *c = lm_head ? ct_lm : ct_layer; *c; ++c) {
        const int ct = *c, groups = (n_tiles + ct - 1) / ct;
        if (ct == 3 && M <= 64) continue;
        const int units = groups * ks, rounds = (units + n_cu - 1) / n_cu;
        const double kb = 2.048 * ct, mfma = 0.0605 * ((ct + cs - 1) / cs) * simd_blocks, load = (kb + 4.096 * blocks) / 45, w = kb / 24.5;
        double win = M > 64 ? (ct > 10 ? 1.0 : 0.6) : 0.45;
        for (double t : {mfma, load, w}) win = t > win ? t : win;
        const double us = rounds * ((n_win + ks - 1) / ks) * win;
        if (us < least + 1e-9) { least = us; best = ct; }                               // (equal: the smaller groups)
    }
    return best;
}

// Which products take k_gemm_ring.  More than 16 rows: those whose workgroups fill at least 70 % of their rounds of the machine (1.5B
// shape, 29 rows, QKV of 6 MB would take 5.4 us in place of 7.3, but with one sum in the place of four).
// Up to 16 rows: matrices from 64 MB on, because a workgroup that fills a CU starts and ends more slowly than the small ones of k_gemm_rows, and of
// these the ones that k_gemm_rows does not spread evenly.  It has all of two or three workgroups a CU resident at once, so where every CU gets nearly
// as many it streams as well as the ring and starts sooner; where some get one more than others they are what the rest waits for.
// Above 4 rows its workgroups pull X in blocks of 8 and 16, and K split over ring workgroups of six tiles and 33 windows or more is as good or better
// all the same (7B calls, six layers, spans of 3 / 4 / 5 / 8 rows, down on k_gemm_rows 885.8 914.5 926.5 937.3 us, on the ring 886.1 915.6 925.2 935.9).
// Measured, us at 3 / 8 / 16 rows, k_gemm_rows (workgroups a CU) and k_gemm_ring:
//   even    14B QKV  73 MB (1.75)  15.8 17.0 19.6 and 19.8 19.9 20.6;  7B down 136 MB (1.75)  25.5 26.4 26.9 and 26.0 26.3 26.1;
//           width 3072 gate/up 101 MB (2)  19.2 19.6 21.6 and 22.6 22.7 23.2;  width 8192 O 134 MB (2)  31.9 32.0 32.8 and 36.3 36.0 37.0;
//           width 4096 gate/up 235 MB (1.75)  45.5 46.2 47.9 and 50.2 50.7 50.9;  width 6144 down 201 MB (3)  46.5 45.7 46.7 and 45.6 46.5 48.1
//   uneven  7B gate/up 272 MB (2.3)  52.0 52.4 52.6 and 45.4 45.4 43.4;  14B gate/up 283 MB (3.4)  54.0 56.2 64.1 and 47.6 47.5 47.8;
//           14B down 142 MB (2.5)  27.9 28.6 30.4 and 26.1 26.6 26.8;  width 2560 down 71 MB (1.25)  16.6 17.5 19.3 and 16.1 16.7 17.0
//   below   14B O 52 MB (2.5)  12.3 13.5 15.3 and 13.4 13.8 14.2;  1.5B gate/up 55 MB (2.2), 5 / 8 / 16 rows  14.2 14.3 16.3 and 14.6 14.6 14.1
inline bool ring_layer(int n_cu, int rows, bool gateup, int n_out, int K) {
    const int n_tiles = (n_out + 15) / 16, n_win = K / GEMM_KW;
    if (rows > 16) return split_many(gateup, n_tiles, n_win, n_cu).eff >= 0.7;
    if ((size_t)n_out * (gateup ? 2 : 1) * K * 2 < ((size_t)64 << 20)) return false;
    const int r = gateup ? rows_tiles_whole(n_tiles, n_cu) : rows_tiles(true, n_win), ks = gateup ? 1 : split_few(true, n_tiles, n_win, n_cu);
    const int units = (n_tiles + r - 1) / r * ks, most = (units + n_cu - 1) / n_cu;
    const bool even = (most == 2 || most == 3) && 8 * units >= 7 * n_cu * most;
    return !even || (rows > 4 && !gateup && n_win / ks > 32 && n_tiles * ks >= 6 * n_cu);
}
// LM head: from five column tiles per CU on (a window of fewer costs its dependent steps: vocabulary 8192, one row of the 1.5B shape 12.7 us
// on k_gemm_rows, 16.0 here; 32 000 entries 22.6 and 21.7, 152 064 81.6 and 77.5) and for more than 16 sequences.
inline bool ring_lm_head(int n_cu, int n_seqs, int vocab) { return n_seqs > 16 || (vocab + 15) / 16 >= 5 * n_cu; }

// k_down_direct, rows of W per tile for two to four token rows (mp = 2 or 4 slots) on models up to 2048 wide.  A tile of r rows pulls r rows of W (2 bytes a
// value) and every row of x (4 bytes), r + 2 mp shares; tiles of three read x less often, tiles of two spread better over the CUs where one or two a CU are
// all there are.  So: three where the CU with the most tiles pulls less that way.  us a layer (24 layers, K four times the width), two / three-row tiles:
//   two better    896  2 rows 37.9 and 38.2, 4 rows 45.9 and 47.0;  1024  36.1 and 36.8, 44.6 and 45.2;  256  30.6 and 30.6, 37.6 and 38.3;  512, 3 rows 37.2 and 37.8
//   three better  640, 3 rows 42.6 and 42.2;  768  43.4 and 43.0;  1152, 2 rows 44.9 and 44.4, 4 rows 57.3 and 55.9;  1536  40.4 and 40.0, 50.9 and 49.1;
//                 1920  61.9 and 58.9, 77.5 and 72.8;  2048  56.5 and 55.1, 70.5 and 69.2
inline int down_tile_rows(int d_model, int mp, int n_cu) {
    const auto most = [&](int r) { return ((d_model + r - 1) / r + n_cu - 1) / n_cu * (r + 2 * mp); };
    return most(3) < most(2) ? 3 : 2;
}

}  // namespace rs
