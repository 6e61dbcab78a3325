// Arithmetic of the walked attention's work split, shared by the kernels and the host launcher.  Plain C++ without HIP
// types, so that it can also be compiled and checked on a CPU.
#pragma once

#ifdef __HIPCC__
#define RS_HD __host__ __device__ __forceinline__
#else
#define RS_HD inline
#endif

namespace rs {

constexpr int ATT_BT = 64;        // positions per workgroup and pass
constexpr int ATT_SMAX = 192;     // context slices, at most (a multiple of 64: the merge gives each lane ATT_SMAX / 64 of them)

// positions per context slice when S slices share n positions: whole 64-position passes
RS_HD int attn_slice_len(int n, int S) { return ((n + S - 1) / S + ATT_BT - 1) / ATT_BT * ATT_BT; }

// Start of the pass that is requested while the pass at t0 (of a slice that ends before t_end) is multiplied.  It stays on
// the slice's grid of whole passes: V pieces are 16-byte loads of 8 positions, which are aligned only at starts that are a
// multiple of 8.  The last pass requests itself once more (its lines are in the cache; the values are not used).
RS_HD int walk_next_pass(int t0, int t_end) { return t0 + ATT_BT < t_end ? t0 + ATT_BT : t0; }

// ------------------------------------------------------------------------------------------------
// Split of a call's attention into the pieces that workgroups of k_attn_walk take: a piece is one slice of the context of
// one group of row slots (four slots of 16 / G rows of one sequence) for one KV head.
//   fixed  one sequence, or a decode step on a short cache that one slice per sequence fills the machine with: S slices
//          divide the longest context of the call, the grid is slices x KV heads x groups
//   list   several sequences: their rows and contexts are known on the device only, so the row-table kernel
//          picks one slice length for the call and lists the pieces that exist.  What a workgroup walks is then bounded by
//          about twice the average share whatever the contexts and spans are.  (A fixed grid has to assume that any sequence
//          has the longest span there can be and the longest context: 32 sequences of 2 rows, one at 4500 positions and the
//          rest at 300, became one slice of 71 passes.  Attention of a layer on the 7B shape, us, for one pass per
//          workgroup / fixed grid / list: those 53 / 112 / 20; 128 decode rows, one at 10000 148 / 161 / 33; 20 x 5 rows up to 9163
//          141 / 230 / 48; 16 x 8 rows at 4000 135 / 119 / 51; 16 decode rows at 4500 54 / 33 / 33.)
// ------------------------------------------------------------------------------------------------
constexpr int WALK_SLOTS_MAX = 512;           // workgroups per KV head that a list aims at, at most
constexpr int WALK_GROUPS_MAX = 128;          // groups of row slots in a call (each has a row)
constexpr int WALK_FIXED_PASSES = 16;         // longest cache, in passes, whose decode steps keep one slice per sequence
constexpr int WALK_TRIES = 9;                 // slice lengths a list is tried with

struct WalkPlan {
    int walk;                     // k_attn_walk at all
    int share;                    // every sequence has one row slot: the waves of a workgroup share it
    int list;                     // pieces from the device
    int direct;                   // one slice for every row: no merge follows
    int slices;                   // records per row and head, at most
    int groups;                   // groups of row slots: of one sequence (fixed), of the call at most (list)
    int slots;                    // list: workgroups per KV head in one round of the machine
    int pieces;                   // list: entries, at most
    int few;                      // list: rows are expected to have few slices, see plan_walk
};

// n_splits: slices that the record buffer holds for a row
inline WalkPlan plan_walk(int n_rows, int n_seqs, int n_kv, int heads_per_kv, int max_ctx, int n_splits, int n_cu) {
    WalkPlan p{};
    const int rp = 16 / heads_per_kv, one_pass = (max_ctx + ATT_BT - 1) / ATT_BT;
    const int max_slots = (n_rows - n_seqs + 1 + rp - 1) / rp;               // row slots of the longest span there can be
    const int seq_groups = (max_slots + 3) / 4;
    const long base = (long)n_kv * n_seqs * seq_groups;
    // Walk or one pass per workgroup.  While a launch of one-pass workgroups is about one round of the machine, one pass is
    // the shorter chain (1.5B shape, 2 rows: 5.5 us against 6.2; 7B, 2 / 5 rows, 288 workgroups: 6.2 / 8.3 against 8.1 / 9.5); beyond that
    // the walk re-uses its row state, leaves fewer records and needs fewer prologues (7B: 9 rows, 576 workgroups: 10.6 against
    // 13.6; 16 rows 12.0 against 15.7; 8 sequences at 4400 positions 17.6 against 22.1; 14B, 2 rows at 9000: 11.9 against 14.8).
    p.walk = n_rows > 1 && (n_splits < one_pass || one_pass * base > 3L * n_cu / 2);
    if (!p.walk) return p;
    p.share = max_slots == 1;
    const int most = n_splits < one_pass ? n_splits : one_pass;
    // One round of two workgroups per CU, rounded down (a few workgroups in a further round cost a whole one: 14B, 61 rows,
    // 22 / 21 slices of 48 workgroups: 61 / 53 us)
    const long S = 2L * n_cu / base;
    const bool short_direct = n_rows == n_seqs && S <= 1 && one_pass <= WALK_FIXED_PASSES;
    if (n_seqs == 1 || short_direct) {
        p.slices = (int)(S < 1 ? 1 : S < most ? S : most);
        p.groups = seq_groups;
        p.direct = n_rows == n_seqs && p.slices == 1;
        return p;
    }
    p.list = 1;
    p.groups = n_seqs + (n_rows - n_seqs) / (4 * rp);                        // a sequence of r rows has ceil(r / 4 rp)
    p.slots = 2 * n_cu / n_kv;
    if (p.slots < 1) p.slots = 1;
    if (p.slots > WALK_SLOTS_MAX) p.slots = WALK_SLOTS_MAX;
    p.pieces = p.slots + p.groups;
    // A row has about slots / groups slices.  Up to 32 a wave per row and head merges them, at most 64; from there on a workgroup
    // per half head is better off (attention of 1.5B decode steps at 9000 positions, 2 / 4 sequences: 18.0 / 19.6 us with waves, 14.6 /
    // 17.2 with workgroups; 7B, 8 sequences of 16 slices: 22.8 with waves).
    p.few = p.slots < 32 * p.groups;
    p.slices = most < (p.few ? 64 : ATT_SMAX) ? most : p.few ? 64 : ATT_SMAX;
    return p;
}

// Calls of spans that do not walk take k_attn_span, one 64-position pass per workgroup.  As it schedules best, its registers fill a
// SIMD and a CU holds one workgroup, so that a launch with more workgroups than CUs has a second turn.  Few rows that fit one
// row slot per sequence are short enough for that turn to show; they take a build of which a CU holds two (six layers, contexts of
// 0.2 / 0.8 / 1.0 of the cache, one / two workgroups per CU, us: 7B, 2 rows, 288 workgroups 656 / 666 / 686 and 660 / 671 / 672; 1.5B,
// 2 x 2 rows 336 / 342 / 361 and 338 / 348 / 347; workgroups past the context leave at once).  From five rows on the shared
// CU costs more than the turn (7B, 5 rows at 0.8: 773 and 783).
inline bool span_pairs(int n_rows, int n_seqs, int n_kv, int heads_per_kv, int n_splits, int n_cu) {
    return n_rows <= 4 && n_rows <= 16 / heads_per_kv * n_seqs && (long)n_splits * n_kv * n_seqs > n_cu;
}

// Passes per slice of a list, from the passes of all groups and of the longest one.  The first length gives every workgroup of a
// round its average share; sum of ceil(p / length) is then at most slots + groups.  Up to twice that length is tried
// for one that fits one round (a workgroup that starts when others end would add its whole slice).
RS_HD int walk_first_len(int total, int longest, int slots, int slices) {
    const int share = (total + slots - 1) / slots, least = (longest + slices - 1) / slices;
    const int len = share > least ? share : least;
    return len < 1 ? 1 : len;
}
RS_HD int walk_try_len(int first, int k) {
    const int len = first + k * ((first + WALK_TRIES - 2) / (WALK_TRIES - 1));
    return len < 2 * first ? len : 2 * first;
}

}  // namespace rs
