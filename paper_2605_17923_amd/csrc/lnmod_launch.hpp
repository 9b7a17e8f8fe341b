// lnmod_launch.hpp -- host-side launch interface between the C ABI (lnmod_api.cpp) and the
// translation units that instantiate the gfx950 kernels.  Plain data in, hipError_t out.
#pragma once
#include <hip/hip_runtime_api.h>
#include <stddef.h>
#include <stdint.h>

namespace lnmod {

constexpr int kNumCU = 256;            // MI355X: 8 XCDs x 32 CUs
constexpr int64_t kMaxD = 8192;

// n / d for 0 <= n < 2^31 and a d >= 1 that every division of a launch shares: the high half of one multiplication and a
// shift.  d a power of two: n >> sh.  Else, with 2^sh < d < 2^(sh+1), mul = floor(2^(32+sh) / d) + 1 is below 2^32 and
// exceeds 2^(32+sh) / d by e / d with e <= d, so the quotient's error is at most n e / (d 2^(32+sh)) <= n / 2^(32+sh) < 1 / d.
struct Divider {
    uint32_t mul = 0, keep = ~uint32_t(0), sh = 0;
    Divider() = default;
    explicit Divider(uint32_t d) {
        while (sh < 31 && d >> (sh + 1) != 0) ++sh;
        if ((d & (d - 1)) != 0) {
            mul = static_cast<uint32_t>((uint64_t{1} << (32 + sh)) / d) + 1;
            keep = 0;
        }
    }
#ifdef __HIPCC__
    __host__ __device__
#endif
    uint32_t operator()(uint32_t n) const {
        return (static_cast<uint32_t>((static_cast<uint64_t>(n) * mul) >> 32) + (n & keep)) >> sh;
    }
};

// Launch shape of a row kernel: K waves per row, VPL 16-byte chunks per lane, R rows per block and
// step, per_cu resident blocks per compute unit that the grid is sized for.
struct Shape {
    int K;
    int VPL;
    int R;
    int per_cu;
    // The tables leave these 0; they are set by a shaped call of the measurement library and, clusters and interleave,
    // by bwd_shape_within:
    int clusters = 0;      // > 0: this many clusters of blocks instead of the plan's choice
    int interleave = 0;    // 1: cluster = block index modulo the cluster count (with 8 clusters every
                           // cluster then sits on one XCD, because consecutive blocks go to the XCDs in
                           // turn); 0: consecutive blocks form a cluster (every cluster on all XCDs)
    int flat = 0;          // per-sample forward: 1 one loop over all rows of a block's region (modulation
                           // registers reloaded where the segment changes), 2 one loop per segment,
                           // 0 the launcher's choice
};

struct Problem {
    int dtype;                 // LNMOD_BF16 / LNMOD_F32
    const int32_t* cu;         // device segment offsets or nullptr (fixed length)
    int64_t nseg;              // samples or segments
    int64_t S;                 // tokens per sample when cu == nullptr
    int64_t T;                 // total tokens
    int64_t D;
    float eps;
    // Launch shape to use instead of the measured table's entry, or nullptr.  The operator entry
    // points pass nullptr, except the backward with the static workspace where the table's plan needs more
    // slots than that holds; the measurement library's shaped calls pass the caller's shape,
    // per call, so that a sweep can time candidates without any process-wide state.
    const Shape* force = nullptr;
};

// How the token rows are spread over the grid.  `clusters` groups of `nb` blocks each own one
// contiguous region of `rows_per_cluster` rows; inside its region a cluster's blocks take
// consecutive rows, so the cluster streams through one moving window of memory (HBM rewards
// few concurrent sequential streams far more than one private stream per block).  nb shrinks
// when there are many segments, because every (cluster, segment) pair costs nb reloads of the
// modulation rows (forward) or nb partial-sum slots (backward).
struct RowPlan {
    int64_t blocks;            // clusters * nb
    int64_t clusters;
    int64_t rows_per_cluster;
    int32_t nb;
};

// Clusters a forward launch with one loop per segment should use when the batch has several
// segments.  Every block restarts its software pipeline once per segment of its cluster's region
// (about 2.2 us: the modulation rows, then the first rows, arrive with nothing else in flight), so
// more clusters mean fewer segments per block, but concurrent windows cost bandwidth.  The count
// that minimises
//     stream_us * penalty(C) + (nseg / C + 1) * 2.2 us,   penalty = 1, 1.01, 1.03, 1.06, 1.10
// over C = 2, 4, 8, 16, 32 is taken, a larger C only if it wins by 2 %.  A batch of several segments
// never gets a single cluster: all its blocks would reach every boundary at the same moment and
// the whole chip would drain (fp32, D = 5120, 8 equal segments: 566 us with one cluster, 541 with
// two, 535 with four).  Measured with 2 ... 32 clusters on 24 mixed, 8, 96 and 480 equal segments
// at D = 512 ... 2048 bf16 and D = 1536, 5120 fp32: the choice is within 3 % of the best count
// except on 96 segments at D = 2048 (231 us against 221 with eight clusters).
inline int64_t pick_clusters(double stream_us, int64_t nseg) {
    if (nseg <= 1) return 1;
    const int c[] = {2, 4, 8, 16, 32};
    const double penalty[] = {1.0, 1.01, 1.03, 1.06, 1.10};
    int64_t best = 2;
    double best_t = 0.0;
    for (int i = 0; i < 5 && (i == 0 || c[i] <= nseg); ++i) {
        const double t = stream_us * penalty[i] + (static_cast<double>(nseg) / c[i] + 1.0) * 2.2;
        if (i == 0 || t < best_t * 0.98) {
            best = c[i];
            best_t = t;
        }
    }
    return best;
}

// Blocks of a launch: one per rows_per_step rows, at most max_blocks (the resident blocks wanted).
inline int64_t grid_blocks(int64_t T, int64_t max_blocks, int rows_per_step) {
    int64_t g = (T + rows_per_step - 1) / rows_per_step;
    if (g > max_blocks) g = max_blocks;
    return g < 1 ? 1 : g;
}

// g blocks in clusters of nb.
inline RowPlan make_plan(int64_t T, int64_t g, int64_t nb) {
    RowPlan p{0, 0, 1, 1};
    if (T <= 0) return p;
    int64_t clusters = (g + nb - 1) / nb;
    const int64_t rpc = (T + clusters - 1) / clusters;
    clusters = (T + rpc - 1) / rpc;
    p.blocks = clusters * nb;
    p.clusters = clusters;
    p.rows_per_cluster = rpc;
    p.nb = static_cast<int32_t>(nb);
    return p;
}

// One cluster: all blocks move through the rows together (nothing changes per segment).
inline RowPlan plan_rows(int64_t T, int64_t max_blocks, int rows_per_step) {
    const int64_t g = grid_blocks(T, max_blocks, rows_per_step);
    return make_plan(T, g, g);
}

// Forward with per-segment modulation rows: `want` clusters (see pick_clusters).
inline RowPlan plan_rows_clusters(int64_t T, int64_t nseg, int64_t max_blocks, int rows_per_step,
                                  int64_t want, int64_t forced = 0) {
    const int64_t g = grid_blocks(T, max_blocks, rows_per_step);
    if (forced > 0) return make_plan(T, g, g / forced > 0 ? g / forced : 1);
    if (nseg <= 1 || want <= 1) return make_plan(T, g, g);
    // `want` clusters of equal size (a power of two of blocks per cluster is not needed: the forward
    // keeps no slots; with 768 blocks it gave 24 clusters where 16 were wanted, 154 against 142 us on
    // 64 segments of 2048 rows at D = 1536)
    const int64_t nb = (g + want - 1) / want;
    return make_plan(T, g, nb);
}

// Fraction of the streaming time a backward launch loses when its blocks form C clusters, i.e.
// move C windows through memory at once instead of one, interpolated in log2 C.  Two measured
// tables (equal segments of about 150 000 tokens in all, slots and restarts taken out): launches of
// one block per CU (D = 5120, 256 blocks): 1.2, 2.2, 4.8, 10.7, 12.4 % at C = 2, 4, 8, 16, 32; launches
// of several small blocks per CU (D = 1536, 768 blocks): 0, 0, 2, 5, 5.5 % and 12 % at C = 768;
// extrapolated in between and beyond.
inline double cluster_penalty(int64_t C, bool one_block_per_cu) {
    static const double wide[] = {0.0, 0.012, 0.022, 0.048, 0.107, 0.124, 0.16, 0.20, 0.24, 0.27, 0.30};
    static const double narrow[] = {0.0, 0.0, 0.0, 0.02, 0.05, 0.055, 0.07, 0.09, 0.10, 0.115, 0.13};
    const double* tab = one_block_per_cu ? wide : narrow;
    if (C <= 1) return 0.0;
    if (C >= 1024) return tab[10];
    int lo = 0;
    while ((int64_t{2} << lo) <= C) ++lo;                    // 2^lo <= C < 2^(lo+1), lo <= 9
    const double frac = static_cast<double>(C - (int64_t{1} << lo)) / static_cast<double>(int64_t{1} << lo);
    return tab[lo] + (tab[lo + 1] - tab[lo]) * frac;
}

// Row plan of a backward that keeps per-(block, segment) partial-sum slots.  With several
// segments the blocks per cluster nb (a power of two) minimise
//     stream_us * cluster_penalty(C)                              windows
//   + max(0, (C + nseg) * nb * slot_rows * stream_us / T - 58 us)  slots written and read back
//   + (nseg / C + 1) * 2 us (4 us with several blocks per CU)     pipeline restarts per block
//   + (nseg - 1) * 8 us if C = 1                                  all blocks restart at once
// where slot_rows is what one slot costs in units of one row's traffic and stream_us the time
// the rows take at the streaming rate.  The first 58 us of slot traffic are free: about 128 MB of
// slots are still in the last-level cache when the second pass reads them (480 segments of 312
// rows at D = 5120: 4088 slots of 41 KB cost 8 us together with the restarts, 15 584 slots 249 us).
// A lone cluster pays for every boundary with the whole chip: all its blocks drain their
// pipelines at the same moment (3 x 75 600 rows at D = 5120: 1233 us with one cluster, 1183 with two).
inline RowPlan plan_rows_slots(int64_t T, int64_t nseg, int64_t max_blocks, int rows_per_step,
                               double stream_us, double slot_rows, int64_t forced = 0) {
    if (T <= 0) return RowPlan{0, 0, 1, 1};
    const int64_t g = grid_blocks(T, max_blocks, rows_per_step);
    int64_t nb = g;
    if (forced > 0) {
        nb = g / forced > 0 ? g / forced : 1;
    } else if (nseg > 1) {
        double best = 0.0;
        bool have = false;
        for (int64_t cand = 1; cand < 2 * g; cand *= 2) {
            if (cand > g) cand = g;                          // the last candidate: one cluster
            int64_t C = (g + cand - 1) / cand;
            const int64_t rpc = (T + C - 1) / C;
            C = (T + rpc - 1) / rpc;
            double slots_us = static_cast<double>(C + nseg) * static_cast<double>(cand) * slot_rows * stream_us /
                                  static_cast<double>(T) - 58.0;
            if (slots_us < 0.0) slots_us = 0.0;
            const bool one_per_cu = max_blocks <= kNumCU;
            const double cost = stream_us * cluster_penalty(C, one_per_cu) + slots_us +
                                (static_cast<double>(nseg) / static_cast<double>(C) + 1.0) * (one_per_cu ? 2.0 : 4.0) +
                                (C == 1 ? static_cast<double>(nseg - 1) * 8.0 : 0.0);
            if (!have || cost < best) {
                have = true;
                best = cost;
                nb = cand;
            }
            if (cand == g) break;
        }
    }
    return make_plan(T, g, nb);
}

// How a row of `nchunks` 16-byte chunks is split: K waves per row, VPL chunks per lane.  A lane
// keeps about 16 features (up to 24 when one wave can take the whole row, which needs no
// barrier at all); longer rows are shared by more waves.
struct Split {
    int K;
    int VPL;
};

inline Split choose_split(int nchunks, int dtype) {
    const int per_feat16 = dtype == 0 ? 2 : 4;          // chunks holding 16 features
    const int solo_max = dtype == 0 ? 3 : 6;            // chunks per lane a single wave may take
    const int need = (nchunks + 63) / 64;
    if (need <= solo_max) {
        int vpl = need;
        if (dtype == 1 && vpl == 5) vpl = 6;            // instantiated: 1, 2, 3, 4, 6
        return {1, vpl};
    }
    int k = (nchunks + per_feat16 * 64 - 1) / (per_feat16 * 64);
    if (k == 7) k = 8;
    return {k, per_feat16};
}

// Launch shape of the row kernels: K waves per row, VPL chunks per lane, R rows per block and step,
// per_cu resident blocks per CU.  The shape comes from a table per element type, indexed by the row length.
// The tables were measured, not derived: every instantiated (K, VPL, R, per_cu) that covers the row with at
// most 50 to 60 % padding and 3 to 16 waves per CU (short forwards: up to 24) was timed on one sample, and the
// entry is the shape with the best run (D = 1536 and 5120 on 770 MB, three times on different machines).  What
// the winners on long launches share: a wave count that is a multiple of the four SIMDs of a CU (or a single
// block of 5 or 6 waves), and 16 to 32 KB of row data in flight per CU.  Neighbouring widths do not share
// winners: an entry that is best at D = 4096 loses 28 % at D = 3584.

// Entry of a per-512-features table (index 1 ... 16; [0] is unused).  A row of at most 64 chunks
// on a single wave needs one chunk per lane whatever the first entry says.
inline Shape table_entry(const Shape (&tab)[17], int nchunks, int dtype) {
    const int per512 = dtype == 0 ? 64 : 128;
    const int cols = (nchunks + per512 - 1) / per512;
    Shape sh = tab[cols < 1 ? 1 : cols > 16 ? 16 : cols];
    if (sh.K == 1 && nchunks <= 64) sh.VPL = 1;
    return sh;
}

// The tables of the per-sample forward, the backward and the recompute backward have an entry per 256
// features, because what is best at a multiple of 512 can be far off half a step below it, where a quarter
// or a third of the lanes have no chunk (D = 768 forward on 400 MB 175 -> 135 us, 3840 165 -> 134, 4864
// 203 -> 135; backward D = 768 333 -> 221, 2304 242 -> 211, 4864 222 -> 200), and the forward wider than 6144
// features gained shapes that cover it more closely (eight waves of two chunks: 6400 199 -> 147).  Mean
// over the 32 widths of 256 features, new over old time: forward bf16 0.91, fp32 0.97; backward 0.96 and 0.98;
// recompute 0.96 and 0.98.  Entries that the sweep moved by less than 1.5 % stayed as they were.
//
// Short launches have tables of their own: a block then runs a handful of steps, so the latency of its
// first rows counts more than how the blocks' windows line up, and more, smaller blocks per CU win
// (forward on 16 and 64 MB tensors: 0.87 of the former time in the mean, fp32 0.92; D = 5120 x 1560 rows 10.6 ->
// 8.8 us, 1536 x 5208 8.8 -> 7.5; on 400 MB the same shapes lose up to 14 %).  The line is 72 MB of x: at 64 MB
// the short entry is the better one at nearly every width, at 96 MB it has lost at half of them.
constexpr int64_t kShortBytes = 72000000;
inline bool short_launch(int64_t T, int nchunks) { return T > 0 && T * nchunks * 16 <= kShortBytes; }

// Entry of a per-256-features table (index 1 ... 32; [0] is unused).
inline Shape fine_entry(const Shape (&tab)[33], int nchunks, int dtype) {
    const int per256 = dtype == 0 ? 32 : 64;
    const int cols = (nchunks + per256 - 1) / per256;
    return tab[cols < 1 ? 1 : cols > 32 ? 32 : cols];
}

// Between the short launches and the 770 MB the long tables were timed at the winners are others again at some widths, and
// at the widths between two multiples of 256 an entry timed at the multiple can be far off.  A size rule names the shape for a
// range of widths, sizes and segments; the first one that holds goes before the tables.  The shapes come from sweeps of every
// compiled shape over 1600 random problems of the plain operator, 610 of the recompute form and 1270 of the other two.  Where
// a rule ends was then looked for with 19 000 problems of its own class (x of 0.3 to 900 MB; one sample, two to four, and
// packed batches of 2 to 256 segments; widths of models and any others), each timed with and without the rule in turn;
// what was more than 2.5 % slower was timed again.  Beside each rule: the share of the table entry's time in the mean, at
// worst, and (the number of problems within its range).
constexpr int32_t kAnyMB = 2000000000;
inline bool launch_mb(int64_t T, int nchunks, int64_t lo, int64_t hi) {      // x of more than lo and at most hi MB
    const int64_t bytes = T * nchunks * 16;
    return bytes > lo * 1000000 && bytes <= hi * 1000000;
}

constexpr int64_t kAnySegs = int64_t(1) << 40;
struct SizeRule {
    int first, last;               // chunks of a row
    int32_t over, to;              // x of more than `over` and at most `to` MB
    Shape sh;
    int64_t segs_from = 0;         // samples or segments
    int64_t segs_to = kAnySegs;
    int rows_per_seg = 0;          // only where samples or segments have at least that many rows in the mean
    bool unaligned = false;        // only rows that are not whole 128-byte lines
};

// Rows that are not whole 128-byte lines (16-byte chunks, eight to a line): a wave's pieces of a row then
// share lines with their neighbours, and at a few widths that turns the order of the shapes around, so the
// entries there were timed on such rows too, at six to eleven widths of each column (the unaligned_rows lines below).
inline bool unaligned_rows(int nchunks) { return nchunks % 8 != 0; }

// The shape of the first rule that holds, or nullptr.  T: the token count if known (0: not known, no rule holds).
template <int N>
inline const Shape* size_rule(const SizeRule (&rules)[N], int nchunks, int64_t T, int64_t nseg = 0) {
    if (T <= 0) return nullptr;
    for (const SizeRule& r : rules)
        if (nchunks >= r.first && nchunks <= r.last && launch_mb(T, nchunks, r.over, r.to) && nseg >= r.segs_from &&
            nseg <= r.segs_to && T >= r.rows_per_seg * nseg && !(r.unaligned && !unaligned_rows(nchunks)))
            return &r.sh;
    return nullptr;
}

// A forward whose rows all find a block of their own takes one row per step: 366 rows at D = 2680 4.8 us
// against 5.5 with two.
inline Shape one_step(Shape sh, int64_t T) {
    if (T <= static_cast<int64_t>(kNumCU) * sh.per_cu) sh.R = 1;
    return sh;
}

// bf16 forward, short launches: the table's entry as it stands, before one_step.  (D = 5128 ... 5376: two blocks of one
// row, 0.81 to 1.0 of the time of six blocks of two rows on one sample of 8 to 65 MB.)
inline Shape fwd_short_entry(int nchunks) {
    static const Shape tab_short[33] = {
        {1, 1, 2, 16},
        {1, 1, 2, 16}, {1, 1, 2, 16}, {1, 2, 2, 16}, {1, 2, 2, 12},   // D <= 1024
        {1, 3, 1, 12}, {1, 3, 2, 8}, {2, 2, 2, 8}, {2, 2, 1, 8},   // D <= 2048
        {2, 3, 2, 6}, {2, 3, 2, 6}, {2, 3, 2, 6}, {2, 3, 2, 12},   // D <= 3072
        {4, 2, 1, 4}, {4, 2, 1, 3}, {4, 2, 2, 3}, {4, 2, 2, 2},   // D <= 4096
        {4, 3, 2, 3}, {4, 3, 1, 3}, {4, 3, 2, 3}, {4, 3, 2, 3},   // D <= 5120
        {4, 3, 1, 2}, {4, 3, 1, 3}, {4, 3, 2, 2}, {4, 3, 1, 2},   // D <= 6144
        {8, 2, 1, 2}, {8, 2, 1, 2}, {8, 2, 1, 2}, {8, 2, 1, 2},   // D <= 7168
        {8, 2, 1, 2}, {8, 2, 1, 2}, {8, 2, 1, 2}, {8, 2, 1, 2}};   // D <= 8192
    return fine_entry(tab_short, nchunks, 0);
}

// T: the token count if known (0: not known, a long launch); nseg: samples or segments (0: not known, or one).
inline Shape fwd_shape(int nchunks, int dtype, int64_t T = 0, int64_t nseg = 0) {
    if (dtype == 0) {
        static const Shape tab[33] = {
            {1, 1, 2, 16},
            {1, 1, 2, 16}, {1, 1, 2, 8}, {1, 2, 1, 12}, {1, 2, 2, 4},   // D <= 1024
            {1, 3, 1, 8}, {1, 3, 2, 4}, {2, 2, 1, 6}, {2, 2, 1, 4},   // D <= 2048
            {2, 3, 1, 4}, {2, 3, 1, 4}, {2, 3, 1, 4}, {4, 2, 1, 3},   // D <= 3072
            {4, 2, 1, 3}, {4, 2, 1, 3}, {4, 2, 1, 3}, {4, 2, 2, 1},   // D <= 4096
            {4, 3, 2, 2}, {4, 3, 1, 2}, {4, 3, 1, 2}, {5, 2, 2, 1},   // D <= 5120
            {4, 3, 1, 2}, {4, 3, 1, 2}, {4, 3, 1, 2}, {4, 3, 1, 2},   // D <= 6144
            {8, 2, 1, 2}, {8, 2, 2, 2}, {5, 3, 1, 1}, {5, 3, 1, 1},   // D <= 7168
            {8, 2, 1, 2}, {5, 3, 1, 1}, {6, 3, 1, 1}, {6, 3, 1, 1}};   // D <= 8192
        static const SizeRule rules[] = {
            {129, 160, 20, 36, {1, 3, 2, 12}, 2},    // D = 1032 ... 1280: 0.937, 1.01 (216); one sample up to 1.06, beyond 36 MB up to 1.045
            {161, 192, 20, 72, {1, 3, 2, 12}},       // D = 1288 ... 1536: 0.952, 1.01 (298)
            {353, 384, 20, 72, {2, 3, 2, 6}},        // D = 2824 ... 3072: 0.917, 1.03 (327)
            {512, 512, 24, 72, {4, 2, 1, 3}, 0, 4},  // D = 4096: 0.968, 1.04 (293); on more segments 1.00, up to 1.07
            {353, 384, 12, 20, {2, 3, 1, 6}},        // D = 2824 ... 3072: 0.898, 1.01 (324)
            {448, 448, 12, 50, {4, 2, 1, 4}},        // D = 3584: 0.964, 1.02 (290)
            {737, 767, 16, 24, {4, 3, 2, 3}},        // D = 5896 ... 6136: 0.925, 1.02 (111); one sample elsewhere up to 72 MB 1.01, up to 1.18
            {737, 767, 12, 30, {4, 3, 2, 3}, 2},     // the same: 0.94, 1.02 (89)
            {97, 108, 72, 150, {1, 2, 1, 12}},       // D = 776 ... 864: 0.889, 1.01 (229)
            {112, 112, 72, 150, {1, 2, 1, 12}},      // D = 896: 0.87, 0.92 (25); between them up to 1.05
            // D = 1544 ... 1784, unaligned: 0.967, 1.02 (312); aligned up to 1.06
            {193, 223, 72, 150, {2, 2, 2, 4}, 0, kAnySegs, 0, true},
            {545, 575, 72, 150, {4, 3, 2, 2}, 13},   // D = 4360 ... 4600: 0.923, 0.99 (110); on fewer segments 1.01, up to 1.06
            {512, 512, 72, 150, {4, 2, 1, 3}},       // D = 4096: 0.935, 1.00 (325)
            {640, 640, 72, 150, {5, 2, 1, 2}},       // D = 5120: 0.959, 1.01 (327)
            {640, 640, 150, 200, {5, 2, 1, 2}, 2},   // the same: 0.962, 1.01 (131); beyond 0.99, up to 1.03
            {384, 384, 72, 300, {2, 3, 1, 4}},       // D = 3072: 0.96, 1.00 (285); 2824 ... 3064 1.00, up to 1.11
            {481, 511, 72, 300, {4, 2, 1, 3}},       // D = 3848 ... 4088: 0.871, 1.01 (327)
            {609, 639, 72, kAnyMB, {4, 3, 1, 2}}};   // D = 4872 ... 5112: 0.709, 0.82 (327)
        if (const Shape* sh = size_rule(rules, nchunks, T, nseg)) return one_step(*sh, T);
        const int col = (nchunks + 31) / 32;
        if (short_launch(T, nchunks)) return one_step(fwd_short_entry(nchunks), T);
        // D = 2632 ... 2808: 100 MB 1 to 3 % slower, 300 MB 1 to 5 % faster; narrower (2568, 2616) 2 to 5 % slower at both
        if (unaligned_rows(nchunks) && col == 11 && nchunks > 328) return {4, 2, 1, 3};
        // D = 7432 ... 7672, 100 and 300 MB: 0.81 to 0.89 of the time
        if (unaligned_rows(nchunks) && col == 30) return {6, 3, 1, 1};
        // D = 1288 ... 1528: the entry was timed at D = 1536.  Aligned rows 0.84 to 1.01 of its time at 79, 119 and 300
        // MB; unaligned ones up to D = 1344 0.89 to 0.99 at 79 and 119 MB, beyond either 1 to 8 % slower
        if (col == 6 && nchunks != 192 &&
            (!unaligned_rows(nchunks) || (nchunks <= 168 && T * nchunks * 16 <= 150000000 && T > 0)))
            return {1, 3, 1, 8};
        // D = 1536: four blocks per CU are 4 % faster on the 32 760 rows of the Wan-1.3B workload,
        // the two tie on 65 520 rows, three are 3 % faster on 131 040 rows and 5 % on 252 000
        if (nchunks == 192) return {1, 3, 2, T >= 98304 ? 3 : 4};
        return fine_entry(tab, nchunks, dtype);
    }
    // fp32: one row per step and two blocks per CU once several waves share a row (a wave's four
    // chunks carry twice the bytes of a bf16 wave's two: 266 against 287 us on 37800 x 5120)
    static const Shape tab32[33] = {
        {1, 1, 2, 8},
        {1, 1, 2, 8}, {1, 2, 2, 8}, {1, 4, 1, 8}, {1, 4, 1, 8},   // D <= 1024
        {1, 6, 1, 6}, {1, 6, 1, 6}, {2, 4, 2, 4}, {2, 4, 2, 2},   // D <= 2048
        {3, 4, 2, 2}, {3, 4, 1, 4}, {4, 4, 1, 2}, {4, 4, 1, 2},   // D <= 3072
        {4, 4, 1, 2}, {4, 4, 1, 2}, {4, 4, 1, 2}, {4, 4, 1, 2},   // D <= 4096
        {5, 4, 1, 2}, {5, 4, 1, 2}, {5, 4, 1, 2}, {5, 4, 1, 2},   // D <= 5120
        {6, 4, 1, 2}, {8, 4, 1, 2}, {6, 4, 1, 1}, {6, 4, 1, 1},   // D <= 6144
        {8, 4, 2, 3}, {8, 4, 2, 3}, {8, 4, 2, 3}, {8, 4, 2, 3},   // D <= 7168
        {8, 4, 2, 3}, {8, 4, 2, 3}, {8, 4, 2, 3}, {8, 4, 1, 2}};   // D <= 8192
    static const Shape tab32_short[33] = {
        {1, 1, 2, 16},
        {1, 1, 2, 16}, {1, 2, 2, 8}, {1, 3, 2, 8}, {1, 4, 2, 12},   // D <= 1024
        {1, 6, 2, 8}, {1, 6, 2, 8}, {2, 4, 2, 12}, {2, 4, 2, 6},   // D <= 2048
        {3, 4, 2, 4}, {3, 4, 2, 8}, {4, 4, 1, 4}, {3, 4, 2, 3},   // D <= 3072
        {4, 4, 1, 3}, {4, 4, 1, 3}, {4, 4, 1, 3}, {4, 4, 1, 2},   // D <= 4096
        {5, 4, 1, 2}, {5, 4, 1, 2}, {5, 4, 1, 2}, {5, 4, 1, 2},   // D <= 5120
        {6, 4, 1, 2}, {6, 4, 1, 2}, {6, 4, 1, 2}, {6, 4, 1, 2},   // D <= 6144
        {8, 4, 1, 1}, {8, 4, 2, 1}, {8, 4, 2, 1}, {8, 4, 1, 1},   // D <= 7168
        {8, 4, 1, 1}, {8, 4, 2, 1}, {8, 4, 2, 2}, {8, 4, 2, 2}};   // D <= 8192
    static const SizeRule rules32[] = {
        {577, 640, 12, 72, {3, 4, 2, 3}},            // D = 2308 ... 2560: 0.888, 1.02 (236)
        {1536, 1536, 20, 72, {6, 4, 2, 1}, 6}};      // D = 6144: 0.942, 1.02 (65); on one to four samples 1.04, up to 1.21
    if (const Shape* sh = size_rule(rules32, nchunks, T, nseg)) return one_step(*sh, T);
    if (short_launch(T, nchunks)) return one_step(fine_entry(tab32_short, nchunks, dtype), T);
    return fine_entry(tab32, nchunks, dtype);
}

constexpr int64_t kNarrowBwdBytes = 40000000;        // the line of the backward at D = 264 ... 504, below

// Size rules of the backwards.  Their shapes all count in bwd_most_slots_one_sample.
constexpr SizeRule kBwdRules[] = {
    {131, 159, 0, 1, {3, 1, 2, 2}, 0, 1},        // D = 1048 ... 1272: 0.944, 1.01 (116)
    {131, 159, 1, 20, {3, 1, 2, 2}},             // the same: 0.869, 1.06 (292)
    {609, 640, 6, 20, {8, 2, 1, 1}},             // D = 4872 ... 5120: 0.978, 1.06 (229); below 1.01, up to 1.21
    {97, 127, 20, 24, {1, 2, 2, 4}, 9},          // D = 776 ... 1016: 0.949, 1.03 (70); on fewer segments up to 1.07
    {97, 127, 24, 72, {1, 2, 2, 4}},             // the same: 0.938, 1.04 (302)
    {257, 287, 40, 72, {5, 1, 2, 2}},            // D = 2056 ... 2296: 0.935, 1.08 (233); below 0.99, up to 1.09
    {97, 127, 72, 150, {1, 2, 2, 6}},            // D = 776 ... 1016: 0.875, 1.03 (327)
    // D = 3584: 0.932, 1.02 (325); on segments of fewer than 512 rows in the mean up to 1.09
    {448, 448, 72, 300, {8, 1, 2, 1}, 0, kAnySegs, 512},
    {640, 640, 72, 300, {5, 2, 2, 1}},           // D = 5120: 0.981, 1.01 (326)
    {97, 127, 150, kAnyMB, {1, 2, 2, 4}, 0, 80},     // D = 776 ... 1016: 0.843, 1.08 (257); on more segments 0.92, up to 1.10
    // D = 1288 ... 1528, unaligned: 0.93, 1.04 (209); aligned 1.03, up to 1.08, more segments 0.98, up to 1.10
    {161, 191, 72, kAnyMB, {3, 1, 2, 3}, 0, 4, 0, true},
    {417, 447, 72, 500, {8, 1, 2, 1}, 0, kAnySegs, 700},     // D = 3336 ... 3576: 0.941, 1.03 (281); beyond 0.97, up to 1.05
    {609, 639, 72, kAnyMB, {6, 2, 2, 1}},        // D = 4872 ... 5112: 0.954, 1.00 (327)
    {768, 768, 72, kAnyMB, {8, 2, 1, 1}}};       // D = 6144: 0.976, 1.02 (327)
constexpr SizeRule kBwdRules32[] = {
    {129, 159, 80, 300, {1, 3, 2, 4}},           // D = 516 ... 636: 0.875, 1.07 (238)
    {160, 191, 80, 300, {1, 3, 2, 4}, 0, 4}};    // D = 640 ... 764: 0.937, 1.03 (155); on more segments up to 1.27, and at 75 MB 1.06
// Without saved statistics.  Up to 20 MB a block has one to four steps: one chunk per lane and one block per CU halve the
// slots and shorten the chain of the first row.
constexpr SizeRule kRcBwdRules[] = {
    {161, 192, 0, 20, {3, 1, 2, 2}},             // D = 1288 ... 1536: 0.895, 1.04 (325)
    {256, 256, 0, 1, {4, 1, 2, 1}, 0, 1},        // D = 2048: 0.98, 1.02 (94); several samples 1.03, up to 1.12
    {256, 256, 1, 20, {4, 1, 2, 1}},             // the same: 0.789, 1.06 (293)
    {193, 255, 0, 1, {4, 1, 2, 2}, 0, 1},        // D = 1544 ... 2040: 0.957, 1.01 (123); several samples 1.00, up to 1.11
    {193, 255, 1, 20, {4, 1, 2, 2}},             // the same: 0.819, 1.02 (294)
    {320, 320, 0, 1, {5, 1, 1, 1}},              // D = 2560: 0.894, 1.01 (137)
    {320, 320, 2, 20, {5, 1, 1, 1}},             // the same: 0.889, 1.07 (271); between them 0.98, up to 1.07
    {257, 319, 0, 1, {5, 1, 1, 2}},              // D = 2056 ... 2552: 0.923, 1.03 (158)
    {257, 319, 5, 20, {5, 1, 1, 2}},             // the same: 0.911, 1.02 (237); between them 1.04, up to 1.20
    {321, 383, 0, 12, {6, 1, 2, 1}},             // D = 2568 ... 3064: 0.934, 1.04 (216); beyond 1.02, up to 1.12
    {384, 384, 0, 2, {6, 1, 2, 1}},              // D = 3072: 0.963, 1.06 (178)
    {384, 384, 4, 12, {6, 1, 2, 1}},             // the same: 0.886, 1.05 (153)
    {384, 384, 12, 16, {6, 1, 2, 1}, 0, 4},      // the same: 0.957, 1.02 (36); elsewhere 1.00, up to 1.22
    {417, 448, 2, 14, {8, 1, 2, 1}},             // D = 3336 ... 3584: 0.807, 0.99 (249); below 1.01, up to 1.24
    {417, 448, 14, 20, {8, 1, 2, 1}, 0, 8},      // the same: 0.923, 1.03 (177); on more segments up to 1.12
    {513, 704, 2, 20, {4, 3, 1, 1}, 0, 8},       // D = 4104 ... 5632: 0.904, 1.05 (316); on more segments 1.03, up to 1.10
    {705, 767, 8, 20, {4, 3, 1, 1}},             // D = 5640 ... 6136: 0.95, 1.01 (170); below up to 1.21
    {65, 96, 36, 50, {1, 2, 2, 8}, 2},           // D = 520 ... 768: 0.935, 1.04 (161); one sample 1.01, up to 1.08
    {65, 96, 50, 72, {1, 2, 2, 8}},              // the same: 0.93, 1.02 (245)
    {193, 255, 20, 50, {4, 1, 2, 2}},            // D = 1544 ... 2040: 0.946, 1.06 (216); beyond 1.02, up to 1.08
    {256, 256, 20, 72, {4, 1, 2, 2}},            // D = 2048: 0.882, 1.03 (259)
    {256, 256, 72, 150, {4, 1, 2, 2}, 0, 64},    // the same: 0.957, 1.00 (322); on more segments 1.01, up to 1.05
    {97, 127, 80, 300, {1, 2, 1, 8}},            // D = 776 ... 1016: 0.948, 1.06 (312)
    {481, 511, 80, 300, {4, 2, 1, 2}}};          // D = 3848 ... 4088: 0.925, 1.03 (312)

// The tables, without the size rules.
inline Shape bwd_table(int nchunks, int dtype, int64_t T) {
    if (dtype == 0) {
        static const Shape tab[33] = {
            {1, 1, 2, 8},
            {1, 1, 2, 8}, {1, 1, 1, 8}, {1, 2, 2, 8}, {1, 2, 2, 3},   // D <= 1024
            {3, 1, 1, 4}, {3, 1, 1, 4}, {4, 1, 2, 3}, {4, 1, 2, 2},   // D <= 2048
            {5, 1, 2, 2}, {5, 1, 2, 2}, {3, 2, 1, 2}, {6, 1, 2, 1},   // D <= 3072
            {8, 1, 2, 1}, {4, 2, 1, 3}, {4, 2, 2, 1}, {4, 2, 2, 1},   // D <= 4096
            {5, 2, 2, 1}, {5, 2, 2, 1}, {6, 2, 2, 1}, {4, 3, 2, 1},   // D <= 5120
            {8, 2, 2, 1}, {6, 2, 1, 1}, {6, 2, 1, 1}, {4, 3, 2, 1},   // D <= 6144
            {8, 2, 1, 1}, {8, 2, 1, 1}, {6, 3, 2, 1}, {6, 3, 2, 1},   // D <= 7168
            {6, 3, 2, 1}, {6, 3, 2, 1}, {6, 3, 2, 1}, {6, 3, 2, 1}};   // D <= 8192
        static const Shape tab_short[33] = {
            {1, 1, 2, 8},
            {1, 1, 2, 8}, {1, 1, 2, 4}, {1, 2, 2, 4}, {1, 2, 2, 3},   // D <= 1024
            {3, 1, 1, 4}, {3, 1, 2, 2}, {4, 1, 2, 2}, {4, 1, 2, 2},   // D <= 2048
            {5, 1, 2, 1}, {5, 1, 2, 1}, {6, 1, 2, 1}, {6, 1, 2, 1},   // D <= 3072
            {8, 1, 2, 1}, {8, 1, 2, 1}, {8, 1, 2, 1}, {8, 1, 1, 1},   // D <= 4096
            {6, 2, 1, 1}, {6, 2, 1, 1}, {5, 2, 2, 1}, {5, 2, 2, 1},   // D <= 5120
            {6, 2, 1, 1}, {8, 2, 1, 1}, {8, 2, 1, 1}, {8, 2, 1, 1},   // D <= 6144
            {8, 2, 1, 1}, {8, 2, 1, 1}, {8, 2, 1, 1}, {8, 2, 1, 1},   // D <= 7168
            {8, 2, 1, 1}, {8, 2, 1, 1}, {8, 2, 2, 1}, {8, 2, 2, 1}};   // D <= 8192
        // D = 264 ... 504 from 40 MB on: the entries were timed at D = 512, where every lane has a chunk (89 and 250 MB:
        // D = 264 80.5 us against 94.5, 190 against 236; 440 153 against 167; 28 MB 32.6 against 30.4)
        if (nchunks > 32 && nchunks < 64 && (T == 0 || T * nchunks * 16 > kNarrowBwdBytes)) return {1, 1, 2, 8};
        if (short_launch(T, nchunks)) return fine_entry(tab_short, nchunks, dtype);
        if (unaligned_rows(nchunks)) {
            const int col = (nchunks + 31) / 32;
            // six widths of each column, 100 and 300 MB, as a share of the entry's time
            if (col == 11) return {6, 1, 2, 1};                              // D = 2568 ... 2808: 0.91 ... 1.0
            if (col == 21) return {6, 2, 1, 1};                              // D = 5128 ... 5368: 0.96 ... 1.0
            if (col == 23) return {4, 3, 2, 1};                              // D = 5640 ... 5880: 0.94 ... 0.99 at 300 MB, 0.99 ... 1.04 at 100
        }
        if (nchunks == 192) return {3, 1, 1, 3};
        return fine_entry(tab, nchunks, dtype);
    }
    // fp32, rows of 1 KB and more: mostly one row per step (a wave's four chunks of one row are as
    // many bytes as two bf16 rows) and, for the wide rows, more waves than the chunks need
    static const Shape tab32[33] = {
        {1, 1, 1, 8},
        {1, 1, 1, 8}, {1, 2, 2, 3}, {1, 4, 1, 3}, {1, 4, 1, 3},   // D <= 1024
        {2, 4, 2, 2}, {2, 4, 1, 2}, {2, 4, 1, 3}, {2, 4, 1, 2},   // D <= 2048
        {3, 4, 2, 1}, {3, 4, 2, 1}, {4, 4, 1, 1}, {4, 4, 1, 1},   // D <= 3072
        {5, 4, 2, 1}, {5, 4, 2, 1}, {5, 4, 2, 1}, {6, 4, 1, 1},   // D <= 4096
        {6, 4, 1, 1}, {6, 4, 1, 1}, {6, 4, 1, 1}, {6, 4, 1, 1},   // D <= 5120
        {6, 4, 1, 1}, {6, 4, 1, 1}, {6, 4, 1, 1}, {8, 4, 1, 1},   // D <= 6144
        {8, 4, 1, 1}, {8, 4, 1, 1}, {8, 4, 1, 1}, {8, 4, 1, 1},   // D <= 7168
        {8, 4, 1, 1}, {8, 4, 1, 1}, {8, 4, 1, 1}, {8, 4, 1, 1}};   // D <= 8192
    static const Shape tab32_short[33] = {
        {1, 1, 2, 6},
        {1, 1, 2, 6}, {1, 2, 2, 3}, {1, 3, 2, 3}, {1, 4, 1, 3},   // D <= 1024
        {2, 4, 1, 2}, {2, 4, 1, 2}, {2, 4, 1, 2}, {3, 4, 2, 1},   // D <= 2048
        {3, 4, 2, 1}, {3, 4, 2, 1}, {4, 4, 1, 1}, {4, 4, 1, 1},   // D <= 3072
        {5, 4, 2, 1}, {5, 4, 1, 1}, {5, 4, 1, 1}, {4, 4, 2, 1},   // D <= 4096
        {6, 4, 1, 1}, {6, 4, 2, 1}, {6, 4, 1, 1}, {6, 4, 1, 1},   // D <= 5120
        {6, 4, 1, 1}, {6, 4, 1, 1}, {6, 4, 1, 1}, {6, 4, 2, 1},   // D <= 6144
        {8, 4, 1, 1}, {8, 4, 1, 1}, {8, 4, 1, 1}, {8, 4, 1, 1},   // D <= 7168
        {8, 4, 1, 1}, {8, 4, 1, 1}, {8, 4, 1, 1}, {8, 4, 2, 1}};   // D <= 8192
    return short_launch(T, nchunks) ? fine_entry(tab32_short, nchunks, dtype) : fine_entry(tab32, nchunks, dtype);
}

// nseg: samples or segments if known (0: not known, or one).
inline Shape bwd_shape(int nchunks, int dtype, int64_t T = 0, int64_t nseg = 0) {
    const Shape* sh = dtype == 0 ? size_rule(kBwdRules, nchunks, T, nseg) : size_rule(kBwdRules32, nchunks, T, nseg);
    return sh ? *sh : bwd_table(nchunks, dtype, T);
}

// Backward that forms the statistics again from x.  It has one more dependent chain per step
// (per-wave mean, four wave sums, the merge with a division and a square root), which fewer waves per
// row with more chunks each, or two blocks per CU, hide better than the shapes above; it runs 2 to 20 %
// behind the backward that reads the saved statistics (D = 5120: 14 %).
inline Shape rc_bwd_table(int nchunks, int dtype, int64_t T) {
    if (dtype == 0) {
        static const Shape tab[33] = {
            {1, 1, 2, 8},
            {1, 1, 2, 8}, {1, 1, 1, 8}, {1, 2, 2, 8}, {1, 2, 2, 4},   // D <= 1024
            {1, 3, 1, 8}, {1, 3, 2, 4}, {2, 2, 1, 6}, {2, 2, 1, 4},   // D <= 2048
            {3, 2, 2, 3}, {3, 2, 2, 3}, {3, 2, 2, 3}, {3, 2, 2, 2},   // D <= 3072
            {4, 2, 1, 3}, {4, 2, 1, 3}, {4, 2, 1, 3}, {4, 2, 2, 1},   // D <= 4096
            {4, 3, 1, 2}, {4, 3, 1, 2}, {4, 3, 1, 2}, {4, 3, 1, 2},   // D <= 5120
            {4, 3, 1, 2}, {4, 3, 1, 2}, {4, 3, 1, 2}, {4, 3, 2, 1},   // D <= 6144
            {8, 2, 2, 1}, {8, 2, 2, 1}, {8, 2, 2, 1}, {8, 2, 2, 1},   // D <= 7168
            {8, 2, 2, 1}, {8, 2, 2, 1}, {8, 2, 2, 1}, {8, 2, 2, 1}};   // D <= 8192
        // short launches: per 512 features (three samples of 2000 rows at D = 768: 18.4 us against 21.9)
        static const Shape tab_short[17] = {
            {1, 1, 2, 8},
            {1, 1, 2, 8}, {1, 2, 2, 4}, {1, 3, 2, 4}, {2, 2, 1, 4},
            {3, 2, 2, 3}, {3, 2, 2, 2}, {4, 2, 1, 3}, {4, 2, 2, 1},
            {4, 3, 1, 2}, {4, 3, 1, 2}, {4, 3, 1, 2}, {4, 3, 2, 1},
            {8, 2, 1, 2}, {8, 2, 2, 1}, {8, 2, 2, 1}, {8, 2, 2, 1}};
        if (short_launch(T, nchunks)) return table_entry(tab_short, nchunks, dtype);
        if (nchunks > 32 && nchunks < 64) return {1, 1, 2, 8};       // D = 264 ... 504: 0.97 in the mean, 264 258 against 281 us
        return fine_entry(tab, nchunks, dtype);
    }
    static const Shape tab32[33] = {
        {1, 1, 1, 8},
        {1, 1, 1, 8}, {1, 2, 2, 3}, {1, 4, 1, 4}, {1, 6, 1, 3},   // D <= 1024
        {2, 4, 1, 4}, {2, 4, 1, 3}, {2, 4, 1, 3}, {3, 4, 1, 2},   // D <= 2048
        {3, 4, 1, 2}, {3, 4, 2, 1}, {4, 4, 1, 1}, {4, 4, 1, 1},   // D <= 3072
        {4, 4, 1, 1}, {5, 4, 2, 1}, {5, 4, 2, 1}, {5, 4, 2, 1},   // D <= 4096
        {6, 4, 1, 1}, {6, 4, 1, 1}, {6, 4, 1, 1}, {6, 4, 1, 1},   // D <= 5120
        {6, 4, 1, 1}, {6, 4, 1, 1}, {8, 4, 1, 1}, {8, 4, 1, 1},   // D <= 6144
        {8, 4, 1, 1}, {8, 4, 1, 1}, {8, 4, 1, 1}, {8, 4, 1, 1},   // D <= 7168
        {8, 4, 1, 1}, {8, 4, 1, 1}, {8, 4, 1, 1}, {8, 4, 1, 1}};   // D <= 8192
    return fine_entry(tab32, nchunks, dtype);
}

inline Shape rc_bwd_shape(int nchunks, int dtype, int64_t T = 0, int64_t nseg = 0) {
    const Shape* sh = dtype == 0 ? size_rule(kRcBwdRules, nchunks, T, nseg) : nullptr;
    return sh ? *sh : rc_bwd_table(nchunks, dtype, T);
}

// The table's entry, or the shape the call carries (Problem::force).  A forced shape that does not
// cover the row makes the launch fail instead of computing on part of the row.
inline Shape pick_shape(const Shape* force, Shape table) { return force ? *force : table; }
inline bool covers(const Shape& s, int nchunks) { return s.K * s.VPL * 64 >= nchunks; }

// Per-token modulation (three input streams forward; three in, three out backward).  bf16: a table
// per 512 features of the same kind, from a sweep over the (K, VPL) these kernels are
// compiled for (one wave alone, or two chunks per lane on 2 to 8 waves, or five chunks per lane on two waves).  Here too neighbours do
// not share winners: D = 2560 forward takes 526 us with {3,2,2,4} and 858 us with the {3,2,1,2}
// that is best at D = 3072.  fp32: tables of the same kind (four chunks per lane once a row is
// shared, up to six on a single wave).
inline Shape tok_fwd_shape(int nchunks, int dtype) {
    if (dtype == 0) {
        static const Shape tab[17] = {
            {1, 1, 2, 8},
            {1, 1, 2, 8}, {1, 2, 2, 4}, {1, 3, 2, 4}, {2, 2, 1, 4},
            {3, 2, 2, 4}, {3, 2, 1, 2}, {4, 2, 2, 3}, {4, 2, 1, 2},
            {5, 2, 1, 3}, {2, 5, 1, 2}, {8, 2, 1, 2}, {6, 2, 2, 2},
            {8, 2, 1, 2}, {8, 2, 1, 2}, {8, 2, 1, 2}, {8, 2, 1, 1}};
        // D = 4616 ... 5120: two waves with five chunks per lane (one wave per SIMD, 5 KB runs per wave and
        // stream, half as many waves at the barrier) take 452 us on 65 520 x 5120 where five waves with two
        // chunks take 476; the same split gained nothing in the per-token backward (750 against 730 us)
        return table_entry(tab, nchunks, dtype);
    }
    static const Shape tab32[17] = {
        {1, 2, 2, 4},
        {1, 2, 2, 4}, {1, 4, 1, 4}, {2, 4, 1, 4}, {2, 4, 2, 2},
        {3, 4, 1, 3}, {4, 4, 2, 4}, {4, 4, 1, 2}, {4, 4, 1, 1},
        {6, 4, 2, 2}, {5, 4, 1, 2}, {8, 4, 2, 2}, {6, 4, 1, 1},
        {8, 4, 1, 1}, {8, 4, 1, 1}, {8, 4, 1, 1}, {8, 4, 1, 2}};
    return table_entry(tab32, nchunks, dtype);
}

// Per-token backward that forms the statistics again from x.
inline Shape tok_rc_bwd_shape(int nchunks, int dtype) {
    if (dtype == 0) {
        static const Shape tab[17] = {
            {1, 1, 1, 6},
            {1, 1, 1, 6}, {1, 2, 2, 3}, {1, 3, 1, 3}, {2, 2, 1, 2},
            {3, 2, 1, 2}, {3, 2, 1, 2}, {4, 2, 1, 2}, {4, 2, 1, 1},
            {6, 2, 1, 2}, {5, 2, 1, 2}, {6, 2, 2, 1}, {8, 2, 2, 1},
            {8, 2, 2, 1}, {8, 2, 2, 1}, {8, 2, 1, 1}, {8, 2, 1, 1}};
        return table_entry(tab, nchunks, dtype);
    }
    static const Shape tab32[17] = {
        {1, 2, 2, 8},
        {1, 2, 2, 8}, {1, 4, 1, 8}, {2, 4, 1, 2}, {2, 4, 2, 2},
        {3, 4, 2, 1}, {3, 4, 1, 1}, {5, 4, 1, 1}, {5, 4, 1, 3},
        {5, 4, 1, 1}, {8, 4, 2, 2}, {6, 4, 1, 1}, {6, 4, 1, 1},
        {8, 4, 1, 1}, {8, 4, 1, 1}, {8, 4, 1, 1}, {8, 4, 1, 2}};
    return table_entry(tab32, nchunks, dtype);
}

// Per-token backward with saved statistics.  writes_dshift: whether the copy of dy goes out (six streams) or not
// (five).  Both take the same waves and chunks per lane at a width, so that they add a row in the same order; rows
// per step and blocks per CU differ where that measured better, and on launches of up to 32 Mi elements.  From a
// sweep of both at every multiple of 512 features on 400 MB and 48 MB tensors; against the former table, six
// streams: bf16 0.98 of the time in the mean, fp32 the same (48 MB: D = 2048 0.94, 5632 0.87, 6144 0.91; slower by
// 1.4 % at 97 656 x 1536, 1.3 % at 20 926 x 7168, 4 % at 813 x 6144, 1 % or less elsewhere); five streams, 400 MB: D = 1024 354 -> 333 us, 2048 378 -> 334, 2560
// 365 -> 324, 4096 362 -> 338, 5632 372 -> 346, 6144 362 -> 337; fp32 D = 2560 356 -> 344, 3584 355 -> 339, 5120
// 358 -> 346.
inline Shape tok_bwd_shape(int nchunks, int dtype, bool writes_dshift = true, int64_t T = 0) {
    if (dtype == 0) {
        static const Shape six[17] = {
            {1, 1, 1, 6},
            {1, 1, 1, 6}, {1, 2, 2, 3}, {3, 1, 2, 2}, {4, 1, 1, 2},
            {8, 1, 1, 2}, {8, 1, 1, 2}, {8, 1, 1, 2}, {8, 1, 1, 1},
            {6, 2, 1, 2}, {5, 2, 1, 2}, {4, 3, 1, 2}, {4, 3, 1, 2},
            {8, 2, 2, 2}, {8, 2, 2, 2}, {8, 2, 1, 1}, {8, 2, 1, 1}};
        static const Shape five[17] = {
            {1, 1, 1, 8},
            {1, 1, 1, 8}, {1, 2, 1, 4}, {3, 1, 2, 2}, {4, 1, 1, 2},
            {8, 1, 1, 2}, {8, 1, 1, 2}, {8, 1, 1, 2}, {8, 1, 1, 1},
            {6, 2, 1, 2}, {5, 2, 1, 2}, {4, 3, 1, 2}, {4, 3, 1, 2},
            {8, 2, 2, 2}, {8, 2, 2, 1}, {8, 2, 2, 1}, {8, 2, 1, 1}};
        static const Shape five_short[17] = {
            {1, 1, 1, 8},
            {1, 1, 1, 8}, {1, 2, 1, 8}, {3, 1, 1, 4}, {4, 1, 1, 3},
            {8, 1, 1, 2}, {8, 1, 1, 2}, {8, 1, 1, 2}, {8, 1, 1, 2},
            {6, 2, 1, 2}, {5, 2, 1, 2}, {4, 3, 1, 2}, {4, 3, 1, 2},
            {8, 2, 1, 2}, {8, 2, 1, 2}, {8, 2, 1, 2}, {8, 2, 1, 2}};
        const int cols = (nchunks + 63) / 64;
        const bool few = T > 0 && T * nchunks * 8 <= (int64_t(32) << 20);
        // D = 3336 ... 4088 beyond short launches (110 and 250 MB): 0.86 to 1.0 of the time with five streams, at six
        // 2 % faster to 8 % slower, but the same waves and chunks as five.  On 10 and 48 MB it lost 0 to 13 % at
        // every width from 3088 on, and below 3336 1 to 5 % at any size.
        if (unaligned_rows(nchunks) && !few && nchunks > 416 && nchunks <= 512) {
            if (!writes_dshift) return {4, 2, 2, 2};
            return {4, 2, 1, cols == 7 ? 2 : 1};
        }
        if (writes_dshift) return table_entry(six, nchunks, dtype);
        return few ? table_entry(five_short, nchunks, dtype) : table_entry(five, nchunks, dtype);
    }
    static const Shape six32[17] = {
        {1, 2, 2, 8},
        {1, 2, 2, 8}, {1, 4, 1, 8}, {2, 4, 1, 2}, {2, 4, 2, 2},
        {3, 4, 2, 1}, {3, 4, 1, 1}, {4, 4, 1, 1}, {5, 4, 1, 3},
        {5, 4, 1, 1}, {6, 4, 1, 1}, {6, 4, 1, 1}, {6, 4, 1, 1},
        {8, 4, 1, 1}, {8, 4, 1, 1}, {8, 4, 1, 1}, {8, 4, 1, 2}};
    Shape sh = table_entry(six32, nchunks, dtype);
    const int cols = (nchunks + 127) / 128;
    if (!writes_dshift && cols >= 5 && cols <= 7) {
        sh.R = 1;
        sh.per_cu = 2;
    }
    return sh;
}

// Which blocks form a cluster.  Consecutive blocks go to the eight XCDs in turn, so with
// cluster = block index modulo the cluster count (and a count that is a multiple of 8) all blocks
// of a cluster sit on one XCD and that XCD streams through one contiguous region; clusters of
// consecutive blocks are each spread over all XCDs.  Measured on packed batches (forward /
// backward us, same cluster count): 24 mixed segments at D = 5120 554 / 834 -> 550 / 828, 96 segments
// of 1560 rows 566 / 858 -> 559 / 844, 8 segments of 16 380 rows backward 687 -> 676, 64 segments of
// 2048 rows at D = 1536 forward 150 -> 146.  So every launch with more than one cluster interleaves;
// a shaped call says for itself.
inline int cluster_interleave(const Shape* force, const RowPlan& pl) {
    return force ? force->interleave : (pl.clusters > 1 ? 1 : 0);
}

// What a block's index is divided by to find its cluster and its place in it (place_of).
inline int32_t cluster_split(int interleave, const RowPlan& pl) {
    return interleave ? static_cast<int32_t>(pl.clusters) : pl.nb;
}

// Slot of (cluster c, segment m, member j) is (c + m) * nb + j with c < clusters, m < nseg.
inline int64_t bwd_slots(const RowPlan& p, int64_t nseg) {
    return nseg < 1 ? 0 : (p.clusters + nseg - 1) * p.nb;
}

// Shape and row plan of a backward launch: what the launcher uses, what sizes the workspace and
// what describe_bwd() reports.
struct BwdLaunch {
    Shape sh;
    RowPlan pl;
    int nchunks;
};

inline BwdLaunch plan_bwd(int64_t T, int64_t nseg, int64_t D, int dtype, bool per_token, bool recompute,
                          const Shape* force, bool writes_dshift = true) {
    BwdLaunch L;
    const int E = dtype == 0 ? 8 : 4;
    L.nchunks = static_cast<int>(D / E);
    if (per_token) {
        // (the recompute form keeps shapes of its own: 32 760 x 1536 98 us, 109 with the others)
        L.sh = pick_shape(force, recompute ? tok_rc_bwd_shape(L.nchunks, dtype)
                                           : tok_bwd_shape(L.nchunks, dtype, writes_dshift, T));
        L.pl = plan_rows(T, static_cast<int64_t>(kNumCU) * L.sh.per_cu, L.sh.R);
        return L;
    }
    L.sh = pick_shape(force, recompute ? rc_bwd_shape(L.nchunks, dtype, T, nseg)
                                       : bwd_shape(L.nchunks, dtype, T, nseg));
    // a row moves 3 D elements (dy, x, dx), a slot 2 D floats that are written and read back
    const double elem = dtype == 0 ? 2.0 : 4.0;
    const double stream_us = static_cast<double>(T) * static_cast<double>(D) * 3.0 * elem / 5.8e6;
    L.pl = plan_rows_slots(T, nseg, static_cast<int64_t>(kNumCU) * L.sh.per_cu, L.sh.R, stream_us,
                           16.0 / (3.0 * elem), L.sh.clusters);
    return L;
}

// The backward's plan for this problem: the same function sizes the workspace, drives the main
// kernel's grid and tells the second pass which partial-sum slots belong to a segment.
inline RowPlan bwd_plan(int64_t T, int64_t nseg, int64_t D, int dtype, bool recompute, const Shape* force = nullptr) {
    return plan_bwd(T, nseg, D, dtype, false, recompute, force).pl;
}

// Slots of this backward on one sample of T rows with the shape that has most of them at this width, whatever the size:
// a bound on the plan's slots that does not fall as T grows.  These are all the shapes a width can get: the tables' for
// short and long launches and between them for one beyond kNarrowBwdBytes, and those of its size rules.
inline int64_t bwd_most_slots_one_sample(int64_t T, int64_t D, int dtype, bool recompute) {
    if (T <= 0) return 0;
    const int nchunks = static_cast<int>(D / (dtype == 0 ? 8 : 4));
    int64_t most = 0;
    const auto with = [&](const Shape& sh) {
        const int64_t slots = bwd_slots(plan_rows(T, static_cast<int64_t>(kNumCU) * sh.per_cu, sh.R), 1);
        if (slots > most) most = slots;
    };
    const auto with_rules = [&](const auto& rules) {
        for (const SizeRule& r : rules)
            if (nchunks >= r.first && nchunks <= r.last && r.segs_from <= 1) with(r.sh);
    };
    for (const int64_t rows : {int64_t(0), int64_t(1), kNarrowBwdBytes / (nchunks * 16) + 1})
        with(recompute ? rc_bwd_table(nchunks, dtype, rows) : bwd_table(nchunks, dtype, rows));
    if (dtype == 0 && recompute) with_rules(kRcBwdRules);
    else if (dtype == 0) with_rules(kBwdRules);
    else if (!recompute) with_rules(kBwdRules32);
    return most;
}

// For a caller whose workspace cannot grow: the launch shape of this backward whose plan has at most max_slots
// slots -- the table's own if it has, else the same rows per wave with fewer blocks in a cluster or on a CU, always in
// clusters of every C-th block.  False if there is none.
inline bool bwd_shape_within(int64_t T, int64_t nseg, int64_t D, int dtype, bool recompute, int64_t max_slots,
                             Shape* out) {
    const BwdLaunch own = plan_bwd(T, nseg, D, dtype, false, recompute, nullptr);
    *out = own.sh;
    if (bwd_slots(own.pl, nseg) <= max_slots) return true;
    for (int per_cu = own.sh.per_cu; per_cu >= 1; --per_cu) {
        Shape sh = own.sh;
        sh.per_cu = per_cu;
        const int64_t g = grid_blocks(T, static_cast<int64_t>(kNumCU) * per_cu, sh.R);
        for (int64_t nb = own.pl.nb < g ? own.pl.nb : g; nb >= 1; nb /= 2) {
            sh.clusters = static_cast<int>(g / nb);
            sh.interleave = 1;
            if (bwd_slots(plan_bwd(T, nseg, D, dtype, false, recompute, &sh).pl, nseg) <= max_slots) {
                *out = sh;
                return true;
            }
        }
    }
    return false;
}

// Shape of the second pass: W waves per block, G groups of lanes per wave that take different slots; a lane adds
// V features (16 bytes of a slot; D is a multiple of 4), so a block covers 64 / G * V of them.  Wide blocks need enough
// (segment, sum, feature-block) triples to fill the chip; with fewer of them a block is narrower and its waves cover
// several slots per load (second pass of 75 600 x 5120: 6.1 -> 4.9 us with 16 bytes per lane instead of 4, of 32 760 x
// 1536: 8.9 -> 6.4, of 2 x 32 760 x 5120: 9.9 -> 7.8; eight groups of 32 features or sixteen of 16 were slower again).
// A group should have about one batch of slots to add, and a block never more than 16 waves.
struct ReduceShape {
    static constexpr int V = 4;
    int W = 1;
    int G = 1;
};

inline ReduceShape reduce_shape(int64_t nseg, int nsum, int64_t D, int64_t clusters, int64_t nb) {
    ReduceShape sh;
    const int64_t triples = nseg * nsum;
    if (triples * ((D + 255) / 256) < 256) sh.G = triples * ((D + 127) / 128) >= 256 ? 2 : 4;
    const int64_t slots = nb * (1 + (clusters - 1) / nseg);   // typical slots of one segment
    const int64_t each = sh.G == 1 ? 4 : sh.G;
    while (sh.W < 16 && sh.W * 2 * each <= slots) sh.W *= 2;
    return sh;
}

// The backward entry point that allocates nothing keeps its partial-sum slots in a static device
// array of this size (per GPU); static_workspace() returns that array's address on the current
// device.
constexpr size_t kStaticWorkspaceBytes = size_t(64) << 20;
hipError_t static_workspace(float** ptr);

// Text naming the kernel instantiations and grids that a call with these arguments launches.
int describe_fwd(const Problem& p, bool per_token, char* buf, size_t n);
int describe_bwd(const Problem& p, bool per_token, bool recompute, char* buf, size_t n);

struct ReduceArgs;
hipError_t launch_reduce(ReduceArgs r, int64_t clusters, hipStream_t st);

hipError_t launch_fwd_seg(const Problem& p, const void* x, const void* shift, const void* scale,
                          void* y, float* mean, float* rstd, hipStream_t st);
hipError_t launch_fwd_tok(const Problem& p, const void* x, const void* shift, const void* scale,
                          void* y, float* mean, float* rstd, hipStream_t st);
// io_grads: the reduced parameter gradients are written in the I/O element type instead of float32.
hipError_t launch_bwd_seg(const Problem& p, const void* dy, const void* x, const void* scale,
                          const float* mean, const float* rstd, void* dx, void* dshift,
                          void* dscale, bool io_grads, float* ws, hipStream_t st);
hipError_t launch_bwd_tok(const Problem& p, const void* dy, const void* x, const void* scale,
                          const float* mean, const float* rstd, void* dx, void* dshift,
                          void* dscale, hipStream_t st);
hipError_t launch_unfused(const Problem& p, const void* x, const void* shift, const void* scale,
                          void* xhat, void* y, float* mean, float* rstd, hipStream_t st);
hipError_t launch_copy(const void* src, void* dst, size_t bytes, hipStream_t st);
bool probe_mixture_supported(int reads, int writes);
hipError_t launch_stream_probe(const void* const* in, int reads, void* const* out, int writes, size_t bytes,
                               int blocks, int waves, int vecs, hipStream_t st);

// Gated residual + LayerNorm-Modulate (per-sample / per-segment gate, shift, scale).
RowPlan gated_bwd_plan(int64_t T, int64_t nseg, int64_t D, int dtype);
Shape gated_fwd_table_shape(int nchunks, int dtype, int64_t T);  // the tables' entries, no override
Shape gated_bwd_table_shape(int nchunks, int dtype, int64_t T);
hipError_t launch_gated_fwd(const Problem& p, const void* x, const void* u, const void* gate,
                            const void* shift, const void* scale, void* h, void* y, float* mean,
                            float* rstd, hipStream_t st);
hipError_t launch_gate_residual(const Problem& p, const void* x, const void* u, const void* gate,
                                void* h, hipStream_t st);
hipError_t launch_gated_bwd(const Problem& p, const void* dy, const void* dh, const void* h,
                            const void* u, const void* gate, const void* scale, const float* mean,
                            const float* rstd, void* dx, void* du, void* dgate, void* dshift,
                            void* dscale, bool io_grads, float* ws, hipStream_t st);
hipError_t launch_zero_f32(float* p, int64_t n, hipStream_t st);


// Fused Q-Norm + K-Norm (RMS normalisation with a learned weight of two tensors, one launch).
int32_t qknorm_bwd_blocks(int64_t N, int64_t D, int dtype);      // partial-sum slots per tensor
Shape qknorm_table_shape(int nchunks, int dtype, bool backward, int64_t N);  // rows wider than one head; no override
hipError_t launch_qknorm_fwd(int dtype, const void* q, const void* k, const void* wq, const void* wk,
                             int64_t N, int64_t D, float eps, void* q_out, void* k_out,
                             float* rstd_q, float* rstd_k, hipStream_t st);
hipError_t launch_qknorm_bwd(int dtype, const void* dq_out, const void* dk_out, const void* q,
                             const void* k, const void* wq, const void* wk, int64_t N, int64_t D,
                             const float* rstd_q, const float* rstd_k, void* dq, void* dk,
                             void* dwq, void* dwk, bool io_grads, float* ws, hipStream_t st);

}  // namespace lnmod
