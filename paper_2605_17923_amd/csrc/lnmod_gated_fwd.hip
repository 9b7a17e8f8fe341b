// lnmod_gated_fwd.hip -- instantiation and launch of the gated residual + LayerNorm-Modulate
// forward, and of the residual-only kernel that serves as the unfused comparator's first half.
#include "lnmod_gated_kernels.hpp"
#include "lnmod_launch.hpp"

namespace lnmod {
namespace {

// Launch shape (see Shape in lnmod_launch.hpp) of the residual-only kernel at the widths below has this
// rule: the split of choose_split, two rows per step, about five waves per CU.
int blocks_per_cu(int K) {
    if (K == 1) return 4;
    if (K == 3) return 2;              // three waves alone leave a CU short
    const int b = 5 / K;
    return b < 1 ? 1 : b;
}

// (K, VPL, R, blocks per CU) of the fused kernel: a table per 256 features, from a sweep of every compiled
// shape on 200 MB tensors (fp32: 150 MB), and one for short launches (see short_launch) from 32 MB ones.
// Against the rule with overrides per 512 features that stood here: bf16 0.96 of the time in the mean over 32
// widths, short launches 0.94, fp32 0.95 (D = 768 167 -> 136 us, 1280 150 -> 136, 5888 145 -> 138; 32 MB: D =
// 768 31.5 -> 25.5, 4352 28.6 -> 25.3; fp32 D = 1280 113 -> 102, with one row per step as in bf16).
Shape gated_fwd_shape(int nchunks, int dtype, bool ln, int64_t T, int64_t nseg) {
    if (ln && dtype == 0) {
        static const Shape tab[33] = {
            {1, 1, 1, 16},
            {1, 1, 1, 16}, {1, 1, 2, 4}, {1, 2, 1, 6}, {2, 2, 1, 4},   // D <= 1024
            {2, 2, 1, 4}, {2, 2, 1, 3}, {2, 2, 1, 3}, {2, 2, 1, 3},   // D <= 2048
            {3, 2, 1, 2}, {3, 2, 1, 2}, {3, 2, 1, 2}, {3, 2, 1, 2},   // D <= 3072
            {4, 2, 2, 1}, {4, 2, 2, 1}, {5, 2, 1, 1}, {4, 3, 1, 1},   // D <= 4096
            {4, 3, 1, 1}, {6, 2, 1, 1}, {4, 3, 1, 1}, {4, 3, 1, 1},   // D <= 5120
            {4, 3, 1, 1}, {4, 3, 1, 1}, {6, 2, 2, 1}, {8, 2, 2, 1},   // D <= 6144
            {8, 2, 2, 1}, {8, 2, 2, 1}, {8, 2, 2, 1}, {8, 2, 2, 1},   // D <= 7168
            {8, 2, 1, 1}, {8, 2, 1, 1}, {8, 2, 1, 1}, {8, 2, 2, 2}};   // D <= 8192
        static const Shape tab_short[33] = {
            {1, 1, 2, 16},
            {1, 1, 2, 16}, {1, 1, 1, 8}, {1, 2, 1, 6}, {1, 2, 2, 12},   // D <= 1024
            {2, 2, 1, 8}, {1, 3, 1, 8}, {2, 2, 1, 6}, {2, 2, 1, 4},   // D <= 2048
            {3, 2, 1, 4}, {3, 2, 1, 2}, {4, 2, 1, 3}, {4, 2, 1, 3},   // D <= 3072
            {4, 2, 1, 2}, {4, 2, 2, 2}, {4, 2, 1, 2}, {5, 2, 1, 2},   // D <= 4096
            {4, 3, 1, 2}, {4, 3, 2, 2}, {4, 3, 1, 2}, {4, 3, 1, 2},   // D <= 5120
            {4, 3, 1, 1}, {4, 3, 1, 2}, {4, 3, 1, 2}, {4, 3, 1, 2},   // D <= 6144
            {8, 2, 1, 2}, {8, 2, 1, 2}, {8, 2, 2, 1}, {8, 2, 1, 1},   // D <= 7168
            {8, 2, 1, 1}, {8, 2, 1, 1}, {8, 2, 1, 1}, {8, 2, 1, 2}};   // D <= 8192
        // sizes and widths between two multiples of 256: shares of the entry's time (see SizeRule)
        static const SizeRule rules[] = {
            {65, 95, 4, 20, {1, 2, 2, 12}},          // D = 520 ... 760: 0.918, 1.04 (237); below 1.035, up to 1.30
            {65, 95, 20, 72, {1, 2, 2, 8}},          // the same: 0.953, 1.03 (267)
            {65, 95, 72, 150, {1, 2, 2, 8}, 5},      // the same: 0.964, 1.03 (129); on one to four samples 1.00, up to 1.06
            {97, 127, 72, 200, {1, 2, 2, 4}},        // D = 776 ... 1016: 0.96, 1.02 (282)
            {97, 127, 200, 300, {1, 2, 2, 4}, 5},    // the same: 0.952, 1.01 (111); on one to four samples up to 1.05
            {225, 255, 72, 150, {2, 2, 1, 4}},       // D = 1800 ... 2040: 0.943, 1.01 (327)
            {289, 320, 2, 20, {4, 2, 1, 3}},         // D = 2312 ... 2560: 0.958, 1.04 (267)
            {448, 448, 20, 72, {4, 2, 1, 3}, 0, 8}};     // D = 3584: 0.962, 1.03 (310); on more segments 1.01, up to 1.04
        if (const Shape* sh = size_rule(rules, nchunks, T, nseg)) return *sh;
        // D = 4360 ... 6656: two tensors are read, and at 71 MB the short entries lost 3 to 8 % (5048 52.5 -> 56.4 us);
        // elsewhere they win up to 72 MB at most widths (2568 56.2 against 60.3 us, 7096 44.9 against 47.2)
        if (short_launch(T, nchunks) && (nchunks <= 544 || nchunks > 832 || T * nchunks * 16 <= 48000000))
            return fine_entry(tab_short, nchunks, dtype);
        // D = 1160 ... 1272: 0.88 to 0.97 of the time at 85 and 200 MB; narrower (1032 ... 1144) 0.95 to 1.03 at 200 MB
        // and 8 to 14 % slower at 85
        if (unaligned_rows(nchunks) && (nchunks + 31) / 32 == 5 && (nchunks > 144 || T == 0 || T * nchunks * 16 > 128000000))
            return {2, 2, 1, 3};
        return fine_entry(tab, nchunks, dtype);
    }
    if (ln) {
        static const Shape tab32[33] = {
            {1, 1, 1, 8},
            {1, 1, 1, 8}, {1, 2, 2, 4}, {1, 3, 2, 4}, {1, 4, 1, 4},   // D <= 1024
            {2, 4, 1, 3}, {2, 4, 1, 2}, {2, 4, 1, 3}, {2, 4, 1, 3},   // D <= 2048
            {3, 4, 1, 2}, {3, 4, 2, 2}, {4, 4, 1, 2}, {3, 4, 1, 2},   // D <= 3072
            {4, 4, 2, 1}, {4, 4, 1, 2}, {4, 4, 1, 2}, {4, 4, 1, 2},   // D <= 4096
            {5, 4, 2, 1}, {5, 4, 2, 1}, {5, 4, 2, 2}, {5, 4, 1, 1},   // D <= 5120
            {8, 4, 1, 1}, {8, 4, 1, 1}, {8, 4, 1, 1}, {8, 4, 1, 1},   // D <= 6144
            {8, 4, 1, 1}, {8, 4, 1, 1}, {8, 4, 1, 2}, {8, 4, 1, 2},   // D <= 7168
            {8, 4, 1, 1}, {8, 4, 1, 2}, {8, 4, 1, 2}, {8, 4, 1, 2}};   // D <= 8192
        Shape sh = fine_entry(tab32, nchunks, dtype);
        if (short_launch(T, nchunks)) {
            // few rows for each of 256 blocks: two per step (976 x 5120: 15.7 us against 18.4)
            if (sh.per_cu == 1) sh.R = 2;
            // four waves per CU and at most four steps of one row: two per step (2441 x 1024: 9.3 us against 10.2,
            // 1775 x 1408 10.7 against 12.1)
            if (sh.K * sh.per_cu == 4 && T <= 1024 * sh.per_cu) sh.R = 2;
            // five waves, less than three steps of two rows: one block per CU (three segments, 1354 x 4612: 21.8 against 24.2)
            if (sh.K == 5 && T < 1536) sh.per_cu = 1;
            // eight waves: a row for every block, or two rows per step in one or two blocks per CU (488 x 7168: 11.3 us
            // against 14.6 with one row and two blocks, 903 x 6916 19.8 against 21.7; 244 x 8192 one row 9.1 against 10.3)
            if (sh.K == 8 && T <= kNumCU) sh = {8, 4, 1, 1};
            else if (sh.K == 8 && nchunks > 1920) sh = {8, 4, 2, 2};
            else if (sh.K == 8 && T <= 1024) sh = {8, 4, 2, 1};
        }
        return sh;
    }
    const Split sp = choose_split(nchunks, dtype);
    Shape sh{sp.K, sp.VPL, 2, blocks_per_cu(sp.K)};
    if (dtype == 0 && !ln) {
        // the residual-only kernel (first half of the unfused comparator) at the two model widths:
        // D = 1536: 366 against 393 us, D = 5120: 385 against 401 us on 774 MB per tensor
        const int cols = (nchunks + kWave - 1) / kWave;
        if (cols == 3) sh = {3, 2, 2, 2};
        if (cols >= 9 && cols <= 12) sh = {4, 3, 2, 1};
    }
    return sh;
}

template <typename Tag, int VPL, int K, int R, bool LN>
void go_r(const GatedFwdArgs& a, int64_t blocks, hipStream_t st) {
    const dim3 grid(static_cast<unsigned>(blocks)), block(K * kWave);
    if (a.nchunks == K * VPL * kWave)
        hipLaunchKernelGGL((gated_fwd_kernel<Tag, VPL, K, R, true, LN>), grid, block, 0, st, a);
    else
        hipLaunchKernelGGL((gated_fwd_kernel<Tag, VPL, K, R, false, LN>), grid, block, 0, st, a);
}

template <typename Tag, int VPL, int K, bool LN>
void go(const GatedFwdArgs& a, int R, int64_t blocks, hipStream_t st) {
    if constexpr (LN) {
        if (R == 1) {
            go_r<Tag, VPL, K, 1, LN>(a, blocks, st);
            return;
        }
    }
    go_r<Tag, VPL, K, 2, LN>(a, blocks, st);
}

template <typename Tag, bool LN>
bool dispatch(const GatedFwdArgs& a, Shape sh, int64_t blocks, hipStream_t st) {
    switch (sh.VPL * 100 + sh.K) {
        case 101: go<Tag, 1, 1, LN>(a, sh.R, blocks, st); return true;
        case 201: go<Tag, 2, 1, LN>(a, sh.R, blocks, st); return true;
        case 301: go<Tag, 3, 1, LN>(a, sh.R, blocks, st); return true;
        default: break;
    }
    if constexpr (IO<Tag>::E == 8) {
        switch (sh.VPL * 100 + sh.K) {
            case 202: go<Tag, 2, 2, LN>(a, sh.R, blocks, st); return true;
            case 203: go<Tag, 2, 3, LN>(a, sh.R, blocks, st); return true;
            case 204: go<Tag, 2, 4, LN>(a, sh.R, blocks, st); return true;
            case 205: go<Tag, 2, 5, LN>(a, sh.R, blocks, st); return true;
            case 206: go<Tag, 2, 6, LN>(a, sh.R, blocks, st); return true;
            case 208: go<Tag, 2, 8, LN>(a, sh.R, blocks, st); return true;
            case 304: go<Tag, 3, 4, LN>(a, sh.R, blocks, st); return true;
            default: break;
        }
    } else {
        switch (sh.VPL * 100 + sh.K) {
            case 401: go<Tag, 4, 1, LN>(a, sh.R, blocks, st); return true;
            case 601: go<Tag, 6, 1, LN>(a, sh.R, blocks, st); return true;
            case 402: go<Tag, 4, 2, LN>(a, sh.R, blocks, st); return true;
            case 403: go<Tag, 4, 3, LN>(a, sh.R, blocks, st); return true;
            case 404: go<Tag, 4, 4, LN>(a, sh.R, blocks, st); return true;
            case 405: go<Tag, 4, 5, LN>(a, sh.R, blocks, st); return true;
            case 406: go<Tag, 4, 6, LN>(a, sh.R, blocks, st); return true;
            case 408: go<Tag, 4, 8, LN>(a, sh.R, blocks, st); return true;
            default: break;
        }
    }
    return false;
}

template <bool LN>
hipError_t launch(const Problem& p, const void* x, const void* u, const void* gate, const void* shift,
                  const void* scale, void* h, void* y, float* mean, float* rstd, hipStream_t st) {
    const int E = p.dtype == 0 ? 8 : 4;
    GatedFwdArgs a;
    a.x = x;
    a.u = u;
    a.gate = gate;
    a.shift = shift;
    a.scale = scale;
    a.h = h;
    a.y = y;
    a.mean = mean;
    a.rstd = rstd;
    a.seg = Segments{p.cu, p.S, p.nseg};
    a.T = p.T;
    a.D = static_cast<int32_t>(p.D);
    a.nchunks = static_cast<int32_t>(p.D / E);
    a.eps = p.eps;
    a.inv_D = 1.0f / static_cast<float>(p.D);
    const Shape sh = gated_fwd_shape(a.nchunks, p.dtype, LN, p.T, p.nseg);
    if (!covers(sh, a.nchunks)) return hipErrorInvalidConfiguration;
    // bytes of x, u, h and y at 6 TB/s
    const double stream_us = static_cast<double>(p.T) * static_cast<double>(p.D) * (p.dtype == 0 ? 8.0 : 16.0) / 6.0e6;
    const RowPlan pl = plan_rows_clusters(p.T, p.nseg, static_cast<int64_t>(kNumCU) * sh.per_cu, sh.R,
                                          pick_clusters(stream_us, p.nseg));
    a.rows_per_cluster = pl.rows_per_cluster;
    a.nb = pl.nb;
    // two and four clusters on all XCDs (2 to 12 samples, 20 and 200 MB: 0.98 and 0.985 of the time in the mean over 13
    // widths, 2 x 24 800 x 2528 194 -> 184 us), eight and more with an XCD each (40 segments, 20 and 60 MB: 0.97)
    a.interleave = pl.clusters >= 8 ? 1 : 0;
    a.split = cluster_split(a.interleave, pl);
    const bool ok = p.dtype == 0 ? dispatch<bf16_io, LN>(a, sh, pl.blocks, st)
                                 : dispatch<f32_io, LN>(a, sh, pl.blocks, st);
    return ok ? hipGetLastError() : hipErrorInvalidConfiguration;
}

}  // namespace

Shape gated_fwd_table_shape(int nchunks, int dtype, int64_t T) { return gated_fwd_shape(nchunks, dtype, true, T, 0); }

hipError_t launch_gated_fwd(const Problem& p, const void* x, const void* u, const void* gate,
                            const void* shift, const void* scale, void* h, void* y, float* mean,
                            float* rstd, hipStream_t st) {
    return launch<true>(p, x, u, gate, shift, scale, h, y, mean, rstd, st);
}

hipError_t launch_gate_residual(const Problem& p, const void* x, const void* u, const void* gate,
                                void* h, hipStream_t st) {
    return launch<false>(p, x, u, gate, nullptr, nullptr, h, nullptr, nullptr, nullptr, st);
}

}  // namespace lnmod
