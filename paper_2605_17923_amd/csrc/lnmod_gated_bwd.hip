// lnmod_gated_bwd.hip -- instantiation and launch of the gated residual + LayerNorm-Modulate
// backward (dx, du, and the per-sample / per-segment dgate, dshift, dscale) and of its second,
// fixed-order reduction pass.
#include "lnmod_gated_kernels.hpp"
#include "lnmod_launch.hpp"

namespace lnmod {
namespace {

// Launch shape (see Shape in lnmod_launch.hpp).  A lane holds 8 features of a row (one bf16 chunk,
// two fp32 chunks): with five fp32 values per feature living in registers (1+scale, gate, three
// running sums) and four packed input streams prefetched one step ahead, that is what fits
// without spilling.  bf16 rows of 9 to 16 times 512 features take two chunks per lane on 6 or 8
// waves instead (whole multiples of the four SIMDs; D = 5120: 798 against 819 us, and sixteen
// waves would halve the registers a wave may use).  The shapes are a table per 256 features from a sweep of
// every compiled shape on 32 and 200 MB tensors (fp32: 150 MB); against the rule with overrides per 512
// features that stood here they take 0.97 of the time in the mean over 32 widths (200 MB bf16: D = 256 341 ->
// 221 us, 768 267 -> 211, 1280 233 -> 207, 1792 244 -> 222; fp32 D = 1280 186 -> 154, 2304 178 -> 160).
Shape gated_bwd_shape(int nchunks, int dtype, int64_t T) {
    if (dtype == 0) {
        static const Shape tab[33] = {
            {1, 1, 2, 8},
            {1, 1, 2, 8}, {1, 1, 2, 3}, {2, 1, 2, 3}, {2, 1, 1, 2},   // D <= 1024
            {4, 1, 2, 2}, {3, 1, 2, 1}, {4, 1, 2, 1}, {4, 1, 1, 1},   // D <= 2048
            {6, 1, 2, 1}, {5, 1, 1, 1}, {8, 1, 1, 1}, {8, 1, 1, 1},   // D <= 3072
            {8, 1, 2, 1}, {8, 1, 2, 1}, {8, 1, 2, 1}, {8, 1, 2, 1},   // D <= 4096
            {10, 1, 1, 1}, {8, 2, 1, 1}, {10, 1, 1, 1}, {8, 2, 1, 1},   // D <= 5120
            {6, 2, 1, 1}, {6, 2, 1, 1}, {6, 2, 1, 1}, {12, 1, 1, 1},   // D <= 6144
            {8, 2, 1, 1}, {8, 2, 1, 1}, {8, 2, 1, 1}, {8, 2, 1, 1},   // D <= 7168
            {8, 2, 1, 1}, {8, 2, 1, 1}, {8, 2, 1, 1}, {16, 1, 1, 1}};   // D <= 8192
        // widths below a multiple of 256, timed on 0.3 to 900 MB: shares of the entry's time (see SizeRule)
        const int col = (nchunks + 31) / 32;
        if (col == 4 && nchunks < 128) return {2, 1, 2, 2};     // D = 776 ... 1016: 0.952, 1.05 (327)
        if (col == 8 && nchunks < 256) return {4, 1, 2, 1};     // D = 1800 ... 2040: 0.953, 1.09 (327)
        // D = 2568 ... 2808: 0.964, 1.02 (252); up to 20 MB 0.99, up to 1.11
        if (col == 11 && nchunks < 352 && (T == 0 || launch_mb(T, nchunks, 20, kAnyMB))) return {6, 1, 2, 1};
        return fine_entry(tab, nchunks, dtype);
    }
    static const Shape tab32[33] = {
        {1, 2, 1, 6},
        {1, 2, 1, 6}, {1, 2, 1, 3}, {3, 2, 1, 2}, {3, 2, 1, 2},   // D <= 1024
        {3, 2, 1, 2}, {4, 2, 1, 2}, {4, 2, 2, 2}, {4, 2, 2, 2},   // D <= 2048
        {6, 2, 2, 1}, {6, 2, 2, 1}, {6, 2, 2, 1}, {6, 2, 1, 1},   // D <= 3072
        {8, 2, 2, 1}, {8, 2, 2, 1}, {8, 2, 1, 1}, {8, 2, 1, 1},   // D <= 4096
        {10, 2, 1, 1}, {10, 2, 1, 1}, {10, 2, 1, 1}, {10, 2, 1, 1},   // D <= 5120
        {12, 2, 1, 1}, {12, 2, 1, 1}, {12, 2, 1, 1}, {12, 2, 1, 1},   // D <= 6144
        {16, 2, 1, 1}, {16, 2, 1, 1}, {16, 2, 1, 1}, {16, 2, 1, 1},   // D <= 7168
        {16, 2, 1, 1}, {16, 2, 1, 1}, {16, 2, 1, 1}, {16, 2, 1, 1}};   // D <= 8192
    return fine_entry(tab32, nchunks, dtype);
}

template <typename Tag, int VPL, int K, int R>
void go_r(const GatedBwdArgs& a, int64_t blocks, hipStream_t st) {
    const dim3 grid(static_cast<unsigned>(blocks)), block(K * kWave);
    if (a.nchunks == K * VPL * kWave)
        hipLaunchKernelGGL((gated_bwd_kernel<Tag, VPL, K, R, true>), grid, block, 0, st, a);
    else
        hipLaunchKernelGGL((gated_bwd_kernel<Tag, VPL, K, R, false>), grid, block, 0, st, a);
}

template <typename Tag, int VPL, int K>
void go(const GatedBwdArgs& a, int R, int64_t blocks, hipStream_t st) {
    // two rows per step only for rows up to 8 KB: at most 8 waves of 8 features per lane
    if constexpr (K <= 8 && (VPL == 1 || IO<Tag>::E == 4)) {
        if (R == 2) {
            go_r<Tag, VPL, K, 2>(a, blocks, st);
            return;
        }
    }
    go_r<Tag, VPL, K, 1>(a, blocks, st);
}

template <typename Tag, int VPL>
bool dispatch(const GatedBwdArgs& a, Shape sh, int64_t blocks, hipStream_t st) {
    if (sh.VPL != VPL) {                     // the two-chunk shapes of wide bf16 rows
        if (sh.VPL != 2) return false;
        if (sh.K == 8) go<Tag, 2, 8>(a, sh.R, blocks, st);
        else if (sh.K == 6) go<Tag, 2, 6>(a, sh.R, blocks, st);
        else return false;
        return true;
    }
    switch (sh.K) {
        case 1: go<Tag, VPL, 1>(a, sh.R, blocks, st); return true;
        case 2: go<Tag, VPL, 2>(a, sh.R, blocks, st); return true;
        case 3: go<Tag, VPL, 3>(a, sh.R, blocks, st); return true;
        case 4: go<Tag, VPL, 4>(a, sh.R, blocks, st); return true;
        case 5: go<Tag, VPL, 5>(a, sh.R, blocks, st); return true;
        case 6: go<Tag, VPL, 6>(a, sh.R, blocks, st); return true;
        case 8: go<Tag, VPL, 8>(a, sh.R, blocks, st); return true;
        case 10: go<Tag, VPL, 10>(a, sh.R, blocks, st); return true;
        case 12: go<Tag, VPL, 12>(a, sh.R, blocks, st); return true;
        case 16: go<Tag, VPL, 16>(a, sh.R, blocks, st); return true;
        default: return false;
    }
}

}  // namespace

Shape gated_bwd_table_shape(int nchunks, int dtype, int64_t T) {
    return gated_bwd_shape(nchunks, dtype, T);
}

RowPlan gated_bwd_plan(int64_t T, int64_t nseg, int64_t D, int dtype) {
    const int E = dtype == 0 ? 8 : 4;
    const Shape sh = gated_bwd_shape(static_cast<int>(D / E), dtype, T);
    // a row moves 6 D elements (dy, dh, h, u, dx, du), a slot 3 D floats written and read back
    const double elem = dtype == 0 ? 2.0 : 4.0;
    const double stream_us = static_cast<double>(T) * static_cast<double>(D) * 6.0 * elem / 5.8e6;
    return plan_rows_slots(T, nseg, static_cast<int64_t>(kNumCU) * sh.per_cu, sh.R, stream_us,
                           24.0 / (6.0 * elem));
}

hipError_t launch_gated_bwd(const Problem& p, const void* dy, const void* dh, const void* h,
                            const void* u, const void* gate, const void* scale, const float* mean,
                            const float* rstd, void* dx, void* du, void* dgate, void* dshift,
                            void* dscale, bool io_grads, float* ws, hipStream_t st) {
    const int E = p.dtype == 0 ? 8 : 4;
    GatedBwdArgs a;
    a.dy = dy;
    a.dh = dh;
    a.h = h;
    a.u = u;
    a.gate = gate;
    a.scale = scale;
    a.mean = mean;
    a.rstd = rstd;
    a.dx = dx;
    a.du = du;
    a.ws = ws;
    a.seg = Segments{p.cu, p.S, p.nseg};
    a.T = p.T;
    a.D = static_cast<int32_t>(p.D);
    a.nchunks = static_cast<int32_t>(p.D / E);
    a.inv_D = 1.0f / static_cast<float>(p.D);
    const Shape sh = gated_bwd_shape(a.nchunks, p.dtype, p.T);
    if (!covers(sh, a.nchunks)) return hipErrorInvalidConfiguration;
    const RowPlan pl = gated_bwd_plan(p.T, p.nseg, p.D, p.dtype);
    a.rows_per_cluster = pl.rows_per_cluster;
    a.nb = pl.nb;
    a.interleave = cluster_interleave(nullptr, pl);
    a.split = cluster_split(a.interleave, pl);
    const bool ok = p.dtype == 0 ? dispatch<bf16_io, 1>(a, sh, pl.blocks, st)
                                 : dispatch<f32_io, 2>(a, sh, pl.blocks, st);
    if (!ok) return hipErrorInvalidConfiguration;
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;

    ReduceArgs r;
    r.ws = ws;
    r.out[0] = dshift;
    r.out[1] = dscale;
    r.out[2] = dgate;
    r.out_bf16 = io_grads && p.dtype == 0;
    r.seg = a.seg;
    r.T = p.T;
    r.rows_per_cluster = a.rows_per_cluster;
    r.nb = a.nb;
    r.D = a.D;
    r.nsum = 3;
    return launch_reduce(r, pl.clusters, st);
}

}  // namespace lnmod
