// lnmod_qknorm.hip -- instantiation and launch of the fused Q-Norm + K-Norm kernels (forward,
// backward and the fixed-order second pass of the weight gradients).
#include "lnmod_qknorm_kernels.hpp"
#include "lnmod_launch.hpp"

namespace lnmod {
namespace {

constexpr int kRows = 2;           // rows per block and step

// Launch shape of the wide-row kernels (R is fixed by the instantiations; per_cu counts the resident blocks
// of both tensors together, each tensor gets half of them): a table per 256 features from a sweep of every
// compiled shape on 200 MB per tensor (fp32: 150 MB; the bf16 backward 32 and 200 MB), and for short bf16
// forwards (see short_launch) one from 32 MB.  Against the rule with overrides per 512 features that stood here:
// forward 0.98 of the time in the mean over 32 widths, short 0.94, fp32 0.96, backward 0.99 (forward D = 768 151
// -> 138 us, 1792 161 -> 133, short 31.0 -> 24.3; backward D = 768 229 -> 207, 1280 215 -> 202, 3328 209 -> 197).
Shape wide_table_shape(int nchunks, int dtype, bool backward, int64_t N = 0) {
    if (!backward && dtype == 0) {
        static const Shape tab[33] = {
            {1, 1, 2, 8},
            {1, 1, 2, 8}, {1, 1, 2, 8}, {1, 2, 2, 6}, {1, 2, 2, 4},   // D <= 1024
            {2, 2, 2, 4}, {1, 3, 2, 3}, {2, 2, 2, 3}, {2, 2, 2, 2},   // D <= 2048
            {3, 2, 2, 2}, {3, 2, 2, 2}, {3, 2, 2, 2}, {3, 2, 2, 2},   // D <= 3072
            {4, 2, 2, 1}, {4, 2, 2, 1}, {5, 2, 2, 1}, {4, 3, 2, 1},   // D <= 4096
            {5, 2, 2, 1}, {5, 2, 2, 1}, {5, 2, 2, 1}, {5, 2, 2, 1},   // D <= 5120
            {6, 2, 2, 1}, {6, 2, 2, 1}, {8, 2, 2, 1}, {6, 2, 2, 1},   // D <= 6144
            {8, 2, 2, 1}, {8, 2, 2, 1}, {8, 2, 2, 1}, {8, 2, 2, 1},   // D <= 7168
            {8, 2, 2, 1}, {8, 2, 2, 1}, {8, 2, 2, 1}, {8, 2, 2, 1}};   // D <= 8192
        static const Shape tab_short[33] = {
            {1, 1, 2, 8},
            {1, 1, 2, 8}, {1, 1, 2, 16}, {1, 2, 2, 16}, {1, 2, 2, 16},   // D <= 1024
            {2, 2, 2, 8}, {1, 3, 2, 16}, {2, 2, 2, 6}, {2, 2, 2, 8},   // D <= 2048
            {3, 2, 2, 6}, {4, 2, 2, 4}, {4, 2, 2, 3}, {4, 2, 2, 3},   // D <= 3072
            {5, 2, 2, 3}, {4, 2, 2, 4}, {5, 2, 2, 3}, {4, 2, 2, 4},   // D <= 4096
            {6, 2, 2, 3}, {6, 2, 2, 3}, {4, 3, 2, 3}, {4, 3, 2, 3},   // D <= 5120
            {4, 3, 2, 3}, {4, 3, 2, 3}, {4, 3, 2, 3}, {4, 3, 2, 3},   // D <= 6144
            {8, 2, 2, 2}, {8, 2, 2, 2}, {8, 2, 2, 1}, {8, 2, 2, 1},   // D <= 7168
            {8, 2, 2, 1}, {8, 2, 2, 1}, {8, 2, 2, 1}, {8, 2, 2, 1}};   // D <= 8192
        // shares of the entry's time (see SizeRule)
        static const SizeRule rules[] = {
            {129, 159, 4, 20, {1, 3, 2, 16}},        // D = 1032 ... 1272: 0.958, 1.04 (149); below 1.00, up to 1.06
            {320, 320, 4, 20, {3, 2, 2, 8}},         // D = 2560: 0.971, 1.02 (147); below 1.00, up to 1.05
            {384, 384, 4, 20, {3, 2, 2, 6}},         // D = 3072: 0.964, 1.03 (150); below 1.00, up to 1.07
            {512, 512, 20, 72, {4, 2, 2, 3}}};       // D = 4096: 0.969, 1.01 (215)
        if (const Shape* sh = size_rule(rules, nchunks, N)) return *sh;
        // two tensors are read: beyond D = 3840 the short entries lost 3 to 8 % at 62 MB (D = 5128 44.4 -> 48.1 us),
        // below it they still win there at most widths (1808 53.1 -> 47.0, 3136 48.7 -> 43.5)
        const bool few = short_launch(N, nchunks) && (nchunks <= 480 || N * nchunks * 16 <= 36000000);
        return few ? fine_entry(tab_short, nchunks, dtype) : fine_entry(tab, nchunks, dtype);
    }
    if (!backward) {
        static const Shape tab32[33] = {
            {1, 1, 2, 8},
            {1, 1, 2, 8}, {1, 2, 2, 8}, {1, 3, 2, 8}, {1, 4, 2, 6},   // D <= 1024
            {2, 4, 2, 3}, {2, 4, 2, 4}, {2, 4, 2, 2}, {2, 4, 2, 2},   // D <= 2048
            {3, 4, 2, 2}, {3, 4, 2, 3}, {3, 4, 2, 3}, {3, 4, 2, 1},   // D <= 3072
            {4, 4, 2, 1}, {4, 4, 2, 1}, {5, 4, 2, 2}, {5, 4, 2, 2},   // D <= 4096
            {5, 4, 2, 2}, {5, 4, 2, 2}, {5, 4, 2, 2}, {5, 4, 2, 2},   // D <= 5120
            {6, 4, 2, 2}, {6, 4, 2, 1}, {6, 4, 2, 1}, {6, 4, 2, 1},   // D <= 6144
            {8, 4, 2, 1}, {8, 4, 2, 1}, {8, 4, 2, 1}, {8, 4, 2, 1},   // D <= 7168
            {8, 4, 2, 1}, {8, 4, 2, 1}, {8, 4, 2, 1}, {8, 4, 2, 1}};   // D <= 8192
        // the table was timed at 150 MB; shares of the entry's time (see SizeRule)
        static const SizeRule rules32[] = {
            {257, 320, 0, 72, {1, 6, 2, 6}},         // D = 1028 ... 1280: 0.954, 1.02 (215)
            {385, 512, 4, 20, {2, 4, 2, 4}},         // D = 1540 ... 2048: 0.906, 1.02 (139)
            {385, 512, 20, 36, {2, 4, 2, 6}},        // the same: 0.953, 1.02 (118); beyond 1.00, up to 1.06
            {513, 576, 4, 7, {3, 4, 2, 3}},          // D = 2052 ... 2304: 0.921, 1.02 (46)
            {513, 576, 10, 72, {3, 4, 2, 3}},        // the same: 0.942, 1.02 (98); between them up to 1.06
            {768, 768, 4, 72, {3, 4, 2, 3}},         // D = 3072: 0.889, 1.05 (145)
            {1536, 1536, 20, 36, {8, 4, 2, 2}},      // D = 6144: 0.912, 1.02 (147); beyond 1.00, up to 1.04
            {833, 896, 10, 150, {4, 4, 2, 2}}};      // D = 3332 ... 3584: 0.913, 1.02 (150); beyond 1.00, up to 1.07
        if (const Shape* sh = size_rule(rules32, nchunks, N)) return *sh;
        return fine_entry(tab32, nchunks, dtype);
    }
    if (dtype == 0) {
        static const Shape tab[33] = {
            {1, 1, 2, 6},
            {1, 1, 2, 6}, {1, 1, 2, 6}, {1, 2, 2, 6}, {1, 2, 2, 3},   // D <= 1024
            {2, 2, 2, 4}, {2, 2, 2, 3}, {2, 2, 2, 3}, {2, 2, 2, 2},   // D <= 2048
            {3, 2, 2, 2}, {3, 2, 2, 2}, {3, 2, 2, 2}, {3, 2, 2, 1},   // D <= 3072
            {4, 2, 2, 1}, {4, 2, 2, 2}, {4, 2, 2, 1}, {4, 2, 2, 1},   // D <= 4096
            {5, 2, 2, 1}, {5, 2, 2, 1}, {5, 2, 2, 1}, {5, 2, 2, 1},   // D <= 5120
            {6, 2, 2, 1}, {6, 2, 2, 1}, {6, 2, 2, 1}, {6, 2, 2, 1},   // D <= 6144
            {8, 2, 2, 1}, {8, 2, 2, 1}, {8, 2, 2, 1}, {8, 2, 2, 1},   // D <= 7168
            {8, 2, 2, 1}, {8, 2, 2, 1}, {8, 2, 2, 1}, {8, 2, 2, 1}};   // D <= 8192
        static const SizeRule rules[] = {{417, 448, 0, 20, {4, 2, 2, 1}}};       // D = 3336 ... 3584: 0.935, 1.04 (164)
        if (const Shape* sh = size_rule(rules, nchunks, N)) return *sh;
        // D = 1800 ... 1984: the entry was timed at 2048 (1920, 62, 95 and 173 MB: 67.7, 99.1, 176 us against 70.1, 103, 186)
        if (nchunks > 224 && nchunks <= 248) return {2, 2, 2, 3};
        // D = 3080 ... 3320 from 62 MB on: 0.94 to 0.985 of the time (3160 190 against 203 us); aligned rows 4 to 6 % slower
        if (unaligned_rows(nchunks) && (nchunks + 31) / 32 == 13 && (N == 0 || N * nchunks * 16 > 40000000)) return {4, 2, 2, 2};
        return fine_entry(tab, nchunks, dtype);
    }
    static const Shape tab32[33] = {
        {1, 1, 2, 6},
        {1, 1, 2, 6}, {1, 2, 2, 4}, {1, 3, 2, 4}, {1, 4, 2, 4},   // D <= 1024
        {2, 4, 2, 3}, {2, 4, 2, 3}, {2, 4, 2, 3}, {2, 4, 2, 3},   // D <= 2048
        {3, 4, 2, 2}, {3, 4, 2, 2}, {3, 4, 2, 2}, {3, 4, 2, 2},   // D <= 3072
        {4, 4, 2, 2}, {4, 4, 2, 2}, {4, 4, 2, 1}, {4, 4, 2, 1},   // D <= 4096
        {5, 4, 2, 1}, {5, 4, 2, 1}, {5, 4, 2, 1}, {5, 4, 2, 1},   // D <= 5120
        {6, 4, 2, 1}, {6, 4, 2, 1}, {6, 4, 2, 1}, {6, 4, 2, 1},   // D <= 6144
        {8, 4, 2, 1}, {8, 4, 2, 1}, {8, 4, 2, 1}, {8, 4, 2, 1},   // D <= 7168
        {8, 4, 2, 1}, {8, 4, 2, 1}, {8, 4, 2, 1}, {8, 4, 2, 1}};   // D <= 8192
    // D = 1284 ... 1536: three blocks per CU of two waves take 0.94 of the time of one wave with six chunks (90 problems of 2.5
    // to 21 MB; 1.07 at 2032 rows of 1536); two blocks per CU are 0.89 of three at 769 ... 1024 rows but 1.17 at 521 ... 703,
    // and a size at which the slots fell as the rows grow would break a workspace sized for more rows.
    // D = 3332 ... 3584: 0.968, 1.01 (218) beyond 20 MB, below the same
    static const SizeRule rules32[] = {{833, 896, 0, 20, {4, 4, 2, 1}}};
    if (const Shape* sh = size_rule(rules32, nchunks, N)) return *sh;
    return fine_entry(tab32, nchunks, dtype);
}

// The table's shape; ok is false for a shape these kernels are not compiled for or that does not
// cover the row (a mistake in the table then fails the launch instead of computing on part of a row).
Shape wide_shape(int nchunks, int dtype, bool backward, int64_t N, bool* ok) {
    const Shape sh = wide_table_shape(nchunks, dtype, backward, N);
    const int wide = dtype == 0 ? 2 : 4;
    bool compiled;
    if (sh.K == 1) compiled = sh.VPL >= 1 && (sh.VPL <= 3 || (dtype == 1 && (sh.VPL == 4 || sh.VPL == 6)));
    else compiled = (sh.VPL == wide && (sh.K <= 6 || sh.K == 8)) || (dtype == 0 && sh.VPL == 3 && sh.K == 4);
    *ok = compiled && sh.R == kRows && covers(sh, nchunks);
    return sh;
}

int32_t blocks_per_tensor(int64_t N, int per_cu) {
    int64_t nb = static_cast<int64_t>(kNumCU) * per_cu / 2;
    const int64_t need = (N + kRows - 1) / kRows;
    if (nb > need) nb = need;
    return static_cast<int32_t>(nb < 1 ? 1 : nb);
}

template <typename Tag, int VPL, int K>
void go_fwd(const QkFwdArgs& a, hipStream_t st) {
    const dim3 grid(static_cast<unsigned>(2 * a.nb)), block(K * kWave);
    if (a.nchunks == K * VPL * kWave)
        hipLaunchKernelGGL((qknorm_fwd_kernel<Tag, VPL, K, kRows, true>), grid, block, 0, st, a);
    else
        hipLaunchKernelGGL((qknorm_fwd_kernel<Tag, VPL, K, kRows, false>), grid, block, 0, st, a);
}

template <typename Tag, int VPL, int K>
void go_bwd(const QkBwdArgs& a, hipStream_t st) {
    const dim3 grid(static_cast<unsigned>(2 * a.nb)), block(K * kWave);
    if (a.nchunks == K * VPL * kWave)
        hipLaunchKernelGGL((qknorm_bwd_kernel<Tag, VPL, K, kRows, true>), grid, block, 0, st, a);
    else
        hipLaunchKernelGGL((qknorm_bwd_kernel<Tag, VPL, K, kRows, false>), grid, block, 0, st, a);
}

// calls f.template operator()<VPL, K>() for the split; VPL_WIDE as in the other launchers
template <typename Tag, int VPL_WIDE, typename F>
void for_split(Split sp, F&& f) {
    if constexpr (IO<Tag>::E == 8) {             // bf16: three chunks per lane on four waves
        if (sp.VPL == 3 && sp.K == 4) {
            f.template operator()<3, 4>();
            return;
        }
    }
    if (sp.K == 1) {
        switch (sp.VPL) {
            case 1: f.template operator()<1, 1>(); break;
            case 2: f.template operator()<2, 1>(); break;
            case 3: f.template operator()<3, 1>(); break;
            default:                             // 4 and 6 chunks per lane: fp32 rows only
                if constexpr (IO<Tag>::E == 4) {
                    if (sp.VPL == 4) f.template operator()<4, 1>();
                    else f.template operator()<6, 1>();
                }
                break;
        }
        return;
    }
    switch (sp.K) {
        case 2: f.template operator()<VPL_WIDE, 2>(); break;
        case 3: f.template operator()<VPL_WIDE, 3>(); break;
        case 4: f.template operator()<VPL_WIDE, 4>(); break;
        case 5: f.template operator()<VPL_WIDE, 5>(); break;
        case 6: f.template operator()<VPL_WIDE, 6>(); break;
        default: f.template operator()<VPL_WIDE, 8>(); break;
    }
}

template <typename Tag>
struct FwdGo {
    const QkFwdArgs& a;
    hipStream_t st;
    template <int VPL, int K> void operator()() const { go_fwd<Tag, VPL, K>(a, st); }
};
template <typename Tag>
struct BwdGo {
    const QkBwdArgs& a;
    hipStream_t st;
    template <int VPL, int K> void operator()() const { go_bwd<Tag, VPL, K>(a, st); }
};

// Short rows (at most 32 chunks, e.g. one head's width): 16 lanes per row, four rows per wave.
constexpr int kShortMaxChunks = 32;
constexpr int kShortFwdBlocksPerCu = 8;              // blocks of 4 waves, over both tensors
constexpr int kShortBwdBlocksPerCu = 2;

// rows per wave and step = 4 * R: about 8 KB of loads per wave and step
template <int VPL> constexpr int short_fwd_r() { return VPL == 1 ? 8 : 4; }
template <int VPL> constexpr int short_bwd_r() { return VPL == 1 ? 4 : 2; }

int32_t short_blocks_per_tensor(int64_t N, int rows_per_piece, int per_cu) {
    int64_t nb = static_cast<int64_t>(kNumCU) * per_cu / 2;
    const int64_t pieces = (N + rows_per_piece - 1) / rows_per_piece;
    const int64_t need = (pieces + kShortWaves - 1) / kShortWaves;
    if (nb > need) nb = need;
    return static_cast<int32_t>(nb < 1 ? 1 : nb);
}

}  // namespace

int32_t qknorm_bwd_blocks(int64_t N, int64_t D, int dtype) {
    const int E = dtype == 0 ? 8 : 4;
    const int nchunks = static_cast<int>(D / E);
    if (nchunks <= kShortMaxChunks) {
        const int r = nchunks <= 16 ? short_bwd_r<1>() : short_bwd_r<2>();
        return short_blocks_per_tensor(N, 4 * r, kShortBwdBlocksPerCu);
    }
    bool ok;
    const Shape sh = wide_shape(nchunks, dtype, true, N, &ok);
    return blocks_per_tensor(N, sh.per_cu);
}

Shape qknorm_table_shape(int nchunks, int dtype, bool backward, int64_t N) {
    return wide_table_shape(nchunks, dtype, backward, N);
}

hipError_t launch_qknorm_fwd(int dtype, const void* q, const void* k, const void* wq, const void* wk,
                             int64_t N, int64_t D, float eps, void* q_out, void* k_out,
                             float* rstd_q, float* rstd_k, hipStream_t st) {
    const int E = dtype == 0 ? 8 : 4;
    QkFwdArgs a;
    a.x[0] = q; a.x[1] = k;
    a.w[0] = wq; a.w[1] = wk;
    a.y[0] = q_out; a.y[1] = k_out;
    a.rstd[0] = rstd_q; a.rstd[1] = rstd_k;
    a.N = N;
    a.D = static_cast<int32_t>(D);
    a.nchunks = static_cast<int32_t>(D / E);
    a.eps = eps;
    a.inv_D = 1.0f / static_cast<float>(D);
    if (a.nchunks <= kShortMaxChunks) {
        const bool one = a.nchunks <= 16;
        a.nb = short_blocks_per_tensor(N, 4 * (one ? short_fwd_r<1>() : short_fwd_r<2>()), kShortFwdBlocksPerCu);
        const dim3 grid(static_cast<unsigned>(2 * a.nb)), block(kShortWaves * kWave);
        if (dtype == 0) {
            if (one) hipLaunchKernelGGL((qknorm_short_fwd_kernel<bf16_io, 1, short_fwd_r<1>()>), grid, block, 0, st, a);
            else hipLaunchKernelGGL((qknorm_short_fwd_kernel<bf16_io, 2, short_fwd_r<2>()>), grid, block, 0, st, a);
        } else {
            if (one) hipLaunchKernelGGL((qknorm_short_fwd_kernel<f32_io, 1, short_fwd_r<1>()>), grid, block, 0, st, a);
            else hipLaunchKernelGGL((qknorm_short_fwd_kernel<f32_io, 2, short_fwd_r<2>()>), grid, block, 0, st, a);
        }
        return hipGetLastError();
    }
    bool ok;
    const Shape sh = wide_shape(a.nchunks, dtype, false, N, &ok);
    if (!ok) return hipErrorInvalidConfiguration;
    const Split sp{sh.K, sh.VPL};
    a.nb = blocks_per_tensor(N, sh.per_cu);
    if (dtype == 0) for_split<bf16_io, 2>(sp, FwdGo<bf16_io>{a, st});
    else for_split<f32_io, 4>(sp, FwdGo<f32_io>{a, st});
    return hipGetLastError();
}

hipError_t launch_qknorm_bwd(int dtype, const void* dq_out, const void* dk_out, const void* q,
                             const void* k, const void* wq, const void* wk, int64_t N, int64_t D,
                             const float* rstd_q, const float* rstd_k, void* dq, void* dk,
                             void* dwq, void* dwk, bool io_grads, float* ws, hipStream_t st) {
    const int E = dtype == 0 ? 8 : 4;
    QkBwdArgs a;
    a.dy[0] = dq_out; a.dy[1] = dk_out;
    a.x[0] = q; a.x[1] = k;
    a.w[0] = wq; a.w[1] = wk;
    a.rstd[0] = rstd_q; a.rstd[1] = rstd_k;
    a.dx[0] = dq; a.dx[1] = dk;
    a.ws = ws;
    a.N = N;
    a.D = static_cast<int32_t>(D);
    a.nchunks = static_cast<int32_t>(D / E);
    a.inv_D = 1.0f / static_cast<float>(D);
    int32_t slots = qknorm_bwd_blocks(N, D, dtype);              // per tensor
    if (a.nchunks <= kShortMaxChunks) {
        const bool one = a.nchunks <= 16;
        a.nb = slots;
        const dim3 grid(static_cast<unsigned>(2 * a.nb)), block(kShortWaves * kWave);
        if (dtype == 0) {
            if (one) hipLaunchKernelGGL((qknorm_short_bwd_kernel<bf16_io, 1, short_bwd_r<1>()>), grid, block, 0, st, a);
            else hipLaunchKernelGGL((qknorm_short_bwd_kernel<bf16_io, 2, short_bwd_r<2>()>), grid, block, 0, st, a);
        } else {
            if (one) hipLaunchKernelGGL((qknorm_short_bwd_kernel<f32_io, 1, short_bwd_r<1>()>), grid, block, 0, st, a);
            else hipLaunchKernelGGL((qknorm_short_bwd_kernel<f32_io, 2, short_bwd_r<2>()>), grid, block, 0, st, a);
        }
    } else {
        bool ok;
        const Shape sh = wide_shape(a.nchunks, dtype, true, N, &ok);
        if (!ok) return hipErrorInvalidConfiguration;
        const Split sp{sh.K, sh.VPL};
        a.nb = slots;
        if (dtype == 0) for_split<bf16_io, 2>(sp, BwdGo<bf16_io>{a, st});
        else for_split<f32_io, 4>(sp, BwdGo<f32_io>{a, st});
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;

    ReduceArgs r{};
    r.ws = ws;
    r.out[0] = dwq;
    r.out[1] = dwk;
    r.out_bf16 = io_grads && dtype == 0;
    r.seg = Segments{nullptr, N, 1};
    r.T = N;
    r.rows_per_cluster = N;
    r.nb = a.nb;
    r.D = a.D;
    r.nsum = 2;
    return launch_reduce(r, 1, st);
}

}  // namespace lnmod
