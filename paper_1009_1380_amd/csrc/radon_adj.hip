// radon_adj.hip - launchers of the adjoint path (A1 ray FFT, A2 binned
// spreading, A3 split-tile sums + column inverse FFT, A4 row inverse FFT),
// dispatched on the FFT length, kernel width and tile size.
#include "radon_internal.hpp"

namespace rn {

hipError_t launch_a1(const Plan& p, const Work& w, const float* sino, bool filtered, hipStream_t st) {
    const float* wq = filtered ? p.fbpw : nullptr;
    const dim3 grid((p.n_views + 1) / 2, w.slices);
    switch (p.n_det) {
#define RN_CASE(L)                                                                             \
    case L: {                                                                                  \
        constexpr int NT = ray_threads(L);                                                     \
        hipLaunchKernelGGL((k_a1_rays<L, NT>), grid, dim3(NT), 0, st, sino, w.Yh, p.tw_N, wq,   \
                           p.n_views, w.sino_n, w.ray_n);                                      \
        break;                                                                                 \
    }
        RN_FOR_LENGTHS(RN_CASE)
#undef RN_CASE
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int W, int T>
static hipError_t launch_a2_wt(const Plan& p, const Work& w, hipStream_t st) {
    if (p.n_items == 0) return hipSuccess;
    hipLaunchKernelGGL((k_a2_spread<W, T>), dim3(p.n_items, w.slices), dim3(A2_NT), 0, st, p.items,
                       p.recs, w.Yh, p.kbc, w.grid, w.partials, p.G, w.ray_n, w.grid_n, w.part_n);
    return hipGetLastError();
}

template <int W>
static hipError_t launch_a2_w(const Plan& p, const Work& w, hipStream_t st) {
    switch (p.T) {
        case 8: return launch_a2_wt<W, 8>(p, w, st);
        case 16: return launch_a2_wt<W, 16>(p, w, st);
        case 32: return launch_a2_wt<W, 32>(p, w, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_a2(const Plan& p, const Work& w, hipStream_t st) {
    switch (p.W) {
        case 4: return launch_a2_w<4>(p, w, st);
        case 6: return launch_a2_w<6>(p, w, st);
        case 8: return launch_a2_w<8>(p, w, st);
        default: return hipErrorInvalidValue;
    }
}

SplitSums split_sums_of(const Plan& p, const float2* partials) {
    return SplitSums{p.splits, p.split_cols, partials, p.T == 32 ? 5 : (p.T == 16 ? 4 : 3)};
}

hipError_t launch_split_sums(const Plan& p, const Work& w, hipStream_t st) {
    switch (p.n) {
#define RN_CASE(L)                                                                             \
    case L:                                                                                    \
        hipLaunchKernelGGL((k_split_sums<L, col_threads(L)>), dim3(p.n + 1), dim3(col_threads(L)), 0, st, w.grid, \
                           split_sums_of(p, w.partials));                                      \
        break;
        RN_FOR_LENGTHS(RN_CASE)
#undef RN_CASE
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_a3(const Plan& p, const Work& w, hipStream_t st) {
    const dim3 grid(p.n + 1, w.slices);
    switch (p.n) {
#define RN_CASE(L)                                                                             \
    case L: {                                                                                  \
        constexpr int NT = col_threads(L);                                                   \
        hipLaunchKernelGGL((k_a3_cols<L, NT>), grid, dim3(NT), 0, st, w.grid, split_sums_of(p, w.partials), \
                           w.T1, p.shift_n, p.tw_n, w.grid_n, w.part_n, w.t1_n);               \
        break;                                                                                 \
    }
        RN_FOR_LENGTHS(RN_CASE)
#undef RN_CASE
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int L, int LINES>
static void launch_a4_l(const Plan& p, const Work& w, float* img, hipStream_t st) {
    constexpr int NT = row_threads(L, LINES);
    hipLaunchKernelGGL((k_a4_rows<L, NT, LINES>), dim3(row_blocks(L, LINES), w.slices), dim3(NT), 0, st, w.T1, img, p.psi_inv,
                       p.shift_n, p.tw_n, w.t1_n, w.img_n);
}

hipError_t launch_a4(const Plan& p, const Work& w, float* img, hipStream_t st) {
    switch (p.n) {
#define RN_CASE(L)                                                                             \
    case L:                                                                                    \
        if (w.slices == 1) launch_a4_l<L, row_lines_alone(L)>(p, w, img, st);                  \
        else launch_a4_l<L, row_lines(L)>(p, w, img, st);                                      \
        break;
        RN_FOR_LENGTHS(RN_CASE)
#undef RN_CASE
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------- batches

hipError_t launch_pass_adj(PassKind kind, int len, const PassSlice* tab, int ns, int nblocks, hipStream_t st) {
    if (ns <= 0 || nblocks <= 0) return hipSuccess;
    switch (len) {
#define RN_CASE(L)                                                                                         \
    case L:                                                                                                \
        switch (kind) {                                                                                    \
            case PK_A1:                                                                                    \
                hipLaunchKernelGGL((k_a1_multi<L, ray_threads(L)>), dim3(nblocks), dim3(ray_threads(L)),   \
                                   0, st, tab, ns);                                                        \
                break;                                                                                     \
            case PK_A3:                                                                                    \
                hipLaunchKernelGGL((k_a3_multi<L, col_threads(L)>), dim3(nblocks), dim3(col_threads(L)),   \
                                   0, st, tab, ns);                                                        \
                break;                                                                                     \
            case PK_A4:                                                                                    \
                hipLaunchKernelGGL((k_a4_multi<L, row_threads(L, row_lines(L))>), dim3(nblocks), dim3(row_threads(L, row_lines(L))),   \
                                   0, st, tab, ns);                                                        \
                break;                                                                                     \
            default:                                                                                       \
                return hipErrorInvalidValue;                                                               \
        }                                                                                                  \
        break;
        RN_FOR_LENGTHS(RN_CASE)
#undef RN_CASE
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int W, int T>
static hipError_t launch_a2m_wt(const GridLaunch& g, const GridSlice* gs, hipStream_t st) {
    if (g.n_items == 0) return hipSuccess;
    hipLaunchKernelGGL((k_a2_multi<W, T>), dim3(g.n_items), dim3(A2_NT), 0, st, g.items, gs, g.kbc);
    return hipGetLastError();
}

template <int W>
static hipError_t launch_a2m_w(const GridLaunch& g, const GridSlice* gs, hipStream_t st) {
    switch (g.T) {
        case 8: return launch_a2m_wt<W, 8>(g, gs, st);
        case 16: return launch_a2m_wt<W, 16>(g, gs, st);
        case 32: return launch_a2m_wt<W, 32>(g, gs, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_a2_grid(const GridLaunch& g, const GridSlice* gs, hipStream_t st) {
    switch (g.W) {
        case 4: return launch_a2m_w<4>(g, gs, st);
        case 6: return launch_a2m_w<6>(g, gs, st);
        case 8: return launch_a2m_w<8>(g, gs, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace rn
