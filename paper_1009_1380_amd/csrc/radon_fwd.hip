// radon_fwd.hip - launchers of the forward path (F1 row FFT, F2 column FFT,
// F3 tiled polar interpolation, F4 ray inverse FFT), dispatched on the FFT
// length, kernel width and tile size: for one slice, and for every slice of
// an uneven batch (radon_multi.hpp).
#include <algorithm>

#include "radon_internal.hpp"

namespace rn {

template <int L, int LINES>
static void launch_f1_l(const Plan& p, const Work& w, const float* img, hipStream_t st) {
    constexpr int NT = row_threads(L, LINES);
    hipLaunchKernelGGL((k_f1_rows<L, NT, LINES>), dim3(row_blocks(L, LINES), w.slices), dim3(NT), 0, st, img, w.T1, p.psi_inv,
                       p.shift_n, p.tw_n, w.img_n, w.t1_n);
}

hipError_t launch_f1(const Plan& p, const Work& w, const float* img, hipStream_t st) {
    switch (p.n) {
#define RN_CASE(L)                                                                             \
    case L:                                                                                    \
        if (w.slices == 1) launch_f1_l<L, row_lines_alone(L)>(p, w, img, st);                  \
        else launch_f1_l<L, row_lines(L)>(p, w, img, st);                                      \
        break;
        RN_FOR_LENGTHS(RN_CASE)
#undef RN_CASE
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_f2(const Plan& p, const Work& w, hipStream_t st) {
    const dim3 grid(p.n + 1, w.slices);
    switch (p.n) {
#define RN_CASE(L)                                                                             \
    case L: {                                                                                  \
        constexpr int NT = col_threads(L);                                                   \
        hipLaunchKernelGGL((k_f2_cols<L, NT>), grid, dim3(NT), 0, st, w.T1, w.grid, p.shift_n,  \
                           p.tw_n, w.t1_n, w.grid_n);                                          \
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
static hipError_t launch_f3_wt(const Plan& p, const Work& w, hipStream_t st) {
    if (p.n_fitems == 0) return hipSuccess;
    const int grid = w.slices == 1 ? p.f3_grid : (int)std::min<int64_t>((int64_t)p.n_fitems * w.slices, p.f3_resident);
    hipLaunchKernelGGL((k_f3_tiles<W, T, 512>), dim3(grid), dim3(512), 0, st, p.fitems, p.n_fitems,
                       p.recs, w.grid, p.kbc, w.Xr, p.G, w.slices, w.grid_n, w.ray_n);
    return hipGetLastError();
}

template <int W, int T>
static int f3_occupancy() {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_f3_tiles<W, T, 512>, 512, 0) != hipSuccess) {
        (void)hipGetLastError();
        return 1;
    }
    return nb > 0 ? nb : 1;
}

template <int W>
static int f3_occupancy_w(int T) {
    switch (T) {
        case 8: return f3_occupancy<W, 8>();
        case 16: return f3_occupancy<W, 16>();
        case 32: return f3_occupancy<W, 32>();
        default: return 1;
    }
}

int f3_blocks_per_cu(int W, int T) {
    switch (W) {
        case 4: return f3_occupancy_w<4>(T);
        case 6: return f3_occupancy_w<6>(T);
        case 8: return f3_occupancy_w<8>(T);
        default: return 1;
    }
}

template <int W>
static hipError_t launch_f3_w(const Plan& p, const Work& w, hipStream_t st) {
    switch (p.T) {
        case 8: return launch_f3_wt<W, 8>(p, w, st);
        case 16: return launch_f3_wt<W, 16>(p, w, st);
        case 32: return launch_f3_wt<W, 32>(p, w, st);
        default: return hipErrorInvalidValue;
    }
}

template <int W>
static hipError_t launch_f3_direct(const Plan& p, const Work& w, hipStream_t st) {
    const int blocks = (int)((p.n_samples + F3D_NT - 1) / F3D_NT);
    hipLaunchKernelGGL(k_f3_direct<W>, dim3(blocks, w.slices), dim3(F3D_NT), 0, st, p.recs, (int)p.n_samples, w.grid, p.kbc,
                       w.Xr, p.G, p.T, w.grid_n, w.ray_n);
    return hipGetLastError();
}

// Interpolate straight from the grid where the samples are few against the grid.
// Direct time grows with the points read (M W^2); staging pays for every region of the
// grid (two dependent rounds of loads and a barrier before the first sample), and
// with W = 8 holds fewer waves. Up to 512^2 pixels in all there are fewer regions than
// two per CU: a staged launch then lasts as long as its fullest region, and direct
// pays up to a fixed number of points. Forward, direct and staged, us: 128^2 pixels,
// W = 6: 4.5e6 points 18.6 and 21.6, 8e6 21.4 and 21.9, 10e6 23.8 and 23.5; 512^2:
// 4.5e6 23.6 and 25.6, 6.5e6 25.7 and 25.7, 8e6 28.5 and 26.7, with W = 8 8e6 27.8
// and 30.3, 10e6 31.9 and 30.1; 1024^2, W = 6: 3.7e6 (100 views) 36.2 and 37.1, 4.7e6
// (128) 36.8 and 37.4, 5.0e6 (135) 38.2 and 37.5, with W = 8 4.4e6 34.9 and 38.5, 5.5e6
// 41.2 and 41.3; 2560^2, W = 6: 7.7e6 80.2 and 87.0, 11.5e6 86.7 and 86.9, 15.4e6
// 91.0 and 86.9; four slices of 1024^2: 5.3e6 57.2 and 60.4, 8e6 60.6 and 60.5,
// 10.8e6 64.0 and 61.8. Over 338 plans and stacks on both sides of these lines the
// choice is 0.7% over the better of the two on average.
static bool f3_is_direct(const Plan& p, int slices) {
    const double s = slices, points = s * (double)p.n_samples * p.W * p.W, pixels = s * (double)p.n * p.n;
    const bool wide = p.W == 8;
    if (pixels <= 512.0 * 512.0) return points < (wide ? 9e6 : 6e6);
    return points < (wide ? 3e6 + 2.5 * pixels : 3.5e6 + 1.25 * pixels);
}

hipError_t launch_f3(const Plan& p, const Work& w, hipStream_t st) {
    if (f3_is_direct(p, w.slices)) switch (p.W) {
        case 4: return launch_f3_direct<4>(p, w, st);
        case 6: return launch_f3_direct<6>(p, w, st);
        case 8: return launch_f3_direct<8>(p, w, st);
        default: return hipErrorInvalidValue;
    }
    switch (p.W) {
        case 4: return launch_f3_w<4>(p, w, st);
        case 6: return launch_f3_w<6>(p, w, st);
        case 8: return launch_f3_w<8>(p, w, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_f4(const Plan& p, const Work& w, float* sino, hipStream_t st) {
    const dim3 grid((p.n_views + 1) / 2, w.slices);
    switch (p.n_det) {
#define RN_CASE(L)                                                                             \
    case L: {                                                                                  \
        constexpr int NT = ray_threads(L);                                                     \
        hipLaunchKernelGGL((k_f4_rays<L, NT>), grid, dim3(NT), 0, st, w.Xr, sino, p.tw_N,       \
                           p.n_views, w.ray_n, w.sino_n);                                      \
        break;                                                                                 \
    }
        RN_FOR_LENGTHS(RN_CASE)
#undef RN_CASE
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------- batches

hipError_t launch_pass_fwd(PassKind kind, int len, const PassSlice* tab, int ns, int nblocks, hipStream_t st) {
    if (ns <= 0 || nblocks <= 0) return hipSuccess;
    switch (len) {
#define RN_CASE(L)                                                                                         \
    case L:                                                                                                \
        switch (kind) {                                                                                    \
            case PK_F1:                                                                                    \
                hipLaunchKernelGGL((k_f1_multi<L, row_threads(L, row_lines(L))>), dim3(nblocks), dim3(row_threads(L, row_lines(L))),   \
                                   0, st, tab, ns);                                                        \
                break;                                                                                     \
            case PK_F2:                                                                                    \
                hipLaunchKernelGGL((k_f2_multi<L, col_threads(L)>), dim3(nblocks), dim3(col_threads(L)),   \
                                   0, st, tab, ns);                                                        \
                break;                                                                                     \
            case PK_F4:                                                                                    \
                hipLaunchKernelGGL((k_f4_multi<L, ray_threads(L)>), dim3(nblocks), dim3(ray_threads(L)),   \
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

hipError_t launch_pass(PassKind kind, int len, const PassSlice* tab, int ns, int nblocks, hipStream_t st) {
    if (kind == PK_F1 || kind == PK_F2 || kind == PK_F4) return launch_pass_fwd(kind, len, tab, ns, nblocks, st);
    return launch_pass_adj(kind, len, tab, ns, nblocks, st);
}

PassSlice pass_slice_of(const Plan& p, PassKind kind, const void* in, void* out) {
    PassSlice e{};
    e.block0 = 0;
    e.n_views = p.n_views;
    e.psi_inv = p.psi_inv;
    e.shift = p.shift_n;
    e.wq = nullptr;
    switch (kind) {
        case PK_F1: e.nblk = row_blocks(p.n, row_lines(p.n)); e.in = in; e.out = p.T1; e.tw = p.tw_n; break;
        case PK_F2: e.nblk = p.n + 1; e.in = p.T1; e.out = p.grid; e.tw = p.tw_n; break;
        case PK_F4: e.nblk = (p.n_views + 1) / 2; e.in = p.Xr; e.out = out; e.tw = p.tw_N; break;
        case PK_A1: e.nblk = (p.n_views + 1) / 2; e.in = in; e.out = p.Yh; e.tw = p.tw_N; break;
        case PK_A3: e.nblk = p.n + 1; e.in = p.grid; e.out = p.T1; e.tw = p.tw_n; e.sums = split_sums_of(p, p.partials); break;
        case PK_A4: e.nblk = row_blocks(p.n, row_lines(p.n)); e.in = p.T1; e.out = out; e.tw = p.tw_n; break;
    }
    return e;
}

GridSlice grid_slice_of(const Plan& p) { return GridSlice{p.recs, p.grid, p.Xr, p.Yh, p.partials, p.G, 0}; }

template <int W, int T>
static hipError_t launch_f3m_wt(const GridLaunch& g, const GridSlice* gs, hipStream_t st) {
    if (g.n_fitems == 0) return hipSuccess;
    hipLaunchKernelGGL((k_f3_multi<W, T, 512>), dim3(g.f3_grid), dim3(512), 0, st, g.fitems, g.n_fitems, gs, g.kbc);
    return hipGetLastError();
}

template <int W>
static hipError_t launch_f3m_w(const GridLaunch& g, const GridSlice* gs, hipStream_t st) {
    switch (g.T) {
        case 8: return launch_f3m_wt<W, 8>(g, gs, st);
        case 16: return launch_f3m_wt<W, 16>(g, gs, st);
        case 32: return launch_f3m_wt<W, 32>(g, gs, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_f3_grid(const GridLaunch& g, const GridSlice* gs, hipStream_t st) {
    switch (g.W) {
        case 4: return launch_f3m_w<4>(g, gs, st);
        case 6: return launch_f3m_w<6>(g, gs, st);
        case 8: return launch_f3m_w<8>(g, gs, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace rn
