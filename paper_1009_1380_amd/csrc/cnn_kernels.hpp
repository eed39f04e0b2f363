// cnn_kernels.hpp - kernels of the learned warm start: a small BF16
// convolutional encoder-decoder that maps the filtered adjoint of a sinogram
// to a start image for the basis-pursuit solve (gfx950).
//
// Activations are bfloat16 in planes of eight channels, [image][C/8][y][x][8]:
// one 16-byte piece holds eight channels of a pixel, and consecutive pixels
// are consecutive pieces. Every product is accumulated in float32. 3x3
// convolutions are implicit GEMMs on v_mfma_f32_32x32x8_bf16 (M = output
// channels, N = pixels, K = input channels x 9 taps in the order k =
// 9 channel + tap, eight values of K per instruction in ascending order). The
// order is part of the network's definition: activations are rounded to
// bfloat16 after every layer, so a different order of the float32 sums flips
// an occasional rounding, and the flips spread through the layers that follow
// (measured: 3e-4 of the output with the 16-wide instruction and a
// tap-by-tap order). Operand layout of the instruction (lane l of 64, t =
// 0..3): A holds row l % 32, values 4 (l / 32) + t of K; B column l % 32, the
// same values; the 16 results of lane l are rows 8 (r / 4) + 4 (l / 32) +
// (r % 4), column l % 32.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cnn {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// float -> bfloat16 bits, round to nearest even
__device__ __forceinline__ uint16_t f2bf(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }
__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
// two floats -> two packed bfloat16 (the first in the low half)
__device__ __forceinline__ uint32_t pack2(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){a, b}, bf16x2));
}
__device__ __forceinline__ float lo2f(uint32_t v) { return __uint_as_float(v << 16); }
__device__ __forceinline__ float hi2f(uint32_t v) { return __uint_as_float(v & 0xffff0000u); }
__device__ __forceinline__ f32x16 mfma(uint32_t a0, uint32_t a1, uint32_t b0, uint32_t b1, const f32x16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(__builtin_bit_cast(bf16x4, make_uint2(a0, a1)),
                                                    __builtin_bit_cast(bf16x4, make_uint2(b0, b1)), c, 0, 0, 0);
}

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own L2.
// Renumber block b of nb so that each XCD gets a contiguous run of tiles: the
// neighbours that share window rows and cache lines then meet in one L2.
__device__ __forceinline__ int xcd_block(int b, int nb) {
    const int x = b & 7, k = b >> 3, per = nb >> 3, rem = nb & 7;
    return x * per + min(x, rem) + k;
}

// Workgroup barrier that waits for LDS traffic only; loads from global memory
// stay in flight across it and are waited for where they are used.
__device__ __forceinline__ void lds_sync() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Sums over the 2 x 2 pixels of a block, row by row, for eight channels of the 16 x
// 2 pixel block that a wave half's lanes hold (lane bits 0..3: x, bit 4: y): in
// even lanes, channels 0..3 where bit 4 is clear, channels 4..7 where it is set.
// One v_permlane16_swap_b32 gives a lane both rows of one of two channels.
__device__ __forceinline__ float right_of(float v) {   // the lane whose index differs in bit 0
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true));
}
__device__ __forceinline__ void sum4(const float (&a)[8], float (&s)[4]) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a[t]), __float_as_uint(a[t + 4]), false, false);
        const float top = __uint_as_float(r[0]), bot = __uint_as_float(r[1]);
        s[t] = ((top + right_of(top)) + bot) + right_of(bot);
    }
}

// a and b after the upper 32 lanes of a and the lower 32 of b have changed places.
__device__ __forceinline__ uint2 swap_halves(uint32_t a, uint32_t b) {
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    return make_uint2(r[0], r[1]);
}

// max(v, 0) in one instruction (0 for a NaN; fmaxf adds a canonicalising one,
// which the results of a matrix instruction do not need)
__device__ __forceinline__ float relu(float v) {
    float r;
    asm("v_max_f32 %0, 0, %1" : "=v"(r) : "v"(v));
    return r;
}

// One bit per channel of a piece: the value is not zero.
__device__ __forceinline__ unsigned nonzero_bits(uint4 v) {
    // the magnitude plus 0x7fff carries into bit 15 unless it is zero
    auto one = [](uint32_t d) { return ((d & 0x7fff7fffu) + 0x7fff7fffu) & 0x80008000u; };
    const uint32_t m = (one(v.x) >> 6 | one(v.y) >> 4 | one(v.z) >> 2 | one(v.w)) >> 9;   // bits 0, 2, 4, 6 and 16, 18, ..
    return (m | m >> 15) & 0xffu;
}

// A piece with the channels whose bit of m is clear set to zero.
__device__ __forceinline__ uint4 mask_piece(uint4 v, unsigned m) {
    auto two = [&](unsigned b) { return ((b & 1u) ? 0xffffu : 0u) | ((b & 2u) ? 0xffff0000u : 0u); };
    return make_uint4(v.x & two(m), v.y & two(m >> 2), v.z & two(m >> 4), v.w & two(m >> 6));
}

// ---------------------------------------------------------------- epilogues
// What happens to a 32 x 32 block of results (32 channels of a 16 x 2 pixel
// block), as the kernels below leave it in a wave's registers.
//   EPI_ACT    act = [relu](sum + bias), rounded to bf16; mask (if given, with
//              relu) gets the bits act > 0 (a byte per piece); pool (if given) the 2x2
//              averages of act; out gets act, or act + skip if skip is given
//   EPI_SUM4   gradient through a nearest 2x upsampling: the sums over 2x2
//              pixels of the results rounded to bf16, to out at half the size
//   EPI_POOLG  gradient through a 2x2 average pooling and the ReLU before it,
//              joined by a second gradient `skip`: out = (skip + result / 4)
//              where mask's bit is set, else 0, at twice the size
//   EPI_F32    the sums themselves, float32 pieces, to out32
//   EPI_ONE    the first channel alone, float32: out32 = sum + bias + res32
//              (either may be null), an H x W image per batch entry
enum { EPI_ACT, EPI_SUM4, EPI_POOLG, EPI_F32, EPI_ONE };

struct Epilogue {
    const float* bias;
    int relu;
    uint16_t* out;
    uint8_t* mask;
    uint16_t* pool;
    const uint16_t* skip;
    float* out32;
    const float* res32;
};

// acc: the block's results; plane0: plane of its first channel (of P); (gy, gx):
// this lane's pixel of an H x W image; i = lane % 32, kh = lane / 32.
template <int EPI>
__device__ __forceinline__ void epilogue(const Epilogue& e, const f32x16& acc, int b, int P, int plane0, int gy, int gx,
                                         int H, int W, int i, int kh) {
    const bool ok = gy < H && gx < W;
    if constexpr (EPI == EPI_ONE) {
        if (ok && kh == 0) {
            const size_t o = ((size_t)b * H + gy) * W + gx;
            float v = acc[0];
            if (e.bias) v += e.bias[0];
            if (e.res32) v += e.res32[o];
            e.out32[o] = v;
        }
        return;
    }
    if constexpr (EPI == EPI_F32) {
#pragma unroll
        for (int g = 0; g < 4; ++g)
            if (ok)
                reinterpret_cast<float4*>(e.out32)[((((size_t)b * P + plane0 + g) * H + gy) * W + gx) * 2 + kh] =
                    make_float4(acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]);
        return;
    }
    // A lane has channels 4 kh .. 4 kh + 3 of four planes; the halves of the wave
    // exchange them so that each has whole pieces of two planes (2 gp + kh).
#pragma unroll
    for (int gp = 0; gp < 2; ++gp) {
        uint2 h[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int g = 2 * gp + u;
            float v[4] = {acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
            if constexpr (EPI == EPI_ACT) {
                if (e.bias) {
                    const float4 bv = *reinterpret_cast<const float4*>(e.bias + (plane0 + g) * 8 + 4 * kh);
                    v[0] += bv.x; v[1] += bv.y; v[2] += bv.z; v[3] += bv.w;
                }
                if (e.relu) {
#pragma unroll
                    for (int t = 0; t < 4; ++t) v[t] = relu(v[t]);
                }
            }
            h[u] = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
        }
        const uint2 p0 = swap_halves(h[0].x, h[1].x), p1 = swap_halves(h[0].y, h[1].y);
        uint4 r = make_uint4(p0.x, p1.x, p0.y, p1.y);
        const float a[8] = {lo2f(r.x), hi2f(r.x), lo2f(r.y), hi2f(r.y), lo2f(r.z), hi2f(r.z), lo2f(r.w), hi2f(r.w)};
        auto piece = [](const float (&f)[8]) {
            return make_uint4(pack2(f[0], f[1]), pack2(f[2], f[3]), pack2(f[4], f[5]), pack2(f[6], f[7]));
        };
        const size_t pl = (size_t)b * P + plane0 + 2 * gp + kh;
        const size_t half = (pl * (H / 2) + gy / 2) * (W / 2) + gx / 2;   // the pixel's 2x2 block
        if constexpr (EPI == EPI_ACT) {
            const size_t o = (pl * H + gy) * W + gx;
            if (e.mask) {
                const unsigned m = nonzero_bits(r);
                if (ok) e.mask[o] = (uint8_t)m;
            }
            if (e.pool) {
                float s[4];
                sum4(a, s);
                if (ok && !(i & 1))
                    reinterpret_cast<uint2*>(e.pool)[half * 2 + (i >> 4)] =
                        make_uint2(pack2(0.25f * s[0], 0.25f * s[1]), pack2(0.25f * s[2], 0.25f * s[3]));
            }
            if (ok) {
                if (e.skip) {
                    const uint4 q = reinterpret_cast<const uint4*>(e.skip)[o];
                    const float s[8] = {a[0] + lo2f(q.x), a[1] + hi2f(q.x), a[2] + lo2f(q.y), a[3] + hi2f(q.y),
                                        a[4] + lo2f(q.z), a[5] + hi2f(q.z), a[6] + lo2f(q.w), a[7] + hi2f(q.w)};
                    r = piece(s);
                }
                reinterpret_cast<uint4*>(e.out)[o] = r;
            }
        } else if constexpr (EPI == EPI_SUM4) {
            float s[4];
            sum4(a, s);
            if (ok && !(i & 1))
                reinterpret_cast<uint2*>(e.out)[half * 2 + (i >> 4)] = make_uint2(pack2(s[0], s[1]), pack2(s[2], s[3]));
        } else {   // EPI_POOLG
            if (ok) {
                float q[8];
#pragma unroll
                for (int t = 0; t < 8; ++t) q[t] = bf2f(f2bf(0.25f * a[t]));
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const size_t px = (pl * 2 * H + 2 * gy + (c >> 1)) * (2 * W) + 2 * gx + (c & 1);
                    const uint4 g = reinterpret_cast<const uint4*>(e.skip)[px];
                    const unsigned m = e.mask[px];
                    const float s[8] = {lo2f(g.x) + q[0], hi2f(g.x) + q[1], lo2f(g.y) + q[2], hi2f(g.y) + q[3],
                                        lo2f(g.z) + q[4], hi2f(g.z) + q[5], lo2f(g.w) + q[6], hi2f(g.w) + q[7]};
                    reinterpret_cast<uint4*>(e.out)[px] = mask_piece(piece(s), m);
                }
            }
        }
    }
}

// ---------------------------------------------------------------- convolution
// Implicit-GEMM 3x3 convolution, stride 1, zero padding 1, of an image of
// Pin planes into CoutP channels (a multiple of CB); H x W is the size of the
// result. With UP the input is H/2 x W/2 and is read as its nearest 2x
// upsampling; with a mask the input's pieces are masked as they are read (the
// gradient through a ReLU).
//
// A workgroup takes CB output channels and a 16 x TY pixel tile, its four
// waves MW x NW blocks of 32 channels x (16 x 2) pixels each. The reduction
// runs over chunks of 16 input channels: the chunk's input window (zero
// outside the image) and its weights are staged in LDS, one buffer being
// filled while the other is multiplied (the next chunk's loads are in flight
// during the products).
//
// A lane's operand is, for its pixel, the values k = 8 s + 4 h + t of K (h its
// half of the wave), which run through the taps of one channel before the
// next. Half h reads the nine pieces of the pixel's neighbourhood in plane h of
// the chunk (16-byte reads of consecutive pieces, no bank conflicts), picks the
// values that either half needs of it out in registers (one v_perm_b32 per two
// values), and v_permlane32_swap_b32 gives each half its own of both planes:
// every piece is read once per pixel. A wave of 2 x 2 blocks then reads 36 KB of
// LDS per 72 matrix instructions.
// Blocks of 32 channels have half the products per LDS byte and are bound by
// latency: three waves per SIMD (at most 168 VGPRs) took the layer of 64 -> 32
// channels at 512 x 512 from 199 to 158 us at batch 8.
// Measured (256 -> 128 channels on upsampled 128 x 128, batch 8, 77 GFLOP): 108
// us, 0.72 PFLOP/s of the about 1.25 that this instruction reaches; 350 us for
// the convolution and 61 us for the upsampling when every operand was four
// 2-byte LDS reads and the loads were not overlapped; 125 us with every piece
// read by both halves.
// Grid: x = image tiles, y = channel blocks of CB.
constexpr int CONV_NT = 256;
constexpr int TX = 16;   // pixel tile width

struct ConvIn {
    const uint4* in;       // pieces
    const uint8_t* mask;   // a byte per piece, or null
    const uint4* w;        // [16-channel chunk][pair of instructions][half][CoutP] pieces
    int Pin, CoutP, H, W;
};

template <int CB, int TY, bool UP, int EPI>
__global__ __launch_bounds__(CONV_NT) __attribute__((amdgpu_waves_per_eu(CB == 32 ? 3 : 2))) void k_conv3x3(
    ConvIn a, Epilogue ep) {
    constexpr int WY = UP ? TY / 2 + 2 : TY + 2, WX = UP ? TX / 2 + 2 : TX + 2, WIN = WY * WX;
    constexpr int NX = 2 * WIN, NA = 18 * CB;                    // pieces per chunk: window, weights
    constexpr int RX = (NX + CONV_NT - 1) / CONV_NT, RA = (NA + CONV_NT - 1) / CONV_NT;
    constexpr int WM = (CB == 64 && TY < 16) ? 2 : 1;            // waves along the channels
    constexpr int MW = CB / 32 / WM, NW = TY / 2 / (4 / WM);     // blocks of a wave
    static_assert(MW >= 1 && NW >= 1, "tile too small for four waves");
    __shared__ uint4 sx[2][NX];
    __shared__ uint4 sa[2][NA];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tiles_x = (a.W + TX - 1) / TX, tiles = tiles_x * ((a.H + TY - 1) / TY);
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    const int b = blk / tiles, tr = blk - b * tiles;
    const int ty0 = (tr / tiles_x) * TY, tx0 = (tr - (tr / tiles_x) * tiles_x) * TX;
    const int cb = blockIdx.y * CB;
    const int Hi = UP ? a.H / 2 : a.H, Wi = UP ? a.W / 2 : a.W, HWi = Hi * Wi;
    const int wy0 = (UP ? ty0 / 2 : ty0) - 1, wx0 = (UP ? tx0 / 2 : tx0) - 1;

    // this thread's pieces of a chunk: their place in the first chunk, -1 for zero
    int xo[RX], ao[RA];
#pragma unroll
    for (int k = 0; k < RX; ++k) {
        const int e = tid + k * CONV_NT;
        const int pl = e / WIN, r = e - pl * WIN, y = wy0 + r / WX, x = wx0 + r % WX;
        xo[k] = (e < NX && y >= 0 && y < Hi && x >= 0 && x < Wi) ? pl * HWi + y * Wi + x : -1;
    }
#pragma unroll
    for (int k = 0; k < RA; ++k) {
        const int e = tid + k * CONV_NT;
        ao[k] = e < NA ? (e / CB) * a.CoutP + cb + e % CB : -1;
    }
    const size_t img = (size_t)b * a.Pin * HWi;
    uint4 vx[RX], va[RA];
    unsigned vm[RX] = {};
    auto load = [&](int c) {
        const uint4* px = a.in + img + (size_t)(2 * c) * HWi;
        const uint4* pa = a.w + (size_t)c * 18 * a.CoutP;
#pragma unroll
        for (int k = 0; k < RX; ++k) {
            vx[k] = make_uint4(0u, 0u, 0u, 0u);
            if (xo[k] >= 0) {
                vx[k] = px[xo[k]];
                if (a.mask) vm[k] = a.mask[img + (size_t)(2 * c) * HWi + xo[k]];
            }
        }
#pragma unroll
        for (int k = 0; k < RA; ++k)
            va[k] = ao[k] >= 0 ? pa[ao[k]] : make_uint4(0u, 0u, 0u, 0u);
    };
    auto store = [&](int s) {
#pragma unroll
        for (int k = 0; k < RX; ++k) {
            const int e = tid + k * CONV_NT;
            if (e < NX) sx[s][e] = a.mask ? mask_piece(vx[k], vm[k]) : vx[k];
        }
#pragma unroll
        for (int k = 0; k < RA; ++k)
            if (tid + k * CONV_NT < NA) sa[s][tid + k * CONV_NT] = va[k];
    };

    const int i = lane & 31, kh = lane >> 5;
    const int px = i & 15, wm = wave % WM, wn = wave / WM;
    const int py = wn * NW * 2 + (i >> 4);                       // tile row of the wave's first block
    // window offsets of this lane's pixel under the taps' rows and columns
    int oy[3], ox[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        oy[d] = (UP ? ((py + d - 1) >> 1) + 1 : py + d) * WX;
        ox[d] = kh * WIN + (UP ? ((px + d - 1) >> 1) + 1 : px + d);
    }
    constexpr int NSTEP = (UP ? 1 : 2) * WX;                     // window rows of two tile rows
    f32x16 acc[MW][NW] = {};
    const int nc = a.Pin / 2;
    load(0);
    store(0);
    lds_sync();
    for (int c = 0; c < nc; ++c) {
        if (c + 1 < nc) load(c + 1);
        const uint4* x = sx[c & 1];
        const uint4* w = sa[c & 1] + kh * CB + wm * MW * 32 + i;
        uint32_t fx[2][NW][9][2];   // [plane][block][instruction][dword]
#pragma unroll
        for (int n = 0; n < NW; ++n) {
            uint32_t v[9][4];
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                const uint4 q = x[oy[t / 3] + ox[t % 3] + n * NSTEP];
                v[t][0] = q.x; v[t][1] = q.y; v[t][2] = q.z; v[t][3] = q.w;
            }
            // values k, k + 1 of this lane's plane
            auto pick = [&](int k) {
                const int c0 = k / 9, t0 = k % 9, c1 = (k + 1) / 9, t1 = (k + 1) % 9;
                return __builtin_amdgcn_perm(v[t1][c1 >> 1], v[t0][c0 >> 1],
                                             ((c1 & 1) ? 0x07060000u : 0x05040000u) | ((c0 & 1) ? 0x0302u : 0x0100u));
            };
#pragma unroll
            for (int s = 0; s < 9; ++s)
#pragma unroll
                for (int d = 0; d < 2; ++d) {
                    const uint2 r = swap_halves(pick(8 * s + 2 * d), pick(8 * s + 4 + 2 * d));
                    fx[0][n][s][d] = r.x;
                    fx[1][n][s][d] = r.y;
                }
        }
        uint4 fa[MW];
#pragma unroll
        for (int S = 0; S < 18; ++S) {
            if (S % 2 == 0) {
#pragma unroll
                for (int m = 0; m < MW; ++m) fa[m] = w[S * CB + m * 32];
            }
#pragma unroll
            for (int m = 0; m < MW; ++m)
#pragma unroll
                for (int n = 0; n < NW; ++n)
                    acc[m][n] = S % 2 == 0 ? mfma(fa[m].x, fa[m].y, fx[S / 9][n][S % 9][0], fx[S / 9][n][S % 9][1], acc[m][n])
                                           : mfma(fa[m].z, fa[m].w, fx[S / 9][n][S % 9][0], fx[S / 9][n][S % 9][1], acc[m][n]);
        }
        if (c + 1 < nc) store((c + 1) & 1);
        lds_sync();
    }
#pragma unroll
    for (int m = 0; m < MW; ++m)
#pragma unroll
        for (int n = 0; n < NW; ++n)
            epilogue<EPI>(ep, acc[m][n], b, a.CoutP / 8, (cb + (wm * MW + m) * 32) / 8, ty0 + py + 2 * n, tx0 + px, a.H,
                          a.W, i, kh);
}

// One input channel, 32 output channels: the nine taps take two matrix
// instructions per 32 x (16 x 2) block. Bound by writing the result (the
// forward at batch 8, 512 x 512: 185 MB in 55 us; 26 us without mask and pool).
// T: float
// (rounded to bf16 as it is read) or uint16_t (bf16). w: [half][32] pieces,
// values 0..3 are taps 4 h .., value 4 of half 0 is tap 8.
// Grid: x = image tiles of 16 x 16.
__device__ __forceinline__ uint16_t to_bits(float v) { return f2bf(v); }
__device__ __forceinline__ uint16_t to_bits(uint16_t v) { return v; }

template <class T, int EPI>
__global__ __launch_bounds__(CONV_NT) __attribute__((amdgpu_waves_per_eu(6))) void k_conv3x3_c1(
    const T* __restrict__ in, const uint4* __restrict__ w, int H, int W, Epilogue ep) {
    __shared__ uint16_t sx[18 * 18];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tiles_x = (W + 15) / 16, tiles = tiles_x * ((H + 15) / 16);
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    const int b = blk / tiles, tr = blk - b * tiles;
    const int ty0 = (tr / tiles_x) * 16, tx0 = (tr - (tr / tiles_x) * tiles_x) * 16;
    for (int e = tid; e < 18 * 18; e += CONV_NT) {
        const int y = ty0 + e / 18 - 1, x = tx0 + e % 18 - 1;
        sx[e] = (y >= 0 && y < H && x >= 0 && x < W) ? to_bits(in[((size_t)b * H + y) * W + x]) : (uint16_t)0;
    }
    const int i = lane & 31, kh = lane >> 5, px = i & 15;
    const uint4 fa = w[kh * 32 + i];
    int off[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) off[t] = ((4 * kh + t) / 3) * 18 + (4 * kh + t) % 3;
    lds_sync();
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        const int py = (wave * 2 + n) * 2 + (i >> 4), p = py * 18 + px;
        const uint32_t d0 = sx[p + off[0]] | ((uint32_t)sx[p + off[1]] << 16);
        const uint32_t d1 = sx[p + off[2]] | ((uint32_t)sx[p + off[3]] << 16);
        const uint32_t t8 = kh ? 0u : sx[p + 2 * 18 + 2];
        f32x16 acc = {};
        acc = mfma(fa.x, fa.y, d0, d1, acc);
        acc = mfma(fa.z, fa.w, t8, 0u, acc);
        epilogue<EPI>(ep, acc, b, 4, 0, ty0 + py, tx0 + px, H, W, i, kh);
    }
}

// ---------------------------------------------------------------- weight gradient
// part[chunk][tap][co][ci] = sum over the chunk's pixels p of g[co][p] in[ci][p + tap]
// (M = output channels, N = input channels, the reduction over pixels). A
// chunk is WG_TILES tiles of 8 x 8 pixels, image by image, tiles in row order;
// within a tile one instruction takes the eight pixels of a row. That order is
// fixed (the chunks are then added in order by k_sum_chunks), so the result
// does not depend on how the channels and taps are spread over waves.
//
// A workgroup takes COB output x CIB input channels of one chunk; each wave
// takes 32 x 32 channels and the three taps of one kernel row. Operands are
// four pixels of one channel, so the pieces (eight channels of one pixel) are
// transposed two pixels at a time in registers on their way to LDS. A lane's
// input row is the six pixels around its four (one 16-byte read); the operands
// of the taps left and right of the centre are dword pairs of it, the centre's
// two funnel shifts. The next tile's loads are in flight during the products.
// Channels sit at a swizzled place (wg_pos), so that the transposed writes
// spread over the banks.
// Measured (64 -> 32 channels at 512 x 512, batch 8, 77 GFLOP): 169 us against
// 1191 us with 2-byte operand reads and one tile in flight; 256 -> 128 at 128 x
// 128: 144 against 511 us.
// Grid: x = chunks, y = blocks of CIB input channels, z = of COB output channels.
constexpr int WG_TILES = 64;

__device__ __forceinline__ int wg_pos(int c) { return (c & ~7) | ((c & 7) ^ ((c >> 3) & 7)); }

// Channel c of the pieces of two neighbouring pixels.
__device__ __forceinline__ uint32_t pair_of(uint4 p, uint4 q, int c) {
    const uint32_t a = c < 2 ? p.x : c < 4 ? p.y : c < 6 ? p.z : p.w;
    const uint32_t d = c < 2 ? q.x : c < 4 ? q.y : c < 6 ? q.z : q.w;
    return __builtin_amdgcn_perm(d, a, (c & 1) ? 0x07060302u : 0x05040100u);
}

struct WgradArgs {
    const uint4* g;          // gradient pieces, Pg planes
    const uint8_t* gmask;    // or null
    const uint4* in;         // input pieces, Pi planes, H x W (UP: H/2 x W/2)
    int Pg, Pi, B, H, W, Cout, Cin;
    float* part;
};

constexpr int wgrad_threads(int cob, int cib) { return cob / 32 * (cib / 32) * 3 * 64; }

template <int COB, int CIB, bool UP>
__global__ __launch_bounds__(wgrad_threads(COB, CIB)) void k_conv3x3_wgrad(WgradArgs a) {
    constexpr int NT = wgrad_threads(COB, CIB);
    constexpr int NG = COB / 8 * 8 * 4, NX = CIB / 8 * 10 * 5;   // pixel pairs: planes x rows x pairs
    constexpr int RU = (NG + NX + NT - 1) / NT;
    constexpr int GROW = COB * 4, XROW = 2 * CIB * 4;            // dwords per tile row
    __shared__ __align__(16) uint32_t sh[2][8 * GROW + 10 * XROW];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tiles_x = (a.W + 7) / 8, tiles = tiles_x * ((a.H + 7) / 8);
    const int ntiles = a.B * tiles;
    const int cb = blockIdx.z * COB, ib = blockIdx.y * CIB;
    const int Hi = UP ? a.H / 2 : a.H, Wi = UP ? a.W / 2 : a.W;

    // this thread's pixel pairs: gradient rows 0..7, pixels 2 pr, 2 pr + 1; input
    // rows -1..8, pixels 2 pr - 1, 2 pr
    int upl[RU], urow[RU], upr[RU];
    bool isg[RU], has[RU];
#pragma unroll
    for (int k = 0; k < RU; ++k) {
        const int e = tid + k * NT;
        isg[k] = e < NG;
        const int u = isg[k] ? e : e - NG, np = isg[k] ? COB / 8 : CIB / 8, npr = isg[k] ? 4 : 5;
        upl[k] = u % np;
        upr[k] = (u / np) % npr;
        urow[k] = u / np / npr;
        has[k] = e < NG + NX;
    }
    uint4 v[RU][2];
    unsigned mk[RU][2] = {};
    auto load = [&](int t) {
        const int b = t / tiles, tr = t - b * tiles;
        const int y0 = (tr / tiles_x) * 8, x0 = (tr - (tr / tiles_x) * tiles_x) * 8;
#pragma unroll
        for (int k = 0; k < RU; ++k) {
            const int plane = (isg[k] ? cb : ib) / 8 + upl[k], y = y0 + urow[k] - (isg[k] ? 0 : 1);
            const bool ok = has[k] && plane < (isg[k] ? a.Pg : a.Pi) && y >= 0 && y < a.H;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int x = x0 + 2 * upr[k] + j - (isg[k] ? 0 : 1);
                v[k][j] = make_uint4(0u, 0u, 0u, 0u);
                if (ok && x >= 0 && x < a.W) {
                    if (isg[k]) {
                        const size_t o = (((size_t)b * a.Pg + plane) * a.H + y) * a.W + x;
                        v[k][j] = a.g[o];
                        if (a.gmask) mk[k][j] = a.gmask[o];
                    } else {
                        v[k][j] = a.in[(((size_t)b * a.Pi + plane) * Hi + (UP ? y >> 1 : y)) * Wi + (UP ? x >> 1 : x)];
                    }
                }
            }
        }
    };
    auto store = [&](uint32_t* buf) {
#pragma unroll
        for (int k = 0; k < RU; ++k) {
            if (!has[k]) continue;
            if (isg[k]) {
                // [row pair][half][channel] pieces: the four pixels of the pair's rows
                if (a.gmask) {
                    v[k][0] = mask_piece(v[k][0], mk[k][0]);
                    v[k][1] = mask_piece(v[k][1], mk[k][1]);
                }
                uint32_t* d = buf + ((urow[k] >> 1) * 2 + (upr[k] >> 1)) * COB * 4 + (urow[k] & 1) * 2 + (upr[k] & 1);
#pragma unroll
                for (int c = 0; c < 8; ++c) d[wg_pos(upl[k] * 8 + c) * 4] = pair_of(v[k][0], v[k][1], c);
            } else {
                // [row][half][channel] pieces: pairs 0..2 to half 0, 2..4 to half 1
                uint32_t* d = buf + 8 * GROW + urow[k] * XROW;
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const uint32_t p = pair_of(v[k][0], v[k][1], c);
                    const int at = wg_pos(upl[k] * 8 + c) * 4;
                    if (upr[k] <= 2) d[at + upr[k]] = p;
                    if (upr[k] >= 2) d[CIB * 4 + at + upr[k] - 2] = p;
                }
            }
        }
    };

    const int i = lane & 31, kh = lane >> 5;
    const int dy = wave % 3, wmn = wave / 3, wm = wmn % (COB / 32), wn = wmn / (COB / 32);
    const int go = kh * COB * 4 + wg_pos(wm * 32 + i) * 4;
    const int xo = 8 * GROW + dy * XROW + kh * CIB * 4 + wg_pos(wn * 32 + i) * 4;
    f32x16 acc[3] = {};
    const int t0 = blockIdx.x * WG_TILES, t1 = min(t0 + WG_TILES, ntiles);
    load(t0);
    store(sh[0]);
    lds_sync();
    for (int t = t0; t < t1; ++t) {
        if (t + 1 < t1) load(t + 1);
        const uint32_t* buf = sh[(t - t0) & 1];
        uint4 ga;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            if (r % 2 == 0) ga = *reinterpret_cast<const uint4*>(buf + go + (r >> 1) * 2 * COB * 4);
            const uint32_t a0 = r % 2 ? ga.z : ga.x, a1 = r % 2 ? ga.w : ga.y;
            const uint4 q = *reinterpret_cast<const uint4*>(buf + xo + r * XROW);
            acc[0] = mfma(a0, a1, q.x, q.y, acc[0]);
            acc[1] = mfma(a0, a1, __builtin_amdgcn_alignbit(q.y, q.x, 16), __builtin_amdgcn_alignbit(q.z, q.y, 16), acc[1]);
            acc[2] = mfma(a0, a1, q.y, q.z, acc[2]);
        }
        if (t + 1 < t1) store(sh[(t + 1 - t0) & 1]);
        lds_sync();
    }
    const int ci = ib + wn * 32 + i;
    float* dst = a.part + ((size_t)blockIdx.x * 9 + 3 * dy) * a.Cout * a.Cin;
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int co = cb + wm * 32 + 8 * (r >> 2) + 4 * kh + (r & 3);
            if (co < a.Cout && ci < a.Cin) dst[((size_t)t * a.Cout + co) * a.Cin + ci] = acc[t][r];
        }
}

// Weight gradient between a 32-channel tensor g and a single channel s:
//   part[chunk][tap][c] = sum over the chunk's pixels p of g[c][p] s[p + off],
// off the tap's offset; with FLIP s is the gradient and g the layer's input,
// and the sum is over s[p] g[c][p + off]. The same tiles, chunks and order as
// k_conv3x3_wgrad. The taps are the columns of the products (their rows with
// FLIP the channels' shifted pixels), nine of 32. One wave per workgroup
// computes, all four transpose; bound by reading g. Grid: x = chunks.
template <class T, bool FLIP>
__global__ __launch_bounds__(256) void k_conv3x3_wgrad_c1(const uint4* __restrict__ g, const T* __restrict__ s, int B,
                                                         int H, int W, float* __restrict__ part) {
    // GX: columns of g staged per tile row, 8 (or 10 with FLIP, whose channels are read shifted)
    constexpr int GR = FLIP ? 10 : 8, NP = FLIP ? 5 : 4, NU = 4 * GR * NP;   // rows, pixel pairs, units
    constexpr int SR = FLIP ? 8 : 10;                                         // rows and columns of s
    __shared__ __align__(16) uint32_t sg[2][GR * 2 * 32 * 4];
    __shared__ __align__(16) uint16_t ss[2][SR * SR];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tiles_x = (W + 7) / 8, tiles = tiles_x * ((H + 7) / 8), ntiles = B * tiles;
    const int upl = tid & 3, upr = (tid >> 2) % NP, row = (tid >> 2) / NP;
    const bool has = tid < NU;
    uint4 v[2];
    T sv = (T)0;
    auto load = [&](int t) {
        const int b = t / tiles, tr = t - b * tiles;
        const int y0 = (tr / tiles_x) * 8, x0 = (tr - (tr / tiles_x) * tiles_x) * 8;
        const int y = y0 + row - (FLIP ? 1 : 0);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int x = x0 + 2 * upr + j - (FLIP ? 1 : 0);
            v[j] = (has && y >= 0 && y < H && x >= 0 && x < W) ? g[(((size_t)b * 4 + upl) * H + y) * W + x]
                                                              : make_uint4(0u, 0u, 0u, 0u);
        }
        const int sy = y0 + tid / SR - (FLIP ? 0 : 1), sxx = x0 + tid % SR - (FLIP ? 0 : 1);
        sv = (tid < SR * SR && sy >= 0 && sy < H && sxx >= 0 && sxx < W) ? s[((size_t)b * H + sy) * W + sxx] : (T)0;
    };
    auto store = [&](int p) {
        if (has) {
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const uint32_t q = pair_of(v[0], v[1], c);
                const int at = wg_pos(upl * 8 + c) * 4;
                uint32_t* d = sg[p] + row * 256;
                if (!FLIP) {
                    d[(upr >> 1) * 128 + at + (upr & 1)] = q;
                } else {
                    if (upr <= 2) d[at + upr] = q;
                    if (upr >= 2) d[128 + at + upr - 2] = q;
                }
            }
        }
        if (tid < SR * SR) ss[p][tid] = to_bits(sv);
    };
    const int i = lane & 31, kh = lane >> 5;
    const int t0 = blockIdx.x * WG_TILES, t1 = min(t0 + WG_TILES, ntiles);
    const int go = kh * 128 + wg_pos(i) * 4;
    f32x16 acc[FLIP ? 9 : 1] = {};
    load(t0);
    store(0);
    lds_sync();
    for (int t = t0; t < t1; ++t) {
        if (t + 1 < t1) load(t + 1);
        const uint32_t* bg = sg[(t - t0) & 1];
        const uint16_t* bs = ss[(t - t0) & 1];
        if (!FLIP) {
            if (wave == 0) {
                const int so = i < 9 ? (i / 3) * 10 + i % 3 + 4 * kh : 0;
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    const uint2 ga = *reinterpret_cast<const uint2*>(bg + r * 256 + go);
                    const uint32_t d0 = bs[r * 10 + so] | ((uint32_t)bs[r * 10 + so + 1] << 16);
                    const uint32_t d1 = bs[r * 10 + so + 2] | ((uint32_t)bs[r * 10 + so + 3] << 16);
                    acc[0] = mfma(ga.x, ga.y, i < 9 ? d0 : 0u, i < 9 ? d1 : 0u, acc[0]);
                }
            }
        } else if (wave < 3) {
            // rows: the one channel (row 0 of 32); wave = kernel row
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const uint32_t* q2 = reinterpret_cast<const uint32_t*>(bs + r * 8 + 4 * kh);
                const uint32_t a0 = i == 0 ? q2[0] : 0u, a1 = i == 0 ? q2[1] : 0u;
                const uint4 q = *reinterpret_cast<const uint4*>(bg + (r + wave) * 256 + go);
                acc[0] = mfma(a0, a1, q.x, q.y, acc[0]);
                acc[1] = mfma(a0, a1, __builtin_amdgcn_alignbit(q.y, q.x, 16), __builtin_amdgcn_alignbit(q.z, q.y, 16), acc[1]);
                acc[2] = mfma(a0, a1, q.y, q.z, acc[2]);
            }
        }
        if (t + 1 < t1) store((t + 1 - t0) & 1);
        lds_sync();
    }
    float* dst = part + (size_t)blockIdx.x * 288;
    if (!FLIP) {
        if (wave == 0 && i < 9) {
#pragma unroll
            for (int r = 0; r < 16; ++r) dst[i * 32 + 8 * (r >> 2) + 4 * kh + (r & 3)] = acc[0][r];
        }
    } else if (wave < 3 && kh == 0) {
#pragma unroll
        for (int t = 0; t < 3; ++t) dst[(3 * wave + t) * 32 + i] = acc[t][0];
    }
}

// out[(co Cin + ci) 9 + tap] = sum over chunks, in order, of part[chunk][tap][co][ci]
// (taps = 9), or out[e] = sum of part[chunk][e] (taps = 1). n: values per chunk.
// A workgroup takes 32 values: its eight rows of threads load 8 chunks' values
// at a time (eight loads in flight each) into LDS, the first row adds them in
// order.
constexpr int SC_LD = 8;   // loads in flight per thread
__global__ __launch_bounds__(256) void k_sum_chunks(const float* __restrict__ part, int chunks, int n, int taps,
                                                   float* __restrict__ out) {
    __shared__ float sh[8 * SC_LD][33];
    const int l = threadIdx.x & 31, g = threadIdx.x >> 5;
    const int e = blockIdx.x * 32 + l;
    float s = 0.f;
    for (int c0 = 0; c0 < chunks; c0 += 8 * SC_LD) {
        float v[SC_LD];
#pragma unroll
        for (int k = 0; k < SC_LD; ++k) {
            const int c = c0 + k * 8 + g;
            v[k] = (c < chunks && e < n) ? part[(size_t)c * n + e] : 0.f;
        }
#pragma unroll
        for (int k = 0; k < SC_LD; ++k) sh[k * 8 + g][l] = v[k];
        __syncthreads();
        if (g == 0) {
            const int m = min(8 * SC_LD, chunks - c0);
#pragma unroll 16
            for (int k = 0; k < m; ++k) s += sh[k][l];
        }
        __syncthreads();
    }
    if (g == 0 && e < n) {
        const int per = n / taps, t = e / per;
        out[(size_t)(e - t * per) * taps + t] = s;
    }
}

// Bias gradient, split over chunks of the (image, pixel) pairs:
//   part[chunk][co] = sum over the chunk's pairs of g[b, co, p]
// in a fixed order (per thread in index order, then a tree over the threads);
// the chunks are summed in order by k_sum_chunks. Each thread takes 8
// consecutive pairs of the eight channels of a plane per step; the values are
// added two by two when H * W is a multiple of 8 (a step then never crosses an
// image), else one by one. Grid: x = chunks, y = planes.
constexpr int BG_CHUNK = 16384;   // pairs per chunk (a multiple of 256 * 8)
__global__ __launch_bounds__(256) void k_bias_grad(const uint4* __restrict__ g, const uint8_t* __restrict__ mask, int B,
                                                  int C, int P, int HW, float* __restrict__ part) {
    __shared__ float sh[8][256];
    const int pl = blockIdx.y;
    const long long n = (long long)B * HW, q0 = (long long)blockIdx.x * BG_CHUNK;
    float s[8] = {};
    for (int k = threadIdx.x * 8; k < BG_CHUNK; k += 256 * 8) {
        uint4 v[8];
        unsigned m[8] = {};
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const long long q = q0 + k + j;
            v[j] = make_uint4(0u, 0u, 0u, 0u);
            if (q < n) {
                const int b = (int)(q / HW);
                const size_t o = ((size_t)b * P + pl) * HW + (size_t)(q - (long long)b * HW);
                v[j] = g[o];
                if (mask) m[j] = mask[o];
            }
        }
        if (mask) {
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = mask_piece(v[j], m[j]);
        }
        auto ch = [&](int j, int c) {
            const uint32_t d = c < 2 ? v[j].x : c < 4 ? v[j].y : c < 6 ? v[j].z : v[j].w;
            return (c & 1) ? hi2f(d) : lo2f(d);
        };
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            if (HW % 8 == 0) {
#pragma unroll
                for (int j = 0; j < 8; j += 2) s[c] += ch(j, c) + ch(j + 1, c);
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) s[c] += ch(j, c);
            }
        }
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) sh[c][threadIdx.x] = s[c];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        for (int e = threadIdx.x; e < 8 * w; e += 256) sh[e / w][e % w] += sh[e / w][e % w + w];
        __syncthreads();
    }
    if (threadIdx.x < 8 && pl * 8 + threadIdx.x < C) part[(size_t)blockIdx.x * C + pl * 8 + threadIdx.x] = sh[threadIdx.x][0];
}

// The same of a single channel (C = 1, one value per pair).
__global__ __launch_bounds__(256) void k_bias_grad1(const uint16_t* __restrict__ g, long long n, int HW,
                                                   float* __restrict__ part) {
    __shared__ float sh[256];
    const long long q0 = (long long)blockIdx.x * BG_CHUNK;
    float s = 0.f;
    for (int k = threadIdx.x * 8; k < BG_CHUNK; k += 256 * 8) {
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = q0 + k + j < n ? bf2f(g[q0 + k + j]) : 0.f;
        if (HW % 8 == 0) {
#pragma unroll
            for (int j = 0; j < 8; j += 2) s += v[j] + v[j + 1];
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) s += v[j];
        }
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// ---------------------------------------------------------------- weights
// Float32 weights [Cout][Cin][3][3] -> bf16 operand layouts. `tr` gives those
// of the data gradient, the convolution of the output gradient with the
// flipped, transposed kernel (rows = input channels).
//   WL_CHUNK  [16-channel chunk][pair of instructions][half][rows padded to 32]
//             pieces (k_conv3x3): value j of a pair p and half h is value
//             k = 8 (2 p + j / 4) + 4 h + j % 4 of the chunk's K = 9 channel + tap
//   WL_C1     [half][32] pieces (k_conv3x3_c1): taps 4 h + j for j < 4, then tap 8
enum { WL_CHUNK, WL_C1 };

__device__ __forceinline__ float weight_at(const float* __restrict__ w, int Cin, int Cout, bool tr, int row, int red,
                                           int tap) {
    const int co = tr ? red : row, ci = tr ? row : red;
    if (co >= Cout || ci >= Cin || tap >= 9) return 0.f;
    return w[((size_t)co * Cin + ci) * 9 + (tr ? 8 - tap : tap)];
}

__device__ __forceinline__ float packed_weight(const float* __restrict__ w, int Cin, int Cout, int tr, int layout,
                                               int rowsP, int e) {
    const int j = e & 7, p = e >> 3;
    if (layout == WL_CHUNK) {
        const int row = p % rowsP, ph = (p / rowsP) % 18, c = p / rowsP / 18;
        const int k = 8 * (2 * (ph >> 1) + (j >> 2)) + 4 * (ph & 1) + (j & 3);
        return weight_at(w, Cin, Cout, tr, row, 16 * c + k / 9, k % 9);
    }
    const int h = p >> 5;
    return weight_at(w, Cin, Cout, tr, p & 31, 0, j < 4 ? 4 * h + j : j == 4 && h == 0 ? 8 : 9);
}

// n values of the forward layout, then nt of the data gradient's
__global__ void k_pack_weights(const float* __restrict__ w, int Cin, int Cout, int lg, int rg, int n, int lt, int rt,
                               int nt, uint16_t* __restrict__ Wg, uint16_t* __restrict__ Wt) {
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n + nt; e += gridDim.x * blockDim.x) {
        if (e < n) Wg[e] = f2bf(packed_weight(w, Cin, Cout, 0, lg, rg, e));
        else Wt[e - n] = f2bf(packed_weight(w, Cin, Cout, 1, lt, rt, e - n));
    }
}

// ---------------------------------------------------------------- layouts
// NCHW bf16 <-> planes of eight channels (C padded with zeros to P planes)
__global__ void k_to_planes(const uint16_t* __restrict__ x, uint16_t* __restrict__ y, int B, int C, int P, int HW) {
    const size_t n = (size_t)B * P * HW * 8;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x) {
        const int j = (int)(e & 7);
        const size_t q = e >> 3, px = q % HW, bp = q / HW;
        const int c = (int)(bp % P) * 8 + j;
        y[e] = c < C ? x[((bp / P) * C + c) * HW + px] : (uint16_t)0;
    }
}
// out = [relu](s + bias) [+ res] of float32 sums s (planes of eight, P of them;
// P = 0: NCHW) to NCHW, float32 and/or bf16
__global__ void k_from_sums(const float* __restrict__ s, const float* __restrict__ bias, const uint16_t* __restrict__ res,
                            int relu, uint16_t* __restrict__ out16, float* __restrict__ out32, int B, int C, int P,
                            int HW) {
    const size_t n = (size_t)B * C * HW;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x) {
        const size_t px = e % HW, bc = e / HW;
        const int c = (int)(bc % C);
        const size_t b = bc / C;
        float v = P ? s[((b * P + (c >> 3)) * HW + px) * 8 + (c & 7)] : s[e];
        if (bias) v += bias[c];
        if (relu) v = fmaxf(v, 0.f);
        if (res) v += bf2f(res[e]);
        if (out16) out16[e] = f2bf(v);
        if (out32) out32[e] = v;
    }
}

// ---------------------------------------------------------------- loss, optimiser
// Mean squared error of pred (float32) against target: grad (bf16) =
// 2 (pred - target) / n, per-block partial sums of the squared error.
__global__ __launch_bounds__(256) void k_mse(const float* __restrict__ pred, const float* __restrict__ target,
                                            size_t n, uint16_t* __restrict__ grad, float* __restrict__ part) {
    __shared__ float sh[256];
    float s = 0.f;
    const float sc = 2.0f / (float)n;
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (size_t)gridDim.x * 256) {
        const float d = pred[e] - target[e];
        s += d * d;
        grad[e] = f2bf(sc * d);
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// Adam step on float32 parameters (bias-corrected, step count t >= 1).
__global__ void k_adam(float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, size_t n, float lr, float b1, float b2, float eps, float c1, float c2) {
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x) {
        const float ge = g[e];
        const float me = b1 * m[e] + (1.f - b1) * ge;
        const float ve = b2 * v[e] + (1.f - b2) * ge * ge;
        m[e] = me;
        v[e] = ve;
        w[e] -= lr * (me / c1) / (sqrtf(ve / c2) + eps);
    }
}

}  // namespace cnn
