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

// A piece loaded as one vector (assigning the struct itself into an array of them
// makes the compiler keep the array in LDS).
__device__ __forceinline__ uint4 ld_piece(const uint4* p) {
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 v = *reinterpret_cast<const u32x4*>(p);
    return make_uint4(v.x, v.y, v.z, v.w);
}

// A piece with the channels whose bit of m is clear set to zero.
__device__ __forceinline__ uint4 mask_piece(uint4 v, unsigned m) {
    auto bit = [&](int k) { return (unsigned)((int)(m << (31 - k)) >> 31); };   // all ones where bit k is set
    auto two = [&](int k) { return (bit(k) & 0xffffu) | (bit(k + 1) & 0xffff0000u); };
    return make_uint4(v.x & two(0), v.y & two(2), v.z & two(4), v.w & two(6));
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

// What a block's epilogue reads: the second gradient and the mask of EPI_POOLG, the
// skip of EPI_ACT, the residual of EPI_ONE. Requested for all of a wave's blocks
// (EPI_POOLG: for the next one) before the first is worked on, without branches
// per lane (lanes outside the image read the first piece and store nothing), and
// with the biases in LDS: one memory latency instead of one per piece (batch 8,
// 512 x 512: 64 -> 32 channels with its skip 163 -> 155 us, the pooled gradient
// 64 -> 32 channels 89 -> 77).
template <int EPI>
struct EpiIn {
    uint4 s[2][EPI == EPI_POOLG ? 4 : 1];
    unsigned m[2][EPI == EPI_POOLG ? 4 : 1];
    float r;
};
template <int EPI>
__device__ __forceinline__ void epilogue_load(EpiIn<EPI>& in, const Epilogue& e, int b, int P, int plane0, int gy, int gx,
                                              int H, int W, int kh) {
    const bool ok = gy < H && gx < W;
    if constexpr (EPI == EPI_ONE) in.r = e.res32 ? e.res32[ok ? ((size_t)b * H + gy) * W + gx : 0] : 0.f;
    if constexpr (EPI == EPI_ACT) {
        if (e.skip) {
#pragma unroll
            for (int gp = 0; gp < 2; ++gp) {
                const size_t pl = (size_t)b * P + plane0 + 2 * gp + kh;
                in.s[gp][0] = reinterpret_cast<const uint4*>(e.skip)[ok ? (pl * H + gy) * W + gx : 0];
            }
        }
    }
    if constexpr (EPI == EPI_POOLG) {
#pragma unroll
        for (int gp = 0; gp < 2; ++gp) {
            const size_t pl = (size_t)b * P + plane0 + 2 * gp + kh;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const size_t px = ok ? (pl * 2 * H + 2 * gy + (c >> 1)) * (2 * W) + 2 * gx + (c & 1) : 0;
                in.s[gp][c] = reinterpret_cast<const uint4*>(e.skip)[px];
                in.m[gp][c] = e.mask[px];
            }
        }
    }
}

// acc: the block's results; plane0: plane of its first channel (of P); (gy, gx):
// this lane's pixel of an H x W image; i = lane % 32, kh = lane / 32; sb: the
// block's biases in LDS (EPI_ACT, EPI_ONE with a bias).
template <int EPI>
__device__ __forceinline__ void epilogue(const Epilogue& e, const EpiIn<EPI>& in, const float* sb, const f32x16& acc, int b,
                                         int P, int plane0, int gy, int gx, int H, int W, int i, int kh) {
    const bool ok = gy < H && gx < W;
    if constexpr (EPI == EPI_ONE) {
        if (ok && kh == 0) {
            float v = acc[0];
            if (e.bias) v += sb[0];
            if (e.res32) v += in.r;
            e.out32[((size_t)b * H + gy) * W + gx] = v;
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
                    const float4 bv = *reinterpret_cast<const float4*>(sb + g * 8 + 4 * kh);
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
                    const uint4 q = in.s[gp][0];
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
                    const uint4 g = in.s[gp][c];
                    const float s[8] = {lo2f(g.x) + q[0], hi2f(g.x) + q[1], lo2f(g.y) + q[2], hi2f(g.y) + q[3],
                                        lo2f(g.z) + q[4], hi2f(g.z) + q[5], lo2f(g.w) + q[6], hi2f(g.w) + q[7]};
                    reinterpret_cast<uint4*>(e.out)[px] = mask_piece(piece(s), in.m[gp][c]);
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
// us, 0.72 PFLOP/s of the 1.05 that this instruction reaches on random values
// (1.24 on zeros); 350 us for the convolution and 61 us for the upsampling when every operand was four
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
    __shared__ __align__(16) float sb[CB];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tiles_x = (a.W + TX - 1) / TX, tiles = tiles_x * ((a.H + TY - 1) / TY);
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    const int b = blk / tiles, tr = blk - b * tiles;
    const int ty0 = (tr / tiles_x) * TY, tx0 = (tr - (tr / tiles_x) * tiles_x) * TX;
    const int cb = blockIdx.y * CB;
    const int Hi = UP ? a.H / 2 : a.H, Wi = UP ? a.W / 2 : a.W, HWi = Hi * Wi;
    const int wy0 = (UP ? ty0 / 2 : ty0) - 1, wx0 = (UP ? tx0 / 2 : tx0) - 1;

    // this thread's pieces of a chunk: their place in the first chunk, and for the
    // window whether they lie in the image (all ones) or not: those outside read
    // the first piece, without a branch, and are zeroed when they are stored
    int xo[RX], ao[RA];
    unsigned in[RX];
#pragma unroll
    for (int k = 0; k < RX; ++k) {
        const int e = tid + k * CONV_NT;
        const int pl = e / WIN, r = e - pl * WIN, y = wy0 + r / WX, x = wx0 + r % WX;
        const bool ok = e < NX && y >= 0 && y < Hi && x >= 0 && x < Wi;
        xo[k] = ok ? pl * HWi + y * Wi + x : 0;
        in[k] = ok ? ~0u : 0u;
    }
#pragma unroll
    for (int k = 0; k < RA; ++k) {
        const int e = tid + k * CONV_NT;
        ao[k] = e < NA ? (e / CB) * a.CoutP + cb + e % CB : 0;
    }
    if (ep.bias && tid < (EPI == EPI_ACT ? CB : EPI == EPI_ONE ? 1 : 0)) sb[tid] = ep.bias[cb + tid];
    const size_t img = (size_t)b * a.Pin * HWi;
    uint4 vx[RX], va[RA];
    unsigned vm[RX] = {};
    auto load = [&](int c) {
        const uint4* px = a.in + img + (size_t)(2 * c) * HWi;
        const uint4* pa = a.w + (size_t)c * 18 * a.CoutP;
#pragma unroll
        for (int k = 0; k < RX; ++k) vx[k] = ld_piece(px + xo[k]);
#pragma unroll
        for (int k = 0; k < RA; ++k) va[k] = ld_piece(pa + ao[k]);
        if (a.mask) {
            const uint8_t* pm = a.mask + img + (size_t)(2 * c) * HWi;
#pragma unroll
            for (int k = 0; k < RX; ++k) vm[k] = pm[xo[k]];
        }
    };
    auto store = [&](int s) {
#pragma unroll
        for (int k = 0; k < RX; ++k) {
            const int e = tid + k * CONV_NT;
            const uint4 v = make_uint4(vx[k].x & in[k], vx[k].y & in[k], vx[k].z & in[k], vx[k].w & in[k]);
            if (e < NX) sx[s][e] = a.mask ? mask_piece(v, vm[k]) : v;
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
    // the wave's blocks m, n in order
    constexpr int NB = MW * NW;
    EpiIn<EPI> ein[NB];
    auto ask = [&](int k) {
        epilogue_load<EPI>(ein[k], ep, b, a.CoutP / 8, (cb + (wm * MW + k / NW) * 32) / 8, ty0 + py + 2 * (k % NW), tx0 + px,
                           a.H, a.W, kh);
    };
#pragma unroll
    for (int k = 0; k < (EPI == EPI_POOLG ? 1 : NB); ++k) ask(k);
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        if (EPI == EPI_POOLG && k + 1 < NB) ask(k + 1);
        epilogue<EPI>(ep, ein[k], sb + (wm * MW + k / NW) * 32, acc[k / NW][k % NW], b, a.CoutP / 8,
                      (cb + (wm * MW + k / NW) * 32) / 8, ty0 + py + 2 * (k % NW), tx0 + px, a.H, a.W, i, kh);
    }
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
    __shared__ __align__(16) float sb[32];
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
    if (ep.bias && tid < 32) sb[tid] = ep.bias[tid];
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
        EpiIn<EPI> in;
        epilogue_load<EPI>(in, ep, b, 4, 0, ty0 + py, tx0 + px, H, W, kh);
        epilogue<EPI>(ep, in, sb, acc, b, 4, 0, ty0 + py, tx0 + px, H, W, i, kh);
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
// takes 32 x 32 channels and the three taps of one kernel column. A lane's
// operand is four pixels of one channel, while a piece is eight channels of one
// pixel: ds_read_b64_tr_b16 transposes on the way out of LDS (tr_at), so that
// pieces are staged as they are, the loads run along the pixels of a row, and a
// tap is only another address. A wave reads its 8 gradient and 10 input rows
// once per tile for 24 matrix instructions. WD tiles are in flight during the
// products. Blocks of 32 x 32 channels, for layers whose chunks are few, run
// with one tap per wave: with three waves on a CU the products waited for each
// other (1260 cycles per tile where the instructions take 770).
// Measured at batch 8, 512 x 512: 64 -> 32 channels (77 GFLOP) 139 us, 128 -> 64
// and 256 -> 128 113; 1191, 572 and 511 us with 2-byte operand reads and one
// tile in flight, 169, 152 and 144 with the transposition in registers, whose
// loads touched one cache line per lane.
// Grid: x = chunks, y = blocks of CIB input channels, z = of COB output channels.
constexpr int WG_TILES = 64;

// Transposing LDS read: of the 16 lanes of a group, lane j asks for 8 bytes (four
// values) of row j / 4, and receives value j of the concatenated four chunks of
// each of the rows 0..3. Lane j of a 32-channel operand therefore asks for pixel
// j / 4 of the lane half's four, channels 4 (j % 4) .. of the group's sixteen:
// tr_at gives the byte offset in planes `stride` bytes apart.
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
__device__ __forceinline__ int tr_at(int lane, int stride) {
    const int j = lane & 15, kh = lane >> 5, q = (lane >> 4) & 1;
    return (2 * q + ((j & 3) >> 1)) * stride + (4 * kh + (j >> 2)) * 16 + (j & 1) * 8;
}
__device__ __forceinline__ uint2 read_tr(const void* p) {
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p));
}

// Place of an 8 x 8 tile: image and top left pixel; tiles in row order.
struct TileAt {
    int b, y, x;
    __device__ static TileAt of(int t, int H, int W) {
        const int tx = (W + 7) / 8, n = tx * ((H + 7) / 8), r = t % n;
        return TileAt{t / n, r / tx * 8, r % tx * 8};
    }
    __device__ void next(int H, int W) {
        x += 8;
        if (x >= W) { x = 0; y += 8; }
        if (y >= H) { y = 0; ++b; }
    }
};

struct WgradArgs {
    const uint4* g;          // gradient pieces, Pg planes
    const uint8_t* gmask;    // or null
    const uint4* in;         // input pieces, Pi planes, H x W (UP: H/2 x W/2)
    int Pg, Pi, B, H, W, Cout, Cin;
    float* part;
    int chunk0;              // the launch's first chunk
};

// Pieces of a staged plane: 8 x 8 of the gradient, 10 x 10 of the input; the
// distance of planes in LDS is a quarter of the banks past a full turn, so the
// four planes that half a wave reads together do not conflict.
constexpr int WG_GS = 68, WG_XS = 100;

// TW: taps of a wave, the three of a kernel column or one.
constexpr int wgrad_threads(int cob, int cib, int tw) { return cob / 32 * (cib / 32) * (9 / tw) * 64; }

template <int COB, int CIB, int TW, bool UP, int WD>
__global__ __launch_bounds__((wgrad_threads(COB, CIB, TW))) void k_conv3x3_wgrad(WgradArgs a) {
    constexpr int NT = wgrad_threads(COB, CIB, TW);
    constexpr int NG = COB / 8 * 64, NX = CIB / 8 * 100, RU = (NG + NX + NT - 1) / NT;
    constexpr int GP = COB / 8 * WG_GS, XP = CIB / 8 * WG_XS;   // pieces of a buffer
    __shared__ uint4 sh[2][GP + XP];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ntiles = a.B * ((a.W + 7) / 8) * ((a.H + 7) / 8);
    const int cb = blockIdx.z * COB, ib = blockIdx.y * CIB;
    constexpr int us = UP ? 1 : 0;
    const int Hi = a.H >> us, Wi = a.W >> us;

    // this thread's pieces: place in LDS (-1: none), address in the first tile (input:
    // one row and column before it), row and column in the tile
    int at[RU], row[RU], col[RU];
    const uint4* p0[RU];
    bool isg[RU];
    unsigned has = 0u;                       // a bit per piece whose plane is there
#pragma unroll
    for (int k = 0; k < RU; ++k) {
        const int e = tid + k * NT;
        isg[k] = e < NG;
        const int u = isg[k] ? e : e - NG;
        const int pl = isg[k] ? u / 64 : u / 100, r = isg[k] ? u % 64 : u % 100;
        row[k] = isg[k] ? r / 8 : r / 10 - 1;
        col[k] = isg[k] ? r % 8 : r % 10 - 1;
        const int plane = (isg[k] ? cb : ib) / 8 + pl;
        at[k] = e < NG + NX ? (isg[k] ? pl * WG_GS + r : GP + pl * WG_XS + r) : -1;
        const bool ok = e < NG + NX && plane < (isg[k] ? a.Pg : a.Pi);
        has |= ok ? 1u << k : 0u;
        p0[k] = isg[k] ? a.g + ((ptrdiff_t)plane * a.H + row[k]) * a.W + col[k]
                       : a.in + ((ptrdiff_t)plane * Hi + (row[k] >> us)) * Wi + (col[k] >> us);
    }
    // Requests are made without branches around them (a piece that is not there
    // reads the tensor's first and is zeroed when it is stored): under branches the
    // compiler cannot count the requests in flight, and every store would wait for
    // all of them instead of its own tile's (64 x 64 blocks 119 us with branches, 113
    // without; 32 x 32 blocks 69 and 61).
    const int chunk = a.chunk0 + blockIdx.x, t0 = chunk * WG_TILES, t1 = min(t0 + WG_TILES, ntiles);
    TileAt cur = TileAt::of(t0, a.H, a.W);   // the next tile to request
    uint4 vr[WD][RU];
    unsigned mr[WD][RU], live[WD];           // masks, a bit per piece that is there
    const uint8_t* gmask = a.gmask ? a.gmask : reinterpret_cast<const uint8_t*>(a.g);
    const unsigned nomask = a.gmask ? 0u : 255u;
    auto load = [&](int t, uint4 (&v)[RU], unsigned (&mk)[RU], unsigned& there) {
        const bool inner = t < t1 && cur.y > 0 && cur.x > 0 && cur.y + 8 < a.H && cur.x + 8 < a.W;   // uniform
        const ptrdiff_t dg = ((ptrdiff_t)cur.b * a.Pg * a.H + cur.y) * a.W + cur.x;
        const ptrdiff_t dx = ((ptrdiff_t)cur.b * a.Pi * Hi + (cur.y >> us)) * Wi + (cur.x >> us);
        const uint4* p[RU];
        there = has;
        if (!inner) {
#pragma unroll
            for (int k = 0; k < RU; ++k)
                if (!(t < t1 && (unsigned)(cur.y + row[k]) < (unsigned)a.H && (unsigned)(cur.x + col[k]) < (unsigned)a.W))
                    there &= ~(1u << k);
        }
#pragma unroll
        for (int k = 0; k < RU; ++k) p[k] = (there >> k & 1u) ? p0[k] + (isg[k] ? dg : dx) : a.g;
#pragma unroll
        for (int k = 0; k < RU; ++k) {
            v[k] = *p[k];
            if (k * NT < NG) mk[k] = isg[k] ? gmask[p[k] - a.g] : 0u;
        }
        cur.next(a.H, a.W);
    };
    auto store = [&](uint4* buf, const uint4 (&v)[RU], const unsigned (&mk)[RU], unsigned there) {
#pragma unroll
        for (int k = 0; k < RU; ++k) {
            const unsigned ok = (unsigned)((int)(there << (31 - k)) >> 31);   // all ones where it is there
            uint4 q = make_uint4(v[k].x & ok, v[k].y & ok, v[k].z & ok, v[k].w & ok);
            if (k * NT < NG) q = mask_piece(q, mk[k] | (isg[k] ? nomask : 255u));
            if (at[k] >= 0) buf[at[k]] = q;
        }
    };

    const int i = lane & 31, kh = lane >> 5;
    // the wave's kernel column and (first) kernel row, and its 32 x 32 channels
    const int dx = wave % 3, dy = TW == 3 ? 0 : wave / 3 % 3;
    const int wmn = wave / (9 / TW), wm = wmn % (COB / 32), wn = wmn / (COB / 32);
    const int go = wm * 4 * WG_GS * 16 + tr_at(lane, WG_GS * 16);
    const int xo = (GP + wn * 4 * WG_XS + dy * 10 + dx) * 16 + tr_at(lane, WG_XS * 16);
    f32x16 acc[TW] = {};
#pragma unroll
    for (int d = 0; d < WD; ++d) load(t0 + d, vr[d], mr[d], live[d]);
    store(sh[0], vr[0], mr[0], live[0]);
    lds_sync();
    for (int tb = t0; tb < t1; tb += WD) {
#pragma unroll
        for (int d = 0; d < WD; ++d) {   // slot d of the ring held tile t = tb + d, which is in LDS
            const int t = tb + d;
            if (t >= t1) break;   // uniform
            load(t + WD, vr[d], mr[d], live[d]);
            const char* buf = reinterpret_cast<const char*>(sh[(t - t0) & 1]);
            uint2 ga[8], gx[7 + TW];
#pragma unroll
            for (int r = 0; r < 7 + TW; ++r) {
                if (r < 8) ga[r] = read_tr(buf + go + r * 128);
                gx[r] = read_tr(buf + xo + r * 160);
            }
#pragma unroll
            for (int r = 0; r < 8; ++r)
#pragma unroll
                for (int y = 0; y < TW; ++y) acc[y] = mfma(ga[r].x, ga[r].y, gx[r + y].x, gx[r + y].y, acc[y]);
            store(sh[(t + 1 - t0) & 1], vr[(d + 1) % WD], mr[(d + 1) % WD], live[(d + 1) % WD]);
            lds_sync();
        }
    }
    const int ci = ib + wn * 32 + i;
#pragma unroll
    for (int y = 0; y < TW; ++y) {
        float* dst = a.part + ((size_t)chunk * 9 + 3 * (y + dy) + dx) * a.Cout * a.Cin;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int co = cb + wm * 32 + 8 * (r >> 2) + 4 * kh + (r & 3);
            if (co < a.Cout && ci < a.Cin) dst[(size_t)co * a.Cin + ci] = acc[y][r];
        }
    }
}

// Weight gradient between a 32-channel tensor g and a single channel s:
//   part[chunk][tap][c] = sum over the chunk's pixels p of g[c][p] s[p + off],
// off the tap's offset; with FLIP s is the gradient and g the layer's input,
// and the sum is over s[p] g[c][p + off]. The same tiles, chunks and order as
// k_conv3x3_wgrad. The taps are the columns of the products (with FLIP the
// shifted pixels of g are, and s is their one row). Bound by reading g: TB tiles
// are staged at a time, the next TB in flight; one wave (with FLIP three)
// computes. Grid: x = chunks.
template <class T, bool FLIP>
__global__ __launch_bounds__(256) void k_conv3x3_wgrad_c1(const uint4* __restrict__ g, const T* __restrict__ s, int B,
                                                         int H, int W, float* __restrict__ part) {
    constexpr int GR = FLIP ? 10 : 8, GS = FLIP ? WG_XS : WG_GS;   // rows and columns of g, its planes' distance
    constexpr int SR = FLIP ? 8 : 10, NS = SR * SR;                // rows and columns of s
    constexpr int TB = FLIP ? 3 : 4;
    constexpr int NU = 4 * GR * GR, RU = (NU + 255) / 256;   // pieces of a tile, per thread
    __shared__ uint4 sg[2][TB * 4 * GS];
    __shared__ __align__(16) uint16_t ss[2][TB * NS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ntiles = B * ((W + 7) / 8) * ((H + 7) / 8);
    const int t0 = blockIdx.x * WG_TILES, t1 = min(t0 + WG_TILES, ntiles);
    // this thread's pieces of a tile and its value of s: place, row and column
    constexpr int gd = FLIP ? 1 : 0, sd = FLIP ? 0 : 1;      // border of g, of s
    int at[RU], row[RU], col[RU];
    unsigned off[RU];
#pragma unroll
    for (int k = 0; k < RU; ++k) {
        const int e = tid + 256 * k, pl = e / (GR * GR), r = e - pl * GR * GR;
        row[k] = r / GR - gd;
        col[k] = r % GR - gd;
        at[k] = e < NU ? pl * GS + r : -1;
        off[k] = e < NU ? (unsigned)((pl * H + row[k] + gd) * W + col[k] + gd) : 0u;
    }
    const int srow = tid / SR - sd, scol = tid % SR - sd;
    const unsigned soff = (unsigned)((srow + sd) * W + scol + sd);
    uint4 v[TB][RU];
    T sv[TB];
    TileAt cur = TileAt::of(t0, H, W);   // the next tile to load
    auto load = [&](int t) {
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            const uint4* gp = g + (((ptrdiff_t)cur.b * 4 * H + cur.y - gd) * W + cur.x - gd);
            const T* sp = s + (((ptrdiff_t)cur.b * H + cur.y - sd) * W + cur.x - sd);
            const bool live = t + b < t1;                                                                  // uniform
            const bool inner = live && cur.y > 0 && cur.x > 0 && cur.y + 8 < H && cur.x + 8 < W;           // uniform
            auto in = [&](int r, int c) {
                const int y = cur.y + r, x = cur.x + c;
                return inner || (live && y >= 0 && y < H && x >= 0 && x < W);
            };
#pragma unroll
            for (int k = 0; k < RU; ++k)
                v[b][k] = at[k] >= 0 && in(row[k], col[k]) ? gp[off[k]] : make_uint4(0u, 0u, 0u, 0u);
            sv[b] = tid < NS && in(srow, scol) ? sp[soff] : (T)0;
            cur.next(H, W);
        }
    };
    auto store = [&](int p) {
#pragma unroll
        for (int b = 0; b < TB; ++b) {
#pragma unroll
            for (int k = 0; k < RU; ++k)
                if (at[k] >= 0) sg[p][b * 4 * GS + at[k]] = v[b][k];
            if (tid < NS) ss[p][b * NS + tid] = to_bits(sv[b]);
        }
    };
    const int i = lane & 31, kh = lane >> 5;
    const int go = tr_at(lane, GS * 16) + (FLIP ? wave * 16 : 0);   // with FLIP wave = kernel column
    const int so = i < 9 ? (i / 3) * 10 + i % 3 + 4 * kh : 0;
    f32x16 acc[FLIP ? 3 : 1] = {};
    load(t0);
    store(0);
    lds_sync();
    for (int t = t0, p = 0; t < t1; t += TB, p ^= 1) {
        if (t + TB < t1) load(t + TB);
        if (wave < (FLIP ? 3 : 1)) {
            for (int b = 0; b < TB && t + b < t1; ++b) {
                const char* bg = reinterpret_cast<const char*>(&sg[p][b * 4 * GS]) + go;
                const uint16_t* bs = ss[p] + b * NS;
                if constexpr (!FLIP) {
#pragma unroll
                    for (int r = 0; r < 8; ++r) {
                        const uint2 ga = read_tr(bg + r * 128);
                        const uint32_t d0 = bs[r * 10 + so] | ((uint32_t)bs[r * 10 + so + 1] << 16);
                        const uint32_t d1 = bs[r * 10 + so + 2] | ((uint32_t)bs[r * 10 + so + 3] << 16);
                        acc[0] = mfma(ga.x, ga.y, i < 9 ? d0 : 0u, i < 9 ? d1 : 0u, acc[0]);
                    }
                } else {
                    uint2 gx[10];
#pragma unroll
                    for (int r = 0; r < 10; ++r) gx[r] = read_tr(bg + r * 160);
#pragma unroll
                    for (int r = 0; r < 8; ++r) {
                        const uint2 q = *reinterpret_cast<const uint2*>(bs + r * 8 + 4 * kh);
                        const uint32_t a0 = i == 0 ? q.x : 0u, a1 = i == 0 ? q.y : 0u;   // row 0 of 32
#pragma unroll
                        for (int y = 0; y < 3; ++y) acc[y] = mfma(a0, a1, gx[r + y].x, gx[r + y].y, acc[y]);
                    }
                }
            }
        }
        if (t + TB < t1) store(p ^ 1);
        lds_sync();
    }
    float* dst = part + (size_t)blockIdx.x * 288;
    if constexpr (!FLIP) {
        if (wave == 0 && i < 9) {
#pragma unroll
            for (int r = 0; r < 16; ++r) dst[i * 32 + 8 * (r >> 2) + 4 * kh + (r & 3)] = acc[0][r];
        }
    } else if (wave < 3 && kh == 0) {
#pragma unroll
        for (int y = 0; y < 3; ++y) dst[(3 * y + wave) * 32 + i] = acc[y][0];
    }
}

// Sums over chunks, in order: workgroups below `wblocks` take the weights,
//   out[(co Cin + ci) 9 + tap] = sum of part[chunk][tap][co][ci], n = 9 Cout Cin,
// the others the biases, bout[e] = sum of bpart[chunk][e], nb of them. A
// workgroup takes 32 values: its eight rows of threads load eight chunks each
// at a time into LDS (one thread alone waits out a latency per few chunks), the
// first row adds them in order.
constexpr int SC_LD = 8;   // loads in flight per thread
__global__ __launch_bounds__(256) void k_sum_chunks(const float* __restrict__ part, int chunks, int n,
                                                   float* __restrict__ out, int wblocks, const float* __restrict__ bpart,
                                                   int bchunks, int nb, float* __restrict__ bout) {
    __shared__ float sh[8 * SC_LD][33];
    const bool bias = (int)blockIdx.x >= wblocks;
    const float* src = bias ? bpart : part;
    const int nc = bias ? bchunks : chunks, nv = bias ? nb : n;
    const int l = threadIdx.x & 31, g = threadIdx.x >> 5;
    const int e = ((int)blockIdx.x - (bias ? wblocks : 0)) * 32 + l;
    float s = 0.f;
    for (int c0 = 0; c0 < nc; c0 += 8 * SC_LD) {
        float v[SC_LD];
#pragma unroll
        for (int k = 0; k < SC_LD; ++k) {
            const int c = c0 + k * 8 + g;
            v[k] = (c < nc && e < nv) ? src[(size_t)c * nv + e] : 0.f;
        }
#pragma unroll
        for (int k = 0; k < SC_LD; ++k) sh[k * 8 + g][l] = v[k];
        __syncthreads();
        if (g == 0) {
            const int m = min(8 * SC_LD, nc - c0);
#pragma unroll 16
            for (int k = 0; k < m; ++k) s += sh[k][l];
        }
        __syncthreads();
    }
    if (g == 0 && e < nv) {
        const int per = n / 9, t = e / per;
        if (bias) bout[e] = s;
        else out[(e - t * per) * 9 + t] = s;
    }
}

// Bias gradient, split over chunks of the (image, pixel) pairs:
//   part[chunk][co] = sum over the chunk's pairs of g[b, co, p]
// in a fixed order (per thread in index order, then a tree over the threads);
// the chunks are summed in order by k_sum_chunks. Each thread takes 8
// consecutive pairs of the eight channels of a plane per step; the values are
// added two by two when H * W is a multiple of 8 (a step then never crosses an
// image), else one by one. Grid: x = chunks, y = planes.
constexpr int BG_CHUNK = 16384;   // pairs per chunk (a multiple of 256 * 16)
__global__ __launch_bounds__(256) void k_bias_grad(const uint4* __restrict__ g, const uint8_t* __restrict__ mask, int B,
                                                  int C, int P, int HW, float* __restrict__ part) {
    __shared__ float sh[8][256];
    const int pl = blockIdx.y;
    const long long n = (long long)B * HW, q0 = (long long)blockIdx.x * BG_CHUNK;
    const int b0 = (int)(q0 / HW);                       // the chunk starts at pixel p0 of image b0
    const int p0 = (int)(q0 - (long long)b0 * HW);
    const int left = (int)min((long long)BG_CHUNK, n - q0);
    auto place = [&](int k) {                            // piece of pair q0 + k
        const unsigned p = (unsigned)(p0 + k), b = p / (unsigned)HW;
        return ((size_t)(b0 + b) * P + pl) * HW + (p - b * HW);
    };
    auto ch = [](const uint4& v, int c) {
        const uint32_t d = c < 2 ? v.x : c < 4 ? v.y : c < 6 ? v.z : v.w;
        return (c & 1) ? hi2f(d) : lo2f(d);
    };
    float s[8] = {};
    if (HW % 8 == 0) {   // n and left are multiples of 8 too
#pragma unroll 2
        for (int k = threadIdx.x * 8; k < left; k += 256 * 8) {
            const size_t o = place(k);
            uint4 v[8];
            uint2 m = make_uint2(0u, 0u);
            if (mask) m = *reinterpret_cast<const uint2*>(mask + o);
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = g[o + j];
            if (mask) {
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = mask_piece(v[j], (j < 4 ? m.x : m.y) >> (8 * (j & 3)));
            }
#pragma unroll
            for (int c = 0; c < 8; ++c)
#pragma unroll
                for (int j = 0; j < 8; j += 2) s[c] += ch(v[j], c) + ch(v[j + 1], c);
        }
    } else {
        for (int k = threadIdx.x * 8; k < left; k += 256 * 8)
            for (int j = 0; j < 8 && k + j < left; ++j) {
                const size_t o = place(k + j);
                const uint4 v = mask ? mask_piece(g[o], mask[o]) : g[o];
#pragma unroll
                for (int c = 0; c < 8; ++c) s[c] += ch(v, c);
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

// Place of value (row, reduction index, tap) in an operand layout.
__device__ __forceinline__ size_t packed_at(int layout, int rowsP, int row, int red, int tap) {
    if (layout == WL_CHUNK) {
        const int k = (red & 15) * 9 + tap, S = k >> 3, h = (k >> 2) & 1;
        return ((((size_t)(red >> 4) * 18 + (S >> 1) * 2 + h) * rowsP + row) << 3) + (S & 1) * 4 + (k & 3);
    }
    return tap < 8 ? (((tap >> 2) * 32 + row) << 3) + (tap & 3) : (row << 3) + 4;
}

// Adam step on all float32 parameters (bias-corrected, step count >= 1), and the
// new weights' bf16 operands (the padding of the layouts stays zero). One launch
// for the network: 24 launches, one per tensor and packing, took 110 us.
struct UpdateArgs {
    struct Layer {
        int first, cin, cout;            // its first parameter; weights, then biases
        uint16_t* fwd;                   // operands of the forward ...
        int lf, rf;                      // ... their layout and rows
        uint16_t* dgr;                   // operands of the data gradient (null: none)
        int ld, rd;
    } layer[8];
};
__global__ __launch_bounds__(256) void k_update(UpdateArgs a, float* __restrict__ w, const float* __restrict__ g,
                                               float* __restrict__ m, float* __restrict__ v, int n, float lr, float b1,
                                               float b2, float eps, float c1, float c2) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= n) return;
    const float ge = g[e];
    const float me = b1 * m[e] + (1.f - b1) * ge;
    const float ve = b2 * v[e] + (1.f - b2) * ge * ge;
    m[e] = me;
    v[e] = ve;
    const float we = w[e] - lr * (me / c1) / (sqrtf(ve / c2) + eps);
    w[e] = we;
    UpdateArgs::Layer L = a.layer[0];
#pragma unroll
    for (int l = 1; l < 8; ++l)
        if (e >= a.layer[l].first) L = a.layer[l];
    const int k = e - L.first;
    if (k >= L.cout * L.cin * 9) return;   // a bias
    const int tap = k % 9, cc = k / 9, ci = cc % L.cin, co = cc / L.cin;
    const uint16_t h = f2bf(we);
    L.fwd[packed_at(L.lf, L.rf, co, ci, tap)] = h;
    if (L.dgr) L.dgr[packed_at(L.ld, L.rd, ci, co, 8 - tap)] = h;
}

}  // namespace cnn
