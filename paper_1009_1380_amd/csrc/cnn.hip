// cnn.hip - the learned warm start's network (include/radon.h, radon_cnn_*):
// a 4-level convolutional encoder-decoder, 32-64-128-256 channels, 3x3
// convolutions on BF16 matrix cores with float32 accumulation, trained with
// Adam on pairs that the method itself generates (filtered adjoint -> basis-
// pursuit solution). Hand-written kernels only (cnn_kernels.hpp).
//
//   e0 = relu(conv_a(x))            32 @ H      x: one channel
//   e1 = relu(conv_b(pool(e0)))     64 @ H/2
//   e2 = relu(conv_c(pool(e1)))    128 @ H/4
//   e3 = relu(conv_d(pool(e2)))    256 @ H/8
//   d2 = relu(conv_e(up(e3))) + e2 128 @ H/4
//   d1 = relu(conv_f(up(d2))) + e1  64 @ H/2
//   d0 = relu(conv_g(up(d1))) + e0  32 @ H
//   y  = conv_h(d0) + x              1 @ H     (a correction of the input)
#include <math.h>
#include <stdarg.h>
#include <stdio.h>

#include <algorithm>
#include <new>
#include <random>
#include <utility>
#include <vector>

#include "../../include/radon.h"
#include "cnn_kernels.hpp"
#include "radon_internal.hpp"

namespace {

using cnn::CONV_NT;

radon_status_t errf(radon_status_t st, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
radon_status_t errf(radon_status_t st, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    return rn::api_fail(st, buf);
}

int pad_to(int k, int m) { return (k + m - 1) / m * m; }

// A bf16 operand layout of a layer's weights (cnn_kernels.hpp, WL_*).
struct Packed {
    uint16_t* p = nullptr;
    int layout = cnn::WL_CHUNK, rows = 0;   // rows: output channels padded to 32 (WL_CHUNK)
    size_t count = 0;                       // bf16 values
};

// The layout that the convolution of `cin` into `cout` channels reads.
Packed packed_for(int cin, int cout) {
    Packed q;
    if (cin == 1 && cout == 32) {
        q.layout = cnn::WL_C1;
        q.count = 2 * 32 * 8;
    } else {
        q.rows = pad_to(cout, 32);
        q.count = (size_t)pad_to(cin, 16) / 16 * 18 * q.rows * 8;
    }
    return q;
}

struct Conv {
    int cin = 0, cout = 0;
    float *w = nullptr, *b = nullptr;          // parameters (float32)
    float *gw = nullptr, *gb = nullptr;        // gradients
    Packed fwd, dgr;                           // bf16 operands (forward, data gradient)
    size_t nw() const { return (size_t)cout * cin * 9; }
};

constexpr int NCONV = 8;

}  // namespace

struct radon_cnn_s {
    int device = 0;
    int cus = 1;             // compute units of the device
    int B = 0, H = 0, W = 0;
    int step = 0;
    Conv conv[NCONV];
    // parameters, gradients and Adam moments, each in layer order (weights, biases)
    float *params = nullptr, *grads = nullptr, *mom = nullptr, *var = nullptr;
    void* arena = nullptr;                               // all device memory
    std::vector<std::pair<void**, size_t>> wanted;       // what it will hold: pointer, offset
    size_t bytes = 0;
    // activations (bf16 planes), the ReLU masks of layers 0..6, gradients
    uint16_t *e0 = nullptr, *p0 = nullptr, *e1 = nullptr, *p1 = nullptr, *e2 = nullptr, *p2 = nullptr,
             *e3 = nullptr, *d2 = nullptr, *d1 = nullptr, *d0 = nullptr;
    uint8_t* mask[NCONV - 1] = {};
    uint16_t *gy = nullptr, *gd0 = nullptr, *gd1 = nullptr, *gd2 = nullptr, *ge3 = nullptr, *ge2 = nullptr,
             *ge1 = nullptr, *ge0 = nullptr;
    float *part = nullptr, *bpart = nullptr, *loss_part = nullptr;
    hipError_t err = hipSuccess;

    ~radon_cnn_s() {
        if (arena) (void)hipFree(arena);
    }
    // Ask for `count` values; the pointers are set by allocate(), one device
    // allocation for all of them (a hipMalloc each took most of the set-up).
    template <class T>
    void want(T** out, size_t count) {
        wanted.push_back({reinterpret_cast<void**>(out), bytes});
        bytes += (sizeof(T) * std::max<size_t>(count, 1) + 255) / 256 * 256;
    }
    bool allocate() {
        if (hipMalloc(&arena, bytes) != hipSuccess) {
            (void)hipGetLastError();
            arena = nullptr;
            return false;
        }
        for (auto& w : wanted) *w.first = static_cast<char*>(arena) + w.second;
        return true;
    }
    void chk(hipError_t e) { if (err == hipSuccess && e != hipSuccess) err = e; }
    bool find_device() {
        if (hipGetDevice(&device) == hipSuccess &&
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess && cus > 0)
            return true;
        (void)hipGetLastError();
        return false;
    }
};

namespace {

size_t grid1(size_t n) { return std::min<size_t>((n + 255) / 256, 65535); }
int cdiv(int a, int b) { return (a + b - 1) / b; }

template <int CB, int TY, bool UP, int EPI>
void conv_go(const cnn::ConvIn& a, const cnn::Epilogue& e, int B, hipStream_t st) {
    const dim3 grid((unsigned)(B * cdiv(a.W, cnn::TX) * cdiv(a.H, TY)), (unsigned)(a.CoutP / CB));
    hipLaunchKernelGGL((cnn::k_conv3x3<CB, TY, UP, EPI>), grid, dim3(CONV_NT), 0, st, a, e);
}

// Channel blocks of 64 (32 for layers with 32) and the tile height by the
// workgroups it makes: tall tiles read the weights and the window's border
// fewer times, but two workgroups per CU (512) have to be left. Blocks of 32
// channels take 8 rows, which hold more workgroups per CU (32 -> 1 channel at
// 512 x 512, batch 8: 89 us against 116 with 16 rows), but 16 on an upsampled
// input, whose window is small (64 -> 32: 158 against 164 us).
template <bool UP, int EPI>
void conv_tile(const cnn::ConvIn& a, const cnn::Epilogue& e, int B, hipStream_t st) {
    const int cb = a.CoutP % 64 == 0 ? 64 : 32;
    auto groups = [&](int ty) { return (long long)B * cdiv(a.W, cnn::TX) * cdiv(a.H, ty) * (a.CoutP / cb); };
    if (cb == 64) {
        if (groups(16) >= 512) conv_go<64, 16, UP, EPI>(a, e, B, st);
        else if (groups(8) >= 512) conv_go<64, 8, UP, EPI>(a, e, B, st);
        else conv_go<64, 4, UP, EPI>(a, e, B, st);
    } else if (UP && groups(16) >= 512) {
        conv_go<32, UP ? 16 : 8, UP, EPI>(a, e, B, st);
    } else {
        conv_go<32, 8, UP, EPI>(a, e, B, st);
    }
}

cnn::ConvIn conv_in(const uint16_t* in, const uint8_t* mask, const Packed& w, int cin, int h, int ww) {
    return cnn::ConvIn{reinterpret_cast<const uint4*>(in), mask, reinterpret_cast<const uint4*>(w.p),
                       pad_to(cin, 16) / 8, w.rows, h, ww};
}

// act = relu(conv(in) + bias) with the epilogue EPI_ACT; up: `in` is half the
// size and read as its nearest upsampling
void conv_act(radon_cnn_s& c, const Conv& L, const uint16_t* in, bool up, int h, int w, uint16_t* out, uint8_t* mask,
              uint16_t* pool, const uint16_t* skip, hipStream_t st) {
    const cnn::ConvIn a = conv_in(in, nullptr, L.fwd, L.cin, h, w);
    const cnn::Epilogue e{L.b, 1, out, mask, pool, skip, nullptr, nullptr};
    if (up) conv_tile<true, cnn::EPI_ACT>(a, e, c.B, st);
    else conv_tile<false, cnn::EPI_ACT>(a, e, c.B, st);
}

// data gradient through the layer and the upsampling before it
void dgrad_up(radon_cnn_s& c, const Conv& L, const uint16_t* g, const uint8_t* gmask, int h, int w, uint16_t* out,
              hipStream_t st) {
    const cnn::Epilogue e{nullptr, 0, out, nullptr, nullptr, nullptr, nullptr, nullptr};
    conv_tile<false, cnn::EPI_SUM4>(conv_in(g, gmask, L.dgr, L.cout, h, w), e, c.B, st);
}

// data gradient through the layer, the pooling before it and the ReLU (mask)
// before that, joined by the gradient `skip` of the same activation
void dgrad_pool(radon_cnn_s& c, const Conv& L, const uint16_t* g, const uint8_t* gmask, int h, int w,
                const uint16_t* skip, uint8_t* mask, uint16_t* out, hipStream_t st) {
    const cnn::Epilogue e{nullptr, 0, out, mask, nullptr, skip, nullptr, nullptr};
    conv_tile<false, cnn::EPI_POOLG>(conv_in(g, gmask, L.dgr, L.cout, h, w), e, c.B, st);
}

template <class T, int EPI>
void conv_c1(const T* in, const Packed& w, const cnn::Epilogue& e, int B, int h, int ww, hipStream_t st) {
    hipLaunchKernelGGL((cnn::k_conv3x3_c1<T, EPI>), dim3((unsigned)(B * cdiv(h, 16) * cdiv(ww, 16))), dim3(CONV_NT), 0,
                       st, in, reinterpret_cast<const uint4*>(w.p), h, ww, e);
}

// the one output channel of a layer: out = conv(in) + bias + res (float32)
void conv_one(const uint16_t* in, const Packed& w, int cin, const float* bias, const float* res, float* out, int B, int h,
              int ww, hipStream_t st) {
    const cnn::Epilogue e{bias, 0, nullptr, nullptr, nullptr, nullptr, out, res};
    conv_tile<false, cnn::EPI_ONE>(conv_in(in, nullptr, w, cin, h, ww), e, B, st);
}

// chunks of the weight and bias gradients for B images of h x w
size_t wgrad_chunks(long long B, int h, int w) {
    const long long tiles = B * (long long)cdiv(h, 8) * cdiv(w, 8);
    return (size_t)((tiles + cnn::WG_TILES - 1) / cnn::WG_TILES);
}
size_t bias_chunks(long long B, int h, int w) { return (size_t)((B * h * w + cnn::BG_CHUNK - 1) / cnn::BG_CHUNK); }

constexpr int WGRAD_FLIGHT = 2;   // tiles in flight (1 and 3 are no faster; 3 costs registers)
template <int COB, int CIB, int TW, int WD = WGRAD_FLIGHT>
void wgrad_go(cnn::WgradArgs a, int chunk0, int chunks, bool up, hipStream_t st) {
    if (chunks <= 0) return;
    a.chunk0 = chunk0;
    const dim3 grid((unsigned)chunks, (unsigned)cdiv(a.Cin, CIB), (unsigned)cdiv(a.Cout, COB));
    constexpr int NT = cnn::wgrad_threads(COB, CIB, TW);
    if (up) hipLaunchKernelGGL((cnn::k_conv3x3_wgrad<COB, CIB, TW, true, WD>), grid, dim3(NT), 0, st, a);
    else hipLaunchKernelGGL((cnn::k_conv3x3_wgrad<COB, CIB, TW, false, WD>), grid, dim3(NT), 0, st, a);
}

// Weight and bias gradients of a layer at size h x w; x1: the single-channel
// input of a layer with one (float32 or bf16)
template <class T>
void conv_wgrad(radon_cnn_s& c, Conv& L, const uint16_t* g, const uint8_t* gmask, const uint16_t* in, const T* x1, bool up,
                int h, int w, hipStream_t st) {
    const size_t chunks = wgrad_chunks(c.B, h, w), bchunks = bias_chunks(c.B, h, w);
    const uint4* gp = reinterpret_cast<const uint4*>(g);
    if (L.cin == 1 && L.cout == 32) {
        hipLaunchKernelGGL((cnn::k_conv3x3_wgrad_c1<T, false>), dim3((unsigned)chunks), dim3(256), 0, st, gp, x1, c.B, h, w,
                           c.part);
    } else if (L.cin == 32 && L.cout == 1) {
        hipLaunchKernelGGL((cnn::k_conv3x3_wgrad_c1<uint16_t, true>), dim3((unsigned)chunks), dim3(256), 0, st,
                           reinterpret_cast<const uint4*>(in), g, c.B, h, w, c.part);
    } else {
        const cnn::WgradArgs a{gp, gmask, reinterpret_cast<const uint4*>(in), pad_to(L.cout, 16) / 8, pad_to(L.cin, 16) / 8,
                               c.B, h, w, L.cout, L.cin, c.part};
        // 64 x 64 channels per workgroup read each tile the fewest times; smaller
        // blocks where those would leave CUs without a workgroup. A CU holds one
        // such workgroup, so a last round that fills at most half of the CUs goes
        // to smaller blocks in a launch of its own (264 workgroups, 8 images of 504 x
        // 520: 208 us in one launch, 118 + 57 in two; above half the smaller blocks
        // take as long as the round).
        const int n = (int)chunks, m = (L.cout / 64) * (L.cin / 64), cus = c.cus;
        if (L.cout % 64 == 0 && L.cin % 64 == 0 && n * m >= cus) {
            const int left = n - n * m / cus * cus / m;   // chunks of the last round
            const int tail = left * m <= cus / 2 ? left : 0;
            wgrad_go<64, 64, 3>(a, 0, n - tail, up, st);
            if (tail * m <= cus / 4) wgrad_go<32, 32, 1>(a, n - tail, tail, up, st);
            else wgrad_go<32, 64, 3>(a, n - tail, tail, up, st);
        } else if (L.cin % 64 == 0 && n * cdiv(L.cout, 32) * (L.cin / 64) >= cus) {
            wgrad_go<32, 64, 3>(a, 0, n, up, st);
        } else {
            wgrad_go<32, 32, 1>(a, 0, n, up, st);
        }
    }
    if (L.cin == 32 && L.cout == 1) {
        hipLaunchKernelGGL(cnn::k_bias_grad1, dim3((unsigned)bchunks), dim3(256), 0, st, g, (long long)c.B * h * w, h * w,
                           c.bpart);
    } else {
        hipLaunchKernelGGL(cnn::k_bias_grad, dim3((unsigned)bchunks, (unsigned)cdiv(L.cout, 8)), dim3(256), 0, st, gp, gmask,
                           c.B, L.cout, pad_to(L.cout, 16) / 8, h * w, c.bpart);
    }
    const int nw = (int)L.nw(), wblocks = cdiv(nw, 32);
    hipLaunchKernelGGL(cnn::k_sum_chunks, dim3((unsigned)(wblocks + cdiv(L.cout, 32))), dim3(256), 0, st, c.part,
                       (int)chunks, nw, L.gw, wblocks, c.bpart, (int)bchunks, L.cout, L.gb);
}

void pack(Conv& L, hipStream_t st) {
    hipLaunchKernelGGL(cnn::k_pack_weights, dim3((unsigned)grid1(L.fwd.count + L.dgr.count)), dim3(256), 0, st, L.w, L.cin,
                       L.cout, L.fwd.layout, L.fwd.rows, (int)L.fwd.count, L.dgr.layout, L.dgr.rows, (int)L.dgr.count,
                       L.fwd.p, L.dgr.p);
}

// forward of the whole network; y32 gets the float32 output
void forward(radon_cnn_s& c, const float* x, float* y32, hipStream_t st) {
    const int B = c.B, H = c.H, W = c.W;
    conv_c1<float, cnn::EPI_ACT>(x, c.conv[0].fwd, cnn::Epilogue{c.conv[0].b, 1, c.e0, c.mask[0], c.p0, nullptr, nullptr, nullptr},
                                 B, H, W, st);
    conv_act(c, c.conv[1], c.p0, false, H / 2, W / 2, c.e1, c.mask[1], c.p1, nullptr, st);
    conv_act(c, c.conv[2], c.p1, false, H / 4, W / 4, c.e2, c.mask[2], c.p2, nullptr, st);
    conv_act(c, c.conv[3], c.p2, false, H / 8, W / 8, c.e3, c.mask[3], nullptr, nullptr, st);
    conv_act(c, c.conv[4], c.e3, true, H / 4, W / 4, c.d2, c.mask[4], nullptr, c.e2, st);
    conv_act(c, c.conv[5], c.d2, true, H / 2, W / 2, c.d1, c.mask[5], nullptr, c.e1, st);
    conv_act(c, c.conv[6], c.d1, true, H, W, c.d0, c.mask[6], nullptr, c.e0, st);
    conv_one(c.d0, c.conv[7].fwd, 32, c.conv[7].b, x, y32, B, H, W, st);   // + the float32 input
}

// backward from gy (bf16 gradient of the output; x: the network's input);
// fills every layer's gw, gb. gd0, gd1, gd2, ge3 are the gradients of the
// activations d0, d1, d2, e3 (masked by a layer's ReLU where it reads them),
// ge2, ge1, ge0 those before the ReLUs of e2, e1, e0.
void backward(radon_cnn_s& c, const float* x, hipStream_t st) {
    const int B = c.B, H = c.H, W = c.W;
    const uint16_t* none = nullptr;
    conv_wgrad(c, c.conv[7], c.gy, nullptr, c.d0, none, false, H, W, st);
    conv_c1<uint16_t, cnn::EPI_ACT>(c.gy, c.conv[7].dgr, cnn::Epilogue{nullptr, 0, c.gd0, nullptr, nullptr, nullptr, nullptr, nullptr},
                                    B, H, W, st);
    conv_wgrad(c, c.conv[6], c.gd0, c.mask[6], c.d1, none, true, H, W, st);
    dgrad_up(c, c.conv[6], c.gd0, c.mask[6], H, W, c.gd1, st);
    conv_wgrad(c, c.conv[5], c.gd1, c.mask[5], c.d2, none, true, H / 2, W / 2, st);
    dgrad_up(c, c.conv[5], c.gd1, c.mask[5], H / 2, W / 2, c.gd2, st);
    conv_wgrad(c, c.conv[4], c.gd2, c.mask[4], c.e3, none, true, H / 4, W / 4, st);
    dgrad_up(c, c.conv[4], c.gd2, c.mask[4], H / 4, W / 4, c.ge3, st);
    conv_wgrad(c, c.conv[3], c.ge3, c.mask[3], c.p2, none, false, H / 8, W / 8, st);
    dgrad_pool(c, c.conv[3], c.ge3, c.mask[3], H / 8, W / 8, c.gd2, c.mask[2], c.ge2, st);
    conv_wgrad(c, c.conv[2], c.ge2, nullptr, c.p1, none, false, H / 4, W / 4, st);
    dgrad_pool(c, c.conv[2], c.ge2, nullptr, H / 4, W / 4, c.gd1, c.mask[1], c.ge1, st);
    conv_wgrad(c, c.conv[1], c.ge1, nullptr, c.p0, none, false, H / 2, W / 2, st);
    dgrad_pool(c, c.conv[1], c.ge1, nullptr, H / 2, W / 2, c.gd0, c.mask[0], c.ge0, st);
    conv_wgrad(c, c.conv[0], c.ge0, nullptr, none, x, false, H, W, st);
}

}  // namespace

extern "C" {

radon_status_t radon_cnn_create(radon_cnn_t* out, int batch, int height, int width, uint64_t seed) {
    if (!out) return errf(RADON_ERR_INVALID, "out is NULL");
    *out = nullptr;
    if (batch < 1 || height < 8 || width < 8 || height % 8 || width % 8)
        return errf(RADON_ERR_INVALID, "batch >= 1 and height, width multiples of 8 (got %d, %d, %d)", batch,
                    height, width);
    radon_cnn_s* c = new (std::nothrow) radon_cnn_s();
    if (!c) return errf(RADON_ERR_OOM, "host allocation failed");
    if (!c->find_device()) {
        delete c;
        return errf(RADON_ERR_DEVICE, "no HIP device");
    }
    c->B = batch;
    c->H = height;
    c->W = width;
    const int chans[NCONV][2] = {{1, 32}, {32, 64}, {64, 128}, {128, 256}, {256, 128}, {128, 64}, {64, 32}, {32, 1}};
    size_t part_n = 0, bpart_n = 0;
    const int sizes[NCONV] = {1, 2, 4, 8, 4, 2, 1, 1};   // spatial divisor of each layer
    for (int l = 0; l < NCONV; ++l) {
        Conv& L = c->conv[l];
        L.cin = chans[l][0];
        L.cout = chans[l][1];
        L.fwd = packed_for(L.cin, L.cout);
        L.dgr = packed_for(L.cout, L.cin);
        if (l == 0) L.dgr.count = 0;   // the input needs no gradient
        c->want(&L.fwd.p, L.fwd.count);
        c->want(&L.dgr.p, L.dgr.count);
        part_n = std::max(part_n, wgrad_chunks(batch, height / sizes[l], width / sizes[l]) * L.nw());
        bpart_n = std::max(bpart_n, bias_chunks(batch, height / sizes[l], width / sizes[l]) * L.cout);
    }
    const size_t np = (size_t)radon_cnn_param_count(c);
    for (float** p : {&c->params, &c->grads, &c->mom, &c->var}) c->want(p, np);
    const size_t s0 = (size_t)batch * height * width, s1 = s0 / 4, s2 = s0 / 16, s3 = s0 / 64;
    const size_t acts[NCONV - 1] = {32 * s0, 64 * s1, 128 * s2, 256 * s3, 128 * s2, 64 * s1, 32 * s0};
    for (int l = 0; l < NCONV - 1; ++l) c->want(&c->mask[l], acts[l] / 8);
    for (uint16_t** p : {&c->e0, &c->d0, &c->gd0, &c->ge0}) c->want(p, 32 * s0);
    for (uint16_t** p : {&c->e1, &c->d1, &c->gd1, &c->ge1}) c->want(p, 64 * s1);
    for (uint16_t** p : {&c->e2, &c->d2, &c->gd2, &c->ge2}) c->want(p, 128 * s2);
    for (uint16_t** p : {&c->e3, &c->ge3}) c->want(p, 256 * s3);
    c->want(&c->p0, 32 * s1);
    c->want(&c->p1, 64 * s2);
    c->want(&c->p2, 128 * s3);
    c->want(&c->gy, s0);
    c->want(&c->part, part_n);
    c->want(&c->bpart, bpart_n);
    c->want(&c->loss_part, 1024);
    if (!c->allocate()) {
        delete c;
        return errf(RADON_ERR_OOM, "device allocation failed");
    }
    // He initialisation (the last layer starts at zero: the network begins as the identity)
    std::mt19937_64 rng(seed);
    std::vector<float> init(np, 0.f);
    size_t at = 0;
    for (int l = 0; l < NCONV; ++l) {
        Conv& L = c->conv[l];
        std::normal_distribution<float> nd(0.f, sqrtf(2.0f / (L.cin * 9)));
        if (l < NCONV - 1)
            for (size_t k = 0; k < L.nw(); ++k) init[at + k] = nd(rng);
        L.w = c->params + at;
        L.gw = c->grads + at;
        at += L.nw();
        L.b = c->params + at;
        L.gb = c->grads + at;
        at += L.cout;
    }
    c->chk(hipMemcpy(c->params, init.data(), sizeof(float) * np, hipMemcpyHostToDevice));
    std::fill(init.begin(), init.end(), 0.f);
    for (float* p : {c->mom, c->var}) c->chk(hipMemcpy(p, init.data(), sizeof(float) * np, hipMemcpyHostToDevice));
    for (Conv& L : c->conv) pack(L, 0);
    c->chk(hipDeviceSynchronize());
    if (c->err != hipSuccess) {
        delete c;
        return errf(RADON_ERR_DEVICE, "network set-up failed");
    }
    *out = c;
    return rn::api_ok();
}

void radon_cnn_destroy(radon_cnn_t net) { delete net; }

radon_status_t radon_cnn_forward(radon_cnn_t net, const float* in_dev, float* out_dev, void* stream) {
    if (!net || !in_dev || !out_dev) return errf(RADON_ERR_INVALID, "NULL argument");
    hipStream_t st = (hipStream_t)stream;
    forward(*net, in_dev, out_dev, st);
    if (hipGetLastError() != hipSuccess) return errf(RADON_ERR_DEVICE, "network forward launch failed");
    return rn::api_ok();
}

radon_status_t radon_cnn_train_step(radon_cnn_t net, const float* in_dev, const float* target_dev, float lr,
                                    float* loss_host, float* pred_dev, void* stream) {
    if (!net || !in_dev || !target_dev || !pred_dev) return errf(RADON_ERR_INVALID, "NULL argument");
    if (!(lr >= 0.f)) return errf(RADON_ERR_INVALID, "lr must be >= 0");
    radon_cnn_s& c = *net;
    hipStream_t st = (hipStream_t)stream;
    const size_t n0 = (size_t)c.B * c.H * c.W;
    forward(c, in_dev, pred_dev, st);
    const int nblk = (int)std::min<size_t>((n0 + 255) / 256, 1024);
    hipLaunchKernelGGL(cnn::k_mse, dim3(nblk), dim3(256), 0, st, pred_dev, target_dev, n0, c.gy, c.loss_part);
    backward(c, in_dev, st);
    // Adam
    c.step += 1;
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float c1 = 1.f - powf(b1, (float)c.step), c2 = 1.f - powf(b2, (float)c.step);
    cnn::UpdateArgs u{};
    int at = 0;
    for (int l = 0; l < NCONV; ++l) {
        const Conv& L = c.conv[l];
        u.layer[l] = {at, L.cin, L.cout, L.fwd.p, L.fwd.layout, L.fwd.rows, L.dgr.count ? L.dgr.p : nullptr, L.dgr.layout,
                      L.dgr.rows};
        at += (int)L.nw() + L.cout;
    }
    hipLaunchKernelGGL(cnn::k_update, dim3((unsigned)cdiv(at, 256)), dim3(256), 0, st, u, c.params, c.grads, c.mom, c.var, at,
                       lr, b1, b2, eps, c1, c2);
    if (hipGetLastError() != hipSuccess) return errf(RADON_ERR_DEVICE, "training step launch failed");
    if (loss_host) {
        std::vector<float> part(nblk);
        if (hipMemcpyAsync(part.data(), c.loss_part, sizeof(float) * nblk, hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess) {
            (void)hipGetLastError();
            return errf(RADON_ERR_DEVICE, "loss read-back failed");
        }
        double s = 0.0;
        for (float v : part) s += v;
        *loss_host = (float)(s / (double)n0);
    }
    return rn::api_ok();
}

int64_t radon_cnn_param_count(radon_cnn_t net) {
    if (!net) return -1;
    int64_t n = 0;
    for (const Conv& L : net->conv) n += (int64_t)L.nw() + L.cout;
    return n;
}

// Parameters (or gradients) in layer order: w (Cout x Cin x 3 x 3) then b.
static radon_status_t copy_params(radon_cnn_t net, float* host, int64_t n, bool grads, bool to_device) {
    if (!net || !host) return errf(RADON_ERR_INVALID, "NULL argument");
    if (n != radon_cnn_param_count(net)) return errf(RADON_ERR_INVALID, "need %lld values", (long long)radon_cnn_param_count(net));
    float* dev = grads ? net->grads : net->params;
    const hipError_t e = to_device ? hipMemcpy(dev, host, sizeof(float) * n, hipMemcpyHostToDevice)
                                   : hipMemcpy(host, dev, sizeof(float) * n, hipMemcpyDeviceToHost);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return errf(RADON_ERR_DEVICE, "parameter copy failed");
    }
    if (to_device)
        for (Conv& L : net->conv) pack(L, 0);
    if (hipDeviceSynchronize() != hipSuccess) return errf(RADON_ERR_DEVICE, "parameter copy failed");
    return rn::api_ok();
}

radon_status_t radon_cnn_get_params(radon_cnn_t net, float* host, int64_t n) { return copy_params(net, host, n, false, false); }
radon_status_t radon_cnn_set_params(radon_cnn_t net, const float* host, int64_t n) {
    return copy_params(net, const_cast<float*>(host), n, false, true);
}
radon_status_t radon_cnn_get_grads(radon_cnn_t net, float* host, int64_t n) { return copy_params(net, host, n, true, false); }

// Test hook: one 3x3 convolution with float32 weights w (Cout x Cin x 3 x 3),
// bias (may be null) and bf16 tensors; also its data and weight gradients
// for an output gradient gout (any of the gradient outputs may be null).
radon_status_t radon_cnn_conv_test(const uint16_t* in, const float* w, const float* bias, const uint16_t* res,
                                   uint16_t* out16, float* out32, int relu, const uint16_t* gout, uint16_t* gin,
                                   float* gw, float* gb, int B, int Cin, int Cout, int H, int W, void* stream) {
    if (!in || !w || B < 1 || Cin < 1 || Cout < 1 || H < 1 || W < 1) return errf(RADON_ERR_INVALID, "bad arguments");
    hipStream_t st = (hipStream_t)stream;
    radon_cnn_s c;
    if (!c.find_device()) return errf(RADON_ERR_DEVICE, "no HIP device");
    c.B = B;
    Conv L;
    L.cin = Cin;
    L.cout = Cout;
    L.fwd = packed_for(Cin, Cout);
    L.dgr = packed_for(Cout, Cin);
    L.w = const_cast<float*>(w);
    L.gw = gw;
    L.gb = gb;
    const int HW = H * W, Pi = pad_to(Cin, 16) / 8, Po = pad_to(Cout, 16) / 8;
    const int Cs = std::max(pad_to(Cin, 32), pad_to(Cout, 32));
    uint16_t *xp = nullptr, *gp = nullptr;   // the tensors in planes (one channel: as they are)
    float* sums = nullptr;
    c.want(&L.fwd.p, L.fwd.count);
    c.want(&L.dgr.p, L.dgr.count);
    c.want(&c.part, wgrad_chunks(B, H, W) * L.nw());
    c.want(&c.bpart, bias_chunks(B, H, W) * Cout);
    c.want(&xp, (size_t)B * Pi * HW * 8);
    c.want(&gp, (size_t)B * Po * HW * 8);
    c.want(&sums, (size_t)B * Cs * HW);
    if (!c.allocate())
        return errf(RADON_ERR_OOM, "test buffers");
    auto planes = [&](const uint16_t* src, uint16_t* dst, int C, int P) {
        hipLaunchKernelGGL(cnn::k_to_planes, dim3((unsigned)grid1((size_t)B * P * HW * 8)), dim3(256), 0, st, src, dst, B, C,
                           P, HW);
    };
    // the sums of a convolution of ci into co channels, then [relu](sums + bias) [+ res]
    auto convolve = [&](const uint16_t* nchw, const uint16_t* in, const Packed& pk, int ci, int co, const float* bi,
                        const uint16_t* re, int act, uint16_t* o16, float* o32) {
        const cnn::Epilogue e{nullptr, 0, nullptr, nullptr, nullptr, nullptr, sums, nullptr};
        int P = pk.rows / 8;
        if (pk.layout == cnn::WL_C1) {
            conv_c1<uint16_t, cnn::EPI_F32>(nchw, pk, e, B, H, W, st);
            P = 4;
        } else if (co == 1) {
            conv_one(in, pk, ci, nullptr, nullptr, sums, B, H, W, st);
            P = 0;
        } else {
            conv_tile<false, cnn::EPI_F32>(conv_in(in, nullptr, pk, ci, H, W), e, B, st);
        }
        hipLaunchKernelGGL(cnn::k_from_sums, dim3((unsigned)grid1((size_t)B * co * HW)), dim3(256), 0, st, sums, bi, re, act,
                           o16, o32, B, co, P, HW);
    };
    pack(L, st);
    planes(in, xp, Cin, Pi);
    if (out16 || out32) convolve(in, xp, L.fwd, Cin, Cout, bias, res, relu != 0, out16, out32);
    if (gout) planes(gout, gp, Cout, Po);
    if (gout && gin) convolve(gout, gp, L.dgr, Cout, Cin, nullptr, nullptr, 0, gin, nullptr);
    if (gout && gw && gb) conv_wgrad(c, L, Cout == 1 && Cin == 32 ? gout : gp, nullptr, xp, in, false, H, W, st);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(st) != hipSuccess)
        return errf(RADON_ERR_DEVICE, "convolution test failed");
    return rn::api_ok();
}

}  // extern "C"
