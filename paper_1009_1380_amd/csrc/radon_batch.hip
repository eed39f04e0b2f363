// radon_batch.hip - uneven-slice batches recorded into HIP graphs, and the
// autotuner of a plan's work decomposition (include/radon.h).
//
// Parallel-beam tomography reconstructs every slice of a volume on its own
// (introduction: slices of the imaged samples), and slices differ in size and
// view count. A batch runs each pass of the path once for all its slices
// (radon_multi.hpp): one launch per pass and FFT length for the transforms,
// one launch per kernel width and tile size for the gridding, whose work
// items from every slice form one list drained longest first (the paper's
// balancing of bins over thread blocks, section "fast radon transform",
// paragraph 4, across slices). The launches of one direction are recorded
// once into a HIP graph (launches for different lengths on parallel
// branches) and replayed with one graph launch.
//
// The autotuner revisits the paper's load-balancing choice of bins (the work
// of a bin grows with its samples times its grid points) by measurement: it
// times each candidate decomposition of the same geometry on the device and
// keeps the fastest.
#include <stdarg.h>
#include <stdio.h>

#include <algorithm>
#include <new>
#include <vector>

#include "../../include/radon.h"
#include "radon_internal.hpp"

namespace {

struct Recording {
    std::vector<const void*> in, out;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    rn::PassSlice* tab = nullptr;   // the transform passes' slice tables (device)
    std::vector<void*> owned;
    void release() {
        if (exec) (void)hipGraphExecDestroy(exec);
        if (graph) (void)hipGraphDestroy(graph);
        for (void* p : owned) (void)hipFree(p);
        owned.clear();
        tab = nullptr;
        exec = nullptr;
        graph = nullptr;
        in.clear();
        out.clear();
    }
};

radon_status_t errf(radon_status_t st, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
radon_status_t errf(radon_status_t st, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    return rn::api_fail(st, buf);
}

// Uniform values in [-1, 1) from an integer hash of the index (inputs of the
// autotuner's timing runs; their values do not affect the timing).
__global__ void k_fill_hash(float* __restrict__ x, size_t n, unsigned seed) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        unsigned h = (unsigned)i * 0x9E3779B1u ^ seed;
        h ^= h >> 16;
        h *= 0x85EBCA6Bu;
        h ^= h >> 13;
        h *= 0xC2B2AE35u;
        h ^= h >> 16;
        x[i] = (float)(h >> 8) * (2.0f / 16777216.0f) - 1.0f;
    }
}

}  // namespace

namespace {

using rn::GridSlice;
using rn::PassKind;
using rn::PassSlice;

// Slices that share a kernel width and tile size: their gridding work items,
// concatenated (each naming its slice) and ordered longest first.
struct GridGroup {
    rn::GridLaunch launch{};
};

template <class T>
bool upload_vec(std::vector<void*>& owned, T** dst, const std::vector<T>& v) {
    *dst = nullptr;
    if (v.empty()) return true;
    void* ptr = nullptr;
    if (hipMalloc(&ptr, sizeof(T) * v.size()) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    owned.push_back(ptr);
    if (hipMemcpy(ptr, v.data(), sizeof(T) * v.size(), hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    *dst = static_cast<T*>(ptr);
    return true;
}

}  // namespace

struct radon_batch_s {
    int device = 0;
    std::vector<radon_plan_t> plans;
    std::vector<hipStream_t> streams;
    std::vector<hipEvent_t> events;   // 4 per branch: two forks and two joins per direction
    Recording fwd, adj;
    int recorded = 0;
    // launch structure, fixed at creation
    std::vector<int> lengths_n, lengths_nd;            // distinct image sizes / detector counts
    std::vector<GridGroup> groups;                     // distinct (W, T)
    GridSlice* gs = nullptr;                           // per slice gridding buffers (device)
    std::vector<void*> owned;                          // device buffers of the lists above

    ~radon_batch_s() {
        fwd.release();
        adj.release();
        for (void* p : owned) (void)hipFree(p);
        for (hipEvent_t e : events) (void)hipEventDestroy(e);
        for (hipStream_t s : streams) (void)hipStreamDestroy(s);
    }

    // Group the slices and upload the gridding lists (once per batch).
    radon_status_t build() {
        const int P = (int)plans.size();
        std::vector<GridSlice> gsh(P);
        for (int i = 0; i < P; ++i) {
            const rn::Plan& p = plans[i]->p;
            gsh[i] = rn::grid_slice_of(p);
            if (std::find(lengths_n.begin(), lengths_n.end(), p.n) == lengths_n.end()) lengths_n.push_back(p.n);
            if (std::find(lengths_nd.begin(), lengths_nd.end(), p.n_det) == lengths_nd.end())
                lengths_nd.push_back(p.n_det);
        }
        std::sort(lengths_n.begin(), lengths_n.end());
        std::sort(lengths_nd.begin(), lengths_nd.end());
        if (!upload_vec(owned, &gs, gsh)) return errf(RADON_ERR_OOM, "batch table upload failed");
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus < 1) {
            (void)hipGetLastError();
            cus = 1;
        }
        std::vector<std::pair<int, int>> wts;
        for (int i = 0; i < P; ++i) {
            const std::pair<int, int> wt{plans[i]->p.W, plans[i]->p.T};
            if (std::find(wts.begin(), wts.end(), wt) == wts.end()) wts.push_back(wt);
        }
        for (const auto& wt : wts) {
            rn::GridLaunch g{};
            g.W = wt.first;
            g.T = wt.second;
            std::vector<rn::F3Item> fi;
            std::vector<rn::TileItem> ti;
            for (int i = 0; i < P; ++i) {
                const rn::Plan& p = plans[i]->p;
                if (p.W != g.W || p.T != g.T) continue;
                if (!g.kbc) g.kbc = p.kbc;   // the same table for every slice of one W
                for (rn::F3Item it : p.fitems_h) { it.plan = i; fi.push_back(it); }
                for (rn::TileItem it : p.items_h) { it.plan = i; ti.push_back(it); }
            }
            // longest first, so the tail of each launch is short
            std::stable_sort(fi.begin(), fi.end(), [](const rn::F3Item& a, const rn::F3Item& b) { return a.count > b.count; });
            std::stable_sort(ti.begin(), ti.end(), [](const rn::TileItem& a, const rn::TileItem& b) { return a.count > b.count; });
            g.n_fitems = (int)fi.size();
            g.n_items = (int)ti.size();
            g.f3_grid = std::max(1, std::min(g.n_fitems, rn::f3_blocks_per_cu(g.W, g.T) * cus));
            rn::F3Item* dfi = nullptr;
            rn::TileItem* dti = nullptr;
            if (!upload_vec(owned, &dfi, fi) || !upload_vec(owned, &dti, ti))
                return errf(RADON_ERR_OOM, "batch work-list upload failed");
            g.fitems = dfi;
            g.items = dti;
            groups.push_back(GridGroup{g});
        }
        return RADON_OK;
    }

    // The transform-pass tables of one direction for these I/O pointers: for
    // each launch, its slices' entries; returns the launches' (kind, length,
    // first entry, entries, blocks) in order.
    struct PassLaunch {
        PassKind kind;
        int len, first, count, blocks;
    };
    void pass_tables(bool forward, const float* const* in, float* const* out, std::vector<PassSlice>& tab,
                     std::vector<PassLaunch>& launches) const {
        const int P = (int)plans.size();
        auto add = [&](PassKind kind, int len) {
            PassLaunch L{kind, len, (int)tab.size(), 0, 0};
            const bool by_n = kind == rn::PK_F1 || kind == rn::PK_F2 || kind == rn::PK_A3 || kind == rn::PK_A4;
            for (int i = 0; i < P; ++i) {
                const rn::Plan& p = plans[i]->p;
                if ((by_n ? p.n : p.n_det) != len) continue;
                PassSlice e = rn::pass_slice_of(p, kind, in[i], out[i]);
                e.block0 = L.blocks;
                L.blocks += e.nblk;
                tab.push_back(e);
            }
            L.count = (int)tab.size() - L.first;
            launches.push_back(L);
        };
        if (forward) {
            for (int L : lengths_n) add(rn::PK_F1, L);
            for (int L : lengths_n) add(rn::PK_F2, L);
            for (int L : lengths_nd) add(rn::PK_F4, L);
        } else {
            for (int L : lengths_nd) add(rn::PK_A1, L);
            for (int L : lengths_n) add(rn::PK_A3, L);
            for (int L : lengths_n) add(rn::PK_A4, L);
        }
    }

    // Record one direction for these I/O pointers into rec's graph:
    //   forward: F1 -> F2 per image size (one branch each), F3 per (W, T), F4 per detector count
    //   adjoint: A1 per detector count, A2 per (W, T), A3 (with the split sums) -> A4 per image size
    radon_status_t record(bool forward, const float* const* in, float* const* out, Recording& rec) {
        rec.release();
        std::vector<PassSlice> tab;
        std::vector<PassLaunch> launches;
        pass_tables(forward, in, out, tab, launches);
        if (!upload_vec(rec.owned, &rec.tab, tab)) return errf(RADON_ERR_OOM, "batch table upload failed");
        const int nb = (int)streams.size();
        hipStream_t s0 = streams[0];
        if (hipStreamBeginCapture(s0, hipStreamCaptureModeThreadLocal) != hipSuccess) {
            (void)hipGetLastError();
            return errf(RADON_ERR_DEVICE, "graph capture could not start");
        }
        hipError_t e = hipSuccess;
        int ev = 0;
        auto fork = [&]() {
            const hipEvent_t f = events[ev++];
            if (e == hipSuccess) e = hipEventRecord(f, s0);
            for (int b = 1; b < nb && e == hipSuccess; ++b) e = hipStreamWaitEvent(streams[b], f, 0);
        };
        auto join = [&]() {
            for (int b = 1; b < nb; ++b) {
                const hipEvent_t j = events[ev++];
                if (e == hipSuccess) e = hipEventRecord(j, streams[b]);
                if (e == hipSuccess) e = hipStreamWaitEvent(s0, j, 0);
            }
        };
        auto run = [&](const PassLaunch& L, hipStream_t s) {
            if (e == hipSuccess && L.count > 0) e = rn::launch_pass(L.kind, L.len, rec.tab + L.first, L.count, L.blocks, s);
        };
        const size_t nl_n = lengths_n.size(), nl_nd = lengths_nd.size();
        if (forward) {
            // launches: F1 x nl_n, F2 x nl_n, F4 x nl_nd
            fork();
            for (size_t g = 0; g < nl_n; ++g) {
                hipStream_t s = streams[g % nb];
                run(launches[g], s);
                run(launches[nl_n + g], s);
            }
            join();
            for (const GridGroup& g : groups)
                if (e == hipSuccess) e = rn::launch_f3_grid(g.launch, gs, s0);
            fork();
            for (size_t g = 0; g < nl_nd; ++g) run(launches[2 * nl_n + g], streams[g % nb]);
            join();
        } else {
            // launches: A1 x nl_nd, A3 x nl_n, A4 x nl_n
            fork();
            for (size_t g = 0; g < nl_nd; ++g) run(launches[g], streams[g % nb]);
            join();
            for (const GridGroup& g : groups)
                if (e == hipSuccess) e = rn::launch_a2_grid(g.launch, gs, s0);
            fork();
            for (size_t g = 0; g < nl_n; ++g) {
                hipStream_t s = streams[g % nb];
                run(launches[nl_nd + g], s);
                run(launches[nl_nd + nl_n + g], s);
            }
            join();
        }
        hipGraph_t gr = nullptr;
        const hipError_t ec = hipStreamEndCapture(s0, &gr);
        if (e != hipSuccess || ec != hipSuccess || !gr) {
            (void)hipGetLastError();
            if (gr) (void)hipGraphDestroy(gr);
            return errf(RADON_ERR_DEVICE, "graph capture failed");
        }
        hipGraphExec_t x = nullptr;
        if (hipGraphInstantiate(&x, gr, nullptr, nullptr, 0) != hipSuccess) {
            (void)hipGetLastError();
            (void)hipGraphDestroy(gr);
            return errf(RADON_ERR_DEVICE, "graph instantiation failed");
        }
        rec.graph = gr;
        rec.exec = x;
        rec.in.assign(in, in + plans.size());
        rec.out.assign(out, out + plans.size());
        ++recorded;
        return RADON_OK;
    }

    radon_status_t run(bool forward, const float* const* in, float* const* out, void* stream) {
        int dev = -1;
        if (hipGetDevice(&dev) != hipSuccess || dev != device) {
            (void)hipGetLastError();
            return errf(RADON_ERR_INVALID, "the batch's device %d is not current", device);
        }
        if (!in || !out) return errf(RADON_ERR_INVALID, "NULL pointer array");
        for (size_t i = 0; i < plans.size(); ++i) {
            if (!in[i] || !out[i]) return errf(RADON_ERR_INVALID, "NULL buffer for slice %zu", i);
            if (plans[i]->p.profiling) return errf(RADON_ERR_INVALID, "profiling is on for slice %zu", i);
        }
        Recording& rec = forward ? fwd : adj;
        bool same = rec.exec != nullptr;
        for (size_t i = 0; same && i < plans.size(); ++i) same = rec.in[i] == in[i] && rec.out[i] == out[i];
        if (!same) {
            const radon_status_t st = record(forward, in, out, rec);
            if (st != RADON_OK) return st;
        }
        if (hipGraphLaunch(rec.exec, (hipStream_t)stream) != hipSuccess) {
            (void)hipGetLastError();
            return errf(RADON_ERR_DEVICE, "graph launch failed");
        }
        return rn::api_ok();
    }
};

extern "C" {

radon_status_t radon_batch_create(radon_batch_t* out, int count, const radon_plan_t* plans, int n_branches) {
    if (!out) return errf(RADON_ERR_INVALID, "out is NULL");
    *out = nullptr;
    if (count < 1 || !plans) return errf(RADON_ERR_INVALID, "count=%d must be >= 1 with a plan array", count);
    if (n_branches < 1 || n_branches > 16) return errf(RADON_ERR_INVALID, "n_branches=%d must be 1..16", n_branches);
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return errf(RADON_ERR_DEVICE, "no HIP device");
    }
    std::vector<radon_plan_t> ps(plans, plans + count);
    for (int i = 0; i < count; ++i) {
        if (!ps[i]) return errf(RADON_ERR_INVALID, "plan %d is NULL", i);
        if (ps[i]->p.device != dev) return errf(RADON_ERR_INVALID, "plan %d lives on another device", i);
    }
    std::vector<radon_plan_t> sorted = ps;
    std::sort(sorted.begin(), sorted.end());
    if (std::adjacent_find(sorted.begin(), sorted.end()) != sorted.end())
        return errf(RADON_ERR_INVALID, "a plan appears twice (each slice needs its own workspace)");
    radon_batch_s* b = new (std::nothrow) radon_batch_s();
    if (!b) return errf(RADON_ERR_OOM, "host allocation failed");
    b->device = dev;
    b->plans = ps;
    // Branches share the device's queues: a fork and a join cost some 10 us each, and
    // more of them with more branches, while what they hide is the tail of one
    // length's launches behind another's. So one branch for batches of few pixels
    // and lengths, two up to eight million pixels. Forward and adjoint with 1, 2 and
    // 4 branches: 1.6 million pixels of 2 sides 129, 162, 162 us; 2.4 of 3 199, 201,
    // 235; 2.6 of 6 285, 272, 305; 5.1 of 4 279, 273, 295; 7.7 of 6 414, 373, 370;
    // ten slices of 8 sides up to 2560 654, 579, 554; 42 million of 8 1445, 1334, 1320.
    double pixels = 0;
    std::vector<int> sides;
    for (const radon_plan_t p : ps) {
        pixels += (double)p->p.n * p->p.n;
        if (std::find(sides.begin(), sides.end(), p->p.n) == sides.end()) sides.push_back(p->p.n);
    }
    const int most = pixels >= 8e6 ? 16 : pixels < 4.5e6 && sides.size() <= 5 ? 1 : 2;
    const int nb = std::min({n_branches, count, most});
    for (int i = 0; i < nb; ++i) {
        hipStream_t s = nullptr;
        if (hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess) {
            (void)hipGetLastError();
            delete b;
            return errf(RADON_ERR_DEVICE, "stream creation failed");
        }
        b->streams.push_back(s);
    }
    for (int i = 0; i < 2 * nb; ++i) {   // per direction: two forks and two joins
        hipEvent_t e = nullptr;
        if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
            (void)hipGetLastError();
            delete b;
            return errf(RADON_ERR_DEVICE, "event creation failed");
        }
        b->events.push_back(e);
    }
    const radon_status_t st = b->build();
    if (st != RADON_OK) {
        delete b;
        return st;
    }
    *out = b;
    return rn::api_ok();
}

radon_status_t radon_batch_forward(radon_batch_t batch, const float* const* imgs_dev, float* const* sinos_dev,
                                   void* stream) {
    if (!batch) return errf(RADON_ERR_INVALID, "batch is NULL");
    return batch->run(true, imgs_dev, sinos_dev, stream);
}

radon_status_t radon_batch_adjoint(radon_batch_t batch, const float* const* sinos_dev, float* const* imgs_dev,
                                   void* stream) {
    if (!batch) return errf(RADON_ERR_INVALID, "batch is NULL");
    return batch->run(false, sinos_dev, imgs_dev, stream);
}

int radon_batch_graphs_recorded(radon_batch_t batch) { return batch ? batch->recorded : -1; }

void radon_batch_destroy(radon_batch_t batch) { delete batch; }

radon_status_t radon_plan_tuning(radon_plan_t plan, radon_tuning* out) {
    if (!plan || !out) return errf(RADON_ERR_INVALID, "NULL argument");
    out->tile = plan->p.T;
    out->a2_chunk = plan->p.a2_chunk;
    out->f3_chunk = plan->p.f3_chunk;
    return rn::api_ok();
}

radon_status_t radon_autotune(int n, const double* angles, int n_views, int n_det, double sigma, int W, int repeats,
                              radon_tuning* best, double* best_ms, double* default_ms, void* stream) {
    if (!best || !best_ms) return errf(RADON_ERR_INVALID, "NULL output");
    if (repeats < 1 || repeats > 1000) return errf(RADON_ERR_INVALID, "repeats=%d must be 1..1000", repeats);
    hipStream_t st = (hipStream_t)stream;
    float *img = nullptr, *sino = nullptr, *img_out = nullptr, *sino_out = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    const size_t n_img = (size_t)n * n, n_sino = (size_t)n_views * n_det;
    auto cleanup = [&] {
        for (float* b : {img, sino, img_out, sino_out})
            if (b) (void)hipFree(b);
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
    };
    // validate the geometry once through the ordinary plan path
    radon_plan_t probe = nullptr;
    radon_status_t s = radon_plan_tuned(&probe, n, angles, n_views, n_det, sigma, W, nullptr);
    if (s != RADON_OK) return s;
    radon_tuning def{};
    (void)radon_plan_tuning(probe, &def);
    radon_plan_destroy(probe);
    if (hipMalloc(&img, sizeof(float) * n_img) != hipSuccess || hipMalloc(&sino, sizeof(float) * n_sino) != hipSuccess ||
        hipMalloc(&img_out, sizeof(float) * n_img) != hipSuccess ||
        hipMalloc(&sino_out, sizeof(float) * n_sino) != hipSuccess || hipEventCreate(&e0) != hipSuccess ||
        hipEventCreate(&e1) != hipSuccess) {
        (void)hipGetLastError();
        cleanup();
        return errf(RADON_ERR_OOM, "autotune buffers");
    }
    hipLaunchKernelGGL(k_fill_hash, dim3(1024), dim3(256), 0, st, img, n_img, 12345u);
    hipLaunchKernelGGL(k_fill_hash, dim3(1024), dim3(256), 0, st, sino, n_sino, 67890u);

    // time one decomposition: ms per forward + adjoint pair, or < 0 if it does not fit
    auto time_one = [&](const radon_tuning& t, double* ms) -> radon_status_t {
        radon_plan_t pl = nullptr;
        const radon_status_t ps = radon_plan_tuned(&pl, n, angles, n_views, n_det, sigma, W, &t);
        if (ps == RADON_ERR_UNSUPPORTED) {
            *ms = -1.0;
            return RADON_OK;
        }
        if (ps != RADON_OK) return ps;
        radon_status_t r = RADON_OK;
        for (int k = 0; k <= repeats && r == RADON_OK; ++k) {
            if (k == 1) (void)hipEventRecord(e0, st);
            r = radon_forward(pl, img, sino_out, stream);
            if (r == RADON_OK) r = radon_adjoint(pl, sino, img_out, stream);
        }
        (void)hipEventRecord(e1, st);
        float el = 0.f;
        if (r == RADON_OK && (hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&el, e0, e1) != hipSuccess)) {
            (void)hipGetLastError();
            r = errf(RADON_ERR_DEVICE, "autotune timing failed");
        }
        radon_plan_destroy(pl);
        *ms = el / repeats;
        return r;
    };

    // coordinate search: tile size first, then the spreading chunk, then the
    // forward chunk, each with the others at their current best. A candidate
    // replaces the current best only if it is faster by more than the
    // run-to-run spread: both are timed three times, interleaved, and the
    // candidate's best time must beat the current's best by 3%.
    radon_tuning cur = def;
    double cur_ms = 0.0;
    if ((s = time_one(cur, &cur_ms)) != RADON_OK) { cleanup(); return s; }
    if (default_ms) *default_ms = cur_ms;
    const int tiles[] = {8, 16, 32}, a2s[] = {256, 512}, f3s[] = {1024, 2048, 4096};
    constexpr double kMargin = 0.97;
    auto try_set = [&](radon_tuning cand) -> radon_status_t {
        if (cand.tile == cur.tile && cand.a2_chunk == cur.a2_chunk && cand.f3_chunk == cur.f3_chunk) return RADON_OK;
        double best_c = 1e300, best_cur = 1e300;
        for (int k = 0; k < 3; ++k) {
            double mc = 0.0, mk = 0.0;
            radon_status_t r = time_one(cand, &mc);
            if (r != RADON_OK) return r;
            if (mc < 0.0) return RADON_OK;   // the candidate does not fit this geometry
            if ((r = time_one(cur, &mk)) != RADON_OK) return r;
            best_c = std::min(best_c, mc);
            best_cur = std::min(best_cur, mk);
        }
        if (best_c < kMargin * best_cur) {
            cur = cand;
            cur_ms = best_c;
        } else {
            cur_ms = best_cur;
        }
        return RADON_OK;
    };
    for (int t : tiles) {
        radon_tuning c = cur;
        c.tile = t;
        if ((s = try_set(c)) != RADON_OK) { cleanup(); return s; }
    }
    for (int a : a2s) {
        radon_tuning c = cur;
        c.a2_chunk = a;
        if ((s = try_set(c)) != RADON_OK) { cleanup(); return s; }
    }
    for (int f : f3s) {
        radon_tuning c = cur;
        c.f3_chunk = f;
        if ((s = try_set(c)) != RADON_OK) { cleanup(); return s; }
    }
    cleanup();
    *best = cur;
    *best_ms = cur_ms;
    return rn::api_ok();
}

}  // extern "C"
