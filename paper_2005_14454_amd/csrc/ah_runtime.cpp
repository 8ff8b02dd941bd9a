// Host runtime of libah: parameter validation, device arena layout, the FP64
// per-step coefficient formulas, phi/A ping-pong, state I/O, diagnostics
// assembly and the C ABI declared in include/ah.h.
#include "ah.h"
#include "ah_internal.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <thread>
#include <vector>

using namespace ah;

struct ah_handle {
    ah_params p{};
    int device = 0;
    hipStream_t stream = nullptr;
    bool owns_arena = false;
    void* arena = nullptr;
    size_t arena_bytes = 0;
    int64_t V = 0;  // sites, N^3
    int P = 0;      // row pitch of the stored fields (site (x, y, z) at x + P (y + N z))
    size_t real_bytes = 8;
    // ping-pong phi/A buffers [2][5] (phr, phi, a0, a1, a2) and Pi/E buffers
    // [2][5] (pir, pii, e0, e1, e2).  A single step drifts phi and A into the
    // other buffer and kicks Pi and E in place; a two-step pass writes all
    // ten fields into the other buffers.
    void* pp[2][5] = {};
    void* mom[2][5] = {};
    int curm = 0;  // current Pi/E buffer
    double* partials = nullptr;
    // kSeriesCap folded records in pinned host memory, and the address the
    // device knows them by: the fold writes a record (120 bytes) straight to
    // the host, so no copy follows it
    double* host_series = nullptr;
    double* series = nullptr;
    IoStage io;              // state I/O (io_stage)
    char* io_mem = nullptr;  // its own memory, if it has any
    int cur = 0;
    int64_t step = 0;
    bool ready = false;
    bool timing = false;
    std::vector<hipEvent_t> ev;  // start/stop pairs
    size_t ev_used = 0;
    ah_step_config cfg{AH_KERNEL_AUTO, 0, 0, 0};
    TileConfig two{};  // tiling of the two-step passes an automatic configuration takes (zchunk 0: none)
    // Whether work of this handle has been recorded into a graph (note_capture),
    // and whether the two-step passes of automatic configurations have, all in
    // all, exchanged the buffer pairs, which single steps in their place would
    // have left where they were.
    bool captured = false;
    int swapped = 0;
    int64_t measured_launches = 0;  // timed launches that also formed diagnostics
    std::vector<char> ev_measured;  // per event pair: 1 if that launch formed diagnostics
    std::vector<char> ev_steps;     // per event pair: steps the launch advanced (1 or 2)
    std::string err;
};

namespace ah {
bool tuned_config(const ah_params& p, ah_step_config* out);  // ah_tune.cpp
}

namespace {

constexpr size_t kAlign = 256;
size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

int fail(ah_handle* h, int code, const std::string& msg)
{
    if (h) h->err = msg;
    return code;
}

int hip_fail(ah_handle* h, hipError_t e, const char* what)
{
    std::string m = std::string(what) + ": " + hipGetErrorString(e);
    return fail(h, AH_E_DEVICE, m);
}

double eta_ref_of(const ah_params& p) { return p.eta_ref > 0.0 ? p.eta_ref : 0.5 * p.dx * (double)p.N; }

// Section 2 scalars at snapshot n.
struct Scalars {
    double eta, s, a, f, delta, omega;
};
Scalars scalars_at(const ah_params& p, int64_t n)
{
    Scalars r;
    r.eta = p.eta0 + (double)n * p.deta;
    r.s = r.eta < p.eta_switch ? p.s_early : p.s_late;
    r.a = std::pow(r.eta / eta_ref_of(p), p.m);
    r.f = std::pow(r.a, 2.0 * r.s);
    r.delta = 0.5 * p.alpha * p.m * p.deta / r.eta;
    // artificial damping phase: a constant friction gamma replaces the Hubble term
    if (p.damp_gamma > 0.0 && r.eta < p.eta_damp) r.delta = 0.5 * p.damp_gamma * p.deta;
    r.omega = (1.0 - r.s) * r.delta;
    return r;
}

StepCoef coef_at(const ah_params& p, int64_t n)
{
    const Scalars s = scalars_at(p, n);
    StepCoef c;
    c.cP1 = (1.0 - s.delta) / (1.0 + s.delta);
    c.cP2 = p.deta / (1.0 + s.delta);
    c.cE1 = (1.0 - s.omega) / (1.0 + s.omega);
    c.cE2 = p.deta / (1.0 + s.omega);
    c.lam_half = 0.5 * p.lambda0 * s.f;
    c.kappa = 2.0 * p.e0 * p.e0 * s.f;
    return c;
}

// Coupling c_{n-1/2} of the Gauss residual: the kick keeps
// div E^{n-1/2} = c_{n-1/2} Im[conj(phi^n) Pi^{n-1/2}] exactly when
// c_{n-1/2} = 2 e0^2 f_{n-1} (1+delta_{n-1}) / (1+omega_{n-1}); 2 e0^2 f_0 at n = 0.
double gauss_coupling(const ah_params& p, int64_t n)
{
    if (n <= 0) return 2.0 * p.e0 * p.e0 * scalars_at(p, 0).f;
    const Scalars s = scalars_at(p, n - 1);
    return 2.0 * p.e0 * p.e0 * s.f * (1.0 + s.delta) / (1.0 + s.omega);
}

double stability_margin(const ah_params& p, int64_t n)
{
    const Scalars s = scalars_at(p, n);
    const double g = std::fmax(p.lambda0, 2.0 * p.e0 * p.e0) * s.f * p.sigma * p.sigma + 12.0 / (p.dx * p.dx);
    return p.deta * std::sqrt(g);
}

bool unstable_at(const ah_params& p, int64_t n) { return stability_margin(p, n) >= 2.0; }

}  // namespace

namespace ah {

int validate_params(const ah_params* p, std::string* why)
{
    if (!p) {
        *why = "params is NULL";
        return AH_E_INVAL;
    }
    if (p->N < 4 || p->N > 4096) {
        *why = "N must be in [4, 4096]";
        return AH_E_INVAL;
    }
    if (p->precision != AH_FP64 && p->precision != AH_FP32) {
        *why = "precision must be AH_FP64 or AH_FP32";
        return AH_E_INVAL;
    }
    if (p->gauge_action != AH_COMPACT && p->gauge_action != AH_NONCOMPACT) {
        *why = "gauge_action must be AH_COMPACT or AH_NONCOMPACT";
        return AH_E_INVAL;
    }
    if (p->reserved != 0) {
        *why = "reserved must be 0";
        return AH_E_INVAL;
    }
    if (!(p->dx > 0.0) || !(p->deta > 0.0) || !std::isfinite(p->dx) || !std::isfinite(p->deta)) {
        *why = "dx and deta must be positive and finite";
        return AH_E_INVAL;
    }
    if (!(p->eta0 > 0.0) || !std::isfinite(p->eta0)) {
        *why = "eta0 must be positive";
        return AH_E_INVAL;
    }
    if (!(p->e0 > 0.0) || !std::isfinite(p->lambda0) || !std::isfinite(p->sigma) || !std::isfinite(p->m) ||
        !std::isfinite(p->alpha) || !std::isfinite(p->s_early) || !std::isfinite(p->s_late) ||
        std::isnan(p->eta_switch) || !std::isfinite(p->eta_ref)) {
        *why = "non-finite or invalid coupling / expansion parameter (e0 must be > 0)";
        return AH_E_INVAL;
    }
    if (!(p->damp_gamma >= 0.0) || !std::isfinite(p->damp_gamma) || std::isnan(p->eta_damp)) {
        *why = "damp_gamma must be finite and >= 0, eta_damp not NaN";
        return AH_E_INVAL;
    }
    return AH_OK;
}

}  // namespace ah

namespace {

int validate(const ah_params* p, std::string* why) { return validate_params(p, why); }

size_t field_bytes(const ah_params& p)
{
    const size_t stored = (size_t)p.N * p.N * row_pitch(p.N, p.precision);
    return align_up(stored * (p.precision == AH_FP64 ? 8 : 4));
}


// Diagnostics records a handle can hold: the largest number of workgroups
// of any supported tile shape at the smallest z-chunk.
size_t partial_records(const ah_params& p)
{
    const int N = p.N;
    const int zc = min_zchunk(N);
    const int64_t tz = (N + zc - 1) / zc;
    int64_t best = 0;
    const int shapes[6][2] = {{64, 8}, {64, 4}, {32, 8}, {64, 16}, {128, 4}, {128, 8}};
    for (auto& s : shapes) {
        const int64_t t = (int64_t)((N + s[0] - 1) / s[0]) * ((N + s[1] - 1) / s[1]) * tz;
        if (t > best) best = t;
    }
    return (size_t)(best > kMeasBlocks ? best : kMeasBlocks);
}

constexpr int kSeriesCap = 1024;  // measurement records per ah_step_measured batch

size_t required_bytes(const ah_params& p)
{
    return 20 * field_bytes(p) + align_up(partial_records(p) * kMeasStride * sizeof(double));
}

template <typename R>
Fields<R> fields_of(const ah_handle* h, int buf)
{
    Fields<R> f;
    f.phr = (R*)h->pp[buf][0];
    f.phi = (R*)h->pp[buf][1];
    f.a0 = (R*)h->pp[buf][2];
    f.a1 = (R*)h->pp[buf][3];
    f.a2 = (R*)h->pp[buf][4];
    f.pir = (R*)h->mom[h->curm][0];
    f.pii = (R*)h->mom[h->curm][1];
    f.e0 = (R*)h->mom[h->curm][2];
    f.e1 = (R*)h->mom[h->curm][3];
    f.e2 = (R*)h->mom[h->curm][4];
    return f;
}

LatticeConst lconst(const ah_params& p)
{
    LatticeConst L;
    L.N = p.N;
    L.P = row_pitch(p.N, p.precision);
    L.compact = p.gauge_action == AH_COMPACT ? 1 : 0;
    L.dx = p.dx;
    L.deta = p.deta;
    L.sigma2 = p.sigma * p.sigma;
    return L;
}

}  // namespace

namespace ah {

hipError_t io_events(IoStage* st)
{
    for (hipEvent_t& ev : st->ev)
        if (!ev) {
            const hipError_t e = hipEventCreateWithFlags(&ev, hipEventDisableTiming | hipEventReleaseToSystem);
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}
void io_close(IoStage* st)
{
    for (hipEvent_t& ev : st->ev) {
        if (ev) (void)hipEventDestroy(ev);
        ev = nullptr;
    }
}

namespace {

// One host thread's share of the staging memory.
struct IoLane {
    char *host, *dev;  // kIoSlots slots of `slot` bytes, as the host and as the device know them
    size_t slot;
    const hipEvent_t* ev;
};

// Items [i0, i1) in pieces of `per`, one piece per slot: while the host works
// on one piece (fill, take) kernels move those of the other slots.
template <class Fill, class Launch>
hipError_t pieces_in(const IoLane& l, int64_t i0, int64_t i1, int64_t per, hipStream_t s, Fill fill, Launch launch)
{
    int64_t k = 0;
    for (int64_t i = i0; i < i1; i += per, ++k) {
        const int j = (int)(k % kIoSlots);
        const int64_t n = std::min(per, i1 - i);
        hipError_t e = k >= kIoSlots ? hipEventSynchronize(l.ev[j]) : hipSuccess;
        if (e != hipSuccess) return e;
        fill(l.host + j * l.slot, i, n);
        e = launch(l.dev + j * l.slot, i, n);
        if (e == hipSuccess) e = hipEventRecord(l.ev[j], s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
template <class Launch, class Take>
hipError_t pieces_out(const IoLane& l, int64_t i0, int64_t i1, int64_t per, hipStream_t s, Launch launch, Take take)
{
    const int64_t pieces = (i1 - i0 + per - 1) / per;
    for (int64_t k = 0; k < pieces + kIoSlots; ++k) {
        const int j = (int)(k % kIoSlots);
        hipError_t e = hipSuccess;
        if (k >= kIoSlots) {
            e = hipEventSynchronize(l.ev[j]);
            if (e != hipSuccess) return e;
            const int64_t i = i0 + (k - kIoSlots) * per;
            take(l.host + j * l.slot, i, std::min(per, i1 - i));
        }
        if (k < pieces) {
            const int64_t i = i0 + k * per;
            e = launch(l.dev + j * l.slot, i, std::min(per, i1 - i));
            if (e == hipSuccess) e = hipEventRecord(l.ev[j], s);
            if (e != hipSuccess) return e;
        }
        if (k + 1 >= pieces && k + 1 < kIoSlots) k = kIoSlots - 1;  // fewer pieces than slots: on to the waits
    }
    return hipSuccess;
}

// work(lane, i0, i1) over items [0, n), split between up to `most` host threads
// with a lane each, one for every 16 MB of the caller's array.  A thread
// converts 20 to 30 GB/s, far less into memory it is the first to touch, where
// the host link carries 50.  MI355X, one / two / four threads: 160^3 FP64 out
// 24.0 / 13.6 / 11.3 ms (ten 1-D copies 31.6), 90^3 FP32 out 3.8 / 2.3 / 1.6.
// The way in stops at two: 160^3 FP64 12.1 / 9.3 / 11.6 ms (four threads' pieces
// are so small that the launches bound it; copies 12.0), 90^3 FP32 2.0 / 1.4 /
// 1.3.
template <class Work>
hipError_t split_lanes(const IoStage& st, int64_t n, int most, size_t host_bytes, hipStream_t s, Work work)
{
    constexpr size_t least = 64u << 10;  // a slot; at least a row of the longest side where there is one lane
    // hipStreamPerThread is another stream in each thread: a helper's launches
    // would be ordered neither behind the caller's work nor ahead of its
    // synchronisation, so the caller makes them all
    if (s == hipStreamPerThread) most = 1;
    const size_t lanes = std::min(1 + (host_bytes >> 24), std::max(st.bytes / (kIoSlots * least), (size_t)1));
    const int T = (int)std::min<int64_t>(most, std::min<int64_t>(n, (int64_t)lanes));
    void* dev = nullptr;
    int device = 0;
    hipError_t e = hipHostGetDevicePointer(&dev, st.host, 0);
    if (e == hipSuccess) e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    // so little that the link takes a few us for it goes in one piece: each has
    // a launch and an event (MI355X, windings of 33^3: 38 us in three, 28 in one)
    const bool whole = T == 1 && host_bytes <= std::min(st.bytes, (size_t)128 << 10);
    const size_t slot = whole ? st.bytes : st.bytes / (T * kIoSlots) / 256 * 256;
    hipError_t err[kIoThreads] = {};
    auto run = [&](int t) {
        const IoLane l{st.host + t * kIoSlots * slot, (char*)dev + t * kIoSlots * slot, slot, st.ev + t * kIoSlots};
        err[t] = work(l, n * t / T, n * (t + 1) / T);
    };
    std::thread helpers[kIoThreads];
    for (int t = 1; t < T; ++t) {
        try {
            helpers[t] = std::thread([&, t] {
                err[t] = hipSetDevice(device);
                if (err[t] == hipSuccess) run(t);
            });
        } catch (...) {
            run(t);  // no more threads to be had
        }
    }
    run(0);
    for (int t = 1; t < T; ++t)
        if (helpers[t].joinable()) helpers[t].join();
    for (int t = 0; t < T; ++t)
        if (err[t] != hipSuccess) {
            (void)hipStreamSynchronize(s);  // nothing uses the staging memory once the call has failed
            return err[t];
        }
    return hipSuccess;
}

}  // namespace

template <typename R>
hipError_t state_upload(void* pp, void* mom, size_t fs, const double* host, int N, int P, const IoStage& st, hipStream_t s)
{
    const int64_t rows = 10 * (int64_t)N * N;
    const hipError_t e = split_lanes(st, rows, 2, rows * N * sizeof(double), s, [=](const IoLane& l, int64_t r0, int64_t r1) {
        const int64_t per = (int64_t)(l.slot / (N * sizeof(R)));
        if (per < 1) return hipErrorInvalidValue;
        return pieces_in(
            l, r0, r1, per, s,
            [=](char* slot, int64_t r, int64_t n) {
                const double* src = host + r * N;
                R* dst = (R*)slot;
                for (int64_t i = 0; i < n * N; ++i) dst[i] = (R)src[i];
            },
            [=](char* slot, int64_t r, int64_t n) {
                return launch_state_rows<R>(pp, mom, fs, N, P, r, n, (R*)slot, false, s);
            });
    });
    const hipError_t done = hipStreamSynchronize(s);
    return e != hipSuccess ? e : done;
}
template <typename R>
hipError_t state_download(void* pp, void* mom, size_t fs, double* host, int N, int P, const IoStage& st, hipStream_t s)
{
    const int64_t rows = 10 * (int64_t)N * N;
    return split_lanes(st, rows, kIoThreads, rows * N * sizeof(double), s, [=](const IoLane& l, int64_t r0, int64_t r1) {
        const int64_t per = (int64_t)(l.slot / (N * sizeof(R)));
        if (per < 1) return hipErrorInvalidValue;
        return pieces_out(
            l, r0, r1, per, s,
            [=](char* slot, int64_t r, int64_t n) {
                return launch_state_rows<R>(pp, mom, fs, N, P, r, n, (R*)slot, true, s);
            },
            [=](const char* slot, int64_t r, int64_t n) {
                double* dst = host + r * N;
                const R* src = (const R*)slot;
                for (int64_t i = 0; i < n * N; ++i) dst[i] = (double)src[i];
            });
    });
}
template hipError_t state_upload<double>(void*, void*, size_t, const double*, int, int, const IoStage&, hipStream_t);
template hipError_t state_upload<float>(void*, void*, size_t, const double*, int, int, const IoStage&, hipStream_t);
template hipError_t state_download<double>(void*, void*, size_t, double*, int, int, const IoStage&, hipStream_t);
template hipError_t state_download<float>(void*, void*, size_t, double*, int, int, const IoStage&, hipStream_t);

hipError_t bytes_download(const void* dev, void* host, size_t bytes, const IoStage& st, hipStream_t s)
{
    constexpr int64_t block = 256;
    return split_lanes(st, ((int64_t)bytes + block - 1) / block, kIoThreads, bytes, s, [=](const IoLane& l, int64_t b0, int64_t b1) {
        auto len = [=](int64_t b, int64_t n) { return std::min(n * block, (int64_t)bytes - b * block); };
        return pieces_out(
            l, b0, b1, (int64_t)l.slot / block, s,
            [=](char* slot, int64_t b, int64_t n) {
                return launch_bytes((const char*)dev + b * block, slot, len(b, n), s);
            },
            [=](const char* slot, int64_t b, int64_t n) { std::memcpy((char*)host + b * block, slot, len(b, n)); });
    });
}

}  // namespace ah

namespace {

// The handle's staging memory: its own (an eighth of the lattice's state,
// 512 KB to kIoBytes), allocated at the first use that needs more than the
// record memory holds and kept until the handle is destroyed; the record
// memory (idle between calls) where that is enough, or if no more can be had.
hipError_t io_stage(ah_handle* h, size_t want, IoStage** out)
{
    constexpr size_t records = (size_t)kSeriesCap * kMeasStride * sizeof(double);
    *out = &h->io;
    if (!h->io_mem && want > records) {
        const size_t state = 10 * (size_t)h->V * h->real_bytes;
        const size_t n = std::min(kIoBytes, std::max(align_up(state / 8), (size_t)512 << 10));
        void* m = nullptr;
        if (hipHostMalloc(&m, n, hipHostMallocDefault) == hipSuccess) {
            h->io.host = h->io_mem = (char*)m;
            h->io.bytes = n;
        } else {
            (void)hipGetLastError();
        }
    }
    if (!h->io.host) {
        h->io.host = (char*)h->host_series;
        h->io.bytes = records;
    }
    return io_events(&h->io);
}

struct DeviceGuard {
    int prev = -1;
    explicit DeviceGuard(int dev)
    {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        if (prev != dev) (void)hipSetDevice(dev);
    }
    ~DeviceGuard()
    {
        int now = -1;
        if (prev >= 0 && hipGetDevice(&now) == hipSuccess && now != prev) (void)hipSetDevice(prev);
    }
};


}  // namespace

namespace ah {

// Step rates of the one-step tile shapes on a lattice they tile exactly
// (MI355X, 512^3, best z-chunk; 1e9 site-updates/s; 0: no such instance).
namespace {
struct ShapeRate {
    int tx, ty;
    double fp32, fp64;
};
constexpr ShapeRate kShapeRates[] = {
    {128, 4, 67.0, 0.0}, {128, 8, 65.8, 0.0}, {64, 8, 65.8, 30.2}, {64, 4, 61.3, 29.7}, {32, 8, 60.2, 29.8},
};
}  // namespace

bool default_tile(int precision, int N, int* tx, int* ty)
{
    double best = 0.0;
    for (const ShapeRate& r : kShapeRates) {
        const double rate = precision == AH_FP64 ? r.fp64 : r.fp32;
        if (rate <= 0.0 || !tile_supported(precision, r.tx, r.ty) || !batch_tile_supported(precision, r.tx, r.ty))
            continue;
        // a ragged last tile in x or y runs idle lanes
        const double rx = (double)((N + r.tx - 1) / r.tx * r.tx) / N, ry = (double)((N + r.ty - 1) / r.ty * r.ty) / N;
        const double score = rate / (rx * ry);
        if (score > best) {
            best = score;
            *tx = r.tx;
            *ty = r.ty;
        }
    }
    return best > 0.0;
}

int resident_per_cu(int kernel, int precision, int tx, int ty, bool measured)
{
    if (kernel == AH_KERNEL_TILE2) {
        // waves per SIMD at the pass's registers: FP32 3, FP64 2; the FP64
        // pass's LDS (over 150 KB) admits one workgroup per CU
        if (precision == AH_FP64) return 1;
        const int nt = tx * ty, ring = (tx + 2) * (ty + 2) - nt;
        const int waves = (nt + (ring + 63) / 64 * 64) / 64;
        return std::max(1, 12 / waves);
    }
    // waves per SIMD at the march's registers: plain FP32 4, FP64 2; the
    // measured march 2 in both precisions
    const int waves = (tx * ty + 63) / 64;
    return std::max(1, (precision == AH_FP64 || measured ? 8 : 16) / waves);
}

// Planes' worth of time that a chunk's start takes.
int start_planes(int kernel, int tx, int ty)
{
    return kernel != AH_KERNEL_TILE2 ? 1 : (tx * ty > 256 ? 4 : 3);
}

namespace {

// Estimated time of a tiled launch with z-chunks of zc planes, in units of
// the time a workgroup that has its CU to itself takes for a plane.
//
// Workgroups run in rounds of (CUs x resident workgroups), each as long as
// a chunk's planes and its start (start_planes).  A round in which all
// of a CU's places are taken lasts `full` times as long as one in which a
// workgroup has its CU to itself.  Both fitted to a sweep on MI355X (27 sizes
// of 24 .. 640, seven kernel and tile shapes in both precisions, up to 16
// z-chunks each): the z-chunk chosen by it is within 0.6% of the fastest
// on average (3% for the plain FP32 march on its smallest tiles), where
// rounds x (planes + 2) with no `full` was up to 9% (two-step 32 x 8, which
// then put two workgroups on some CUs of a 48^3 lattice and ran at 10.6
// rather than 7.0 us per step).
double launch_estimate(int kernel, int precision, int N, int tx, int ty, bool measured, int zc, int* nblocks)
{
    constexpr int kCUs = 256;
    const int res = resident_per_cu(kernel, precision, tx, ty, measured);
    const bool two = kernel == AH_KERNEL_TILE2;
    const double full = res == 1 ? 1.0 : two ? 2.0 : (precision == AH_FP64 || measured ? 1.6 : (res == 2 ? 1.4 : 1.8));
    const int ramp = start_planes(kernel, tx, ty);
    const int nb = ((N + tx - 1) / tx) * ((N + ty - 1) / ty) * ((N + zc - 1) / zc);  // < 2^28 for N <= 4096
    const int slots = kCUs * res;
    const int left = (nb % slots + kCUs - 1) / kCUs;  // workgroups per CU of the last round
    double rounds = (double)(nb / slots) * full;
    if (left > 0) rounds += res == 1 ? 1.0 : 1.0 + (full - 1.0) * (double)(left - 1) / (res - 1);
    if (nblocks) *nblocks = nb;
    return rounds * (zc + ramp);
}

}  // namespace

int auto_zchunk(int kernel, int precision, int N, int tx, int ty, bool measured)
{
    // Equal chunks (a short last one would leave most of its round idle), of
    // the least estimated time; among equal estimates the one with more
    // workgroups, which spread more evenly over the XCDs.
    const int zmin = std::min(min_zchunk(N), N);
    int best_zc = N;
    double best_t = -1.0;
    int best_nb = 0;
    for (int nz = 1, last = 0; nz <= N / zmin; ++nz) {
        const int zc = (N + nz - 1) / nz;
        if (zc < zmin) break;
        if (zc == last) continue;
        last = zc;
        int nb = 0;
        const double t = launch_estimate(kernel, precision, N, tx, ty, measured, zc, &nb);
        if (best_t < 0 || t < best_t || (t == best_t && nb > best_nb)) {
            best_t = t;
            best_nb = nb;
            best_zc = zc;
        }
    }
    return best_zc;
}

// Two-step passes of an automatic configuration, where they pay: FP64 on 32 x 8
// (MI355X, 512^3: 3640 us a step, 64 x 4 5310); FP32 on 64 x 8 or 32 x 8,
// whichever the estimate says is faster (a plane takes a workgroup alone on its
// CU 1.5 times as long on 64 x 8).
TileConfig default_two(int precision, int N)
{
    TileConfig two{0, 0, 0};
    if (!two_step_pays(precision, N)) return two;
    double best = 0.0;
    for (const int tx : {64, 32}) {
        if (!tile2_supported(precision, tx, 8)) continue;
        const int zc = auto_zchunk(AH_KERNEL_TILE2, precision, N, tx, 8, false);
        const double t = launch_estimate(AH_KERNEL_TILE2, precision, N, tx, 8, false, zc, nullptr) * (tx == 64 ? 1.5 : 1.0);
        if (two.zchunk == 0 || t < best) {
            best = t;
            two = TileConfig{tx, 8, zc};
        }
    }
    return two;
}

// Any tile shape computes the same fields bit for bit, so the measured march
// may run another shape than the plain step: the fastest measured march
// (measured_tile: 32 x 8).  A one-step march on that shape lends it its z-chunk;
// on another shape it leaves it its own automatic one, no shorter than the
// step's up to 16 planes (a pool's floor of 16 then holds for its measured
// node too).  A two-step pass lends it its z-chunk only where the estimate
// finds that as good: one of its workgroups fills a CU, so its z-chunks are
// long, and on them the measured march has one workgroup on a CU where two fit
// (MI355X, ah_measure in us on the pass's z-chunk / on its own: FP64 96^3 71.5 /
// 59.7, 128^3 131.6 / 102.1, 256^3 902 / 632, FP32 96^3 57.9 / 46.0; but 512^3
// FP64, where the estimates are 0.2% apart, 4820 / 4970).  The diagnostics
// records are summed in tile order, so a lattice measured with the same tiling
// (alone or in a pool) gets the same bits.
TileConfig measured_tiling(const ah_params& p, const ah_step_config& cfg)
{
    int tx = cfg.tile_x, ty = cfg.tile_y;
    const bool march = cfg.kernel == AH_KERNEL_TILE;
    const bool other = measured_tile(&tx, &ty);
    if (!other && march) return TileConfig{tx, ty, cfg.zchunk};
    int zc = auto_zchunk(AH_KERNEL_TILE, p.precision, p.N, tx, ty, true);
    if (march) {
        zc = std::min(std::max(zc, std::min(cfg.zchunk, 16)), p.N);
    } else if (!other && cfg.kernel == AH_KERNEL_TILE2) {
        auto time = [&](int c) { return launch_estimate(AH_KERNEL_TILE, p.precision, p.N, tx, ty, true, c, nullptr); };
        if (time(cfg.zchunk) <= 1.01 * time(zc)) zc = cfg.zchunk;
    }
    return TileConfig{tx, ty, zc};
}

// Resolve automatic choices of a step configuration for the lattice.
int resolve_step_config(const ah_params& p, const ah_step_config& in, ah_step_config* out, std::string* why)
{
    ah_step_config c = in;
    if (c.kernel == AH_KERNEL_AUTO) c.kernel = p.gauge_action == AH_COMPACT ? AH_KERNEL_TILE : AH_KERNEL_SITE;
    if (c.kernel != AH_KERNEL_SITE && c.kernel != AH_KERNEL_TILE && c.kernel != AH_KERNEL_TILE2) {
        *why = "unknown kernel";
        return AH_E_INVAL;
    }
    if (c.kernel == AH_KERNEL_SITE) {
        c.tile_x = c.tile_y = c.zchunk = 0;
        *out = c;
        return AH_OK;
    }
    if (p.gauge_action != AH_COMPACT) {
        *why = "the tiled kernel supports the compact gauge action only";
        return AH_E_INVAL;
    }
    if (c.tile_x == 0 && c.tile_y == 0) {
        // one step: the shape of the highest rate once its ragged edge is
        // paid for; two-step passes: 32 x 8 in both precisions
        c.tile_x = 32;
        c.tile_y = 8;
        if (c.kernel == AH_KERNEL_TILE) (void)default_tile(p.precision, p.N, &c.tile_x, &c.tile_y);
    }
    if (c.kernel == AH_KERNEL_TILE2 ? !tile2_supported(p.precision, c.tile_x, c.tile_y)
                                    : !tile_supported(p.precision, c.tile_x, c.tile_y)) {
        *why = "unsupported tile shape";
        return AH_E_INVAL;
    }
    if (c.zchunk < 0 || (c.zchunk > 0 && c.zchunk < min_zchunk(p.N))) {
        *why = "zchunk must be 0 (automatic) or at least 2 (N <= 128) or 8 (N > 128)";
        return AH_E_INVAL;
    }
    if (c.zchunk == 0) c.zchunk = auto_zchunk(c.kernel, p.precision, p.N, c.tile_x, c.tile_y, false);
    if (c.zchunk > p.N) c.zchunk = p.N;
    *out = c;
    return AH_OK;
}

// One FP64 row of a lattice's coefficient table for snapshot n (kick
// coefficients and diagnostics constants).
void coef_row(const ah_params& p, int64_t n, double* row)
{
    const Scalars s = scalars_at(p, n);
    const StepCoef c = coef_at(p, n);
    for (int k = 0; k < kCoefStride; ++k) row[k] = 0.0;
    row[C_P1] = c.cP1;
    row[C_P2] = c.cP2;
    row[C_E1] = c.cE1;
    row[C_E2] = c.cE2;
    row[C_LAMH] = c.lam_half;
    row[C_KAPPA] = c.kappa;
    row[C_INV2E2F] = 1.0 / (2.0 * p.e0 * p.e0 * s.f);
    row[C_LAMQ] = 0.25 * p.lambda0 * s.f;
    row[C_GAUSS] = gauss_coupling(p, n);
}

// Diagnostics of snapshot `step` from the folded FP64 sums r[M_COUNT].
void to_measurement(const ah_params& p, int64_t step, const double* r, int64_t V, ah_measurement* out)
{
    const Scalars sc = scalars_at(p, step);
    const double dx3 = p.dx * p.dx * p.dx;
    const double vol = std::pow((double)p.N * p.dx, 3.0);
    std::memset(out, 0, sizeof(*out));
    out->step = step;
    out->eta = sc.eta;
    out->a = sc.a;
    out->f = sc.f;
    out->winding_sum_abs = (int64_t)r[M_WABS];
    out->L_W = p.dx * r[M_WABS];
    out->xi_W = std::sqrt(vol / out->L_W);
    out->e_kin = dx3 * r[M_KIN];
    out->e_grad = dx3 * r[M_GRAD];
    out->e_pot = dx3 * r[M_POT];
    out->e_el = dx3 * r[M_EL];
    out->e_mag = dx3 * r[M_MAG];
    out->energy = out->e_kin + out->e_grad + out->e_pot + out->e_el + out->e_mag;
    out->sum_L = dx3 * ((((r[M_KIN] - r[M_GRAD]) - r[M_POT]) + r[M_EL]) - r[M_MAG]);
    out->xi_L = out->sum_L < 0.0 ? std::sqrt(-2.0 * M_PI * p.sigma * p.sigma * vol / out->sum_L) : NAN;
    out->R = r[M_KINL] / r[M_GRADL];
    out->v2_phi = 2.0 * out->R / (1.0 + out->R);
    out->v2_omega = 0.5 * (1.0 + 3.0 * r[M_PL] / r[M_RHOL]);
    out->gauss_rms = std::sqrt(r[M_G2] / (double)V);
    out->gauss_max = r[M_GMAX];
    const double den = std::sqrt(r[M_DIV2] + r[M_CRHO2]);
    out->gauss_rel = den > 0.0 ? std::sqrt(r[M_G2]) / den : 0.0;
    out->nonfinite = (int64_t)r[M_NONFIN];
    out->flags = (unstable_at(p, step) ? AH_FLAG_UNSTABLE : 0u) | (out->nonfinite ? AH_FLAG_NONFINITE : 0u);
}

}  // namespace ah

namespace {

// A handle's configuration; one that leaves everything automatic takes the
// tuned one, or else two-step passes where they are faster (two).
int resolve_config(const ah_params& p, const ah_step_config& in, ah_step_config* out, TileConfig* two,
                   std::string* why)
{
    *two = TileConfig{0, 0, 0};
    if (in.kernel == AH_KERNEL_AUTO && in.tile_x == 0 && in.tile_y == 0 && in.zchunk == 0 &&
        p.gauge_action == AH_COMPACT) {
        ah_step_config tuned;
        if (tuned_config(p, &tuned)) {
            const int rc = resolve_step_config(p, tuned, out, why);
            if (rc == AH_OK && out->kernel == AH_KERNEL_TILE2) *two = TileConfig{out->tile_x, out->tile_y, out->zchunk};
            return rc;
        }
        *two = default_two(p.precision, p.N);
    }
    return resolve_step_config(p, in, out, why);
}

MeasConst meas_const(const ah_params& p, int64_t n)
{
    const Scalars sc = scalars_at(p, n);
    MeasConst mc;
    mc.inv_2e2f = 1.0 / (2.0 * p.e0 * p.e0 * sc.f);
    mc.lam_quarter = 0.25 * p.lambda0 * sc.f;
    mc.gauss_c = gauss_coupling(p, n);
    return mc;
}

// Tiling of the measured march (diagnostics of a compact-action handle).
TileConfig meas_tiles(const ah_handle* h)
{
    return measured_tiling(h->p, h->cfg);
}

// Diagnostics of the current snapshot folded into dst[M_COUNT] (a record of h->series), and
// with `advance` the step of that snapshot in the same pass, which writes Pi
// and E into the other buffer (the Gauss residual reads E of neighbours).
template <typename R>
hipError_t measured_pass(ah_handle* h, double* dst, bool advance)
{
    const ah_params& p = h->p;
    const StepCoef c = coef_at(p, h->step);
    const MeasConst mc = meas_const(p, h->step);
    const TileConfig tc = meas_tiles(h);
    const Fields<R> in = fields_of<R>(h, h->cur);
    Fields<R> out = fields_of<R>(h, h->cur ^ 1);
    const int om = h->curm ^ 1;
    out.pir = (R*)h->mom[om][0];
    out.pii = (R*)h->mom[om][1];
    out.e0 = (R*)h->mom[om][2];
    out.e1 = (R*)h->mom[om][3];
    out.e2 = (R*)h->mom[om][4];
    hipError_t e;
    if (advance && h->timing) {
        if (h->ev_used + 2 > h->ev.size()) {
            for (int k = 0; k < 2; ++k) {
                hipEvent_t ev;
                e = hipEventCreate(&ev);
                if (e != hipSuccess) return e;
                h->ev.push_back(ev);
            }
        }
        e = hipEventRecord(h->ev[h->ev_used], h->stream);
        if (e != hipSuccess) return e;
    }
    const int nb = step_tile_blocks(p.N, tc);
    e = launch_step_tile<R>(in, out, lconst(p), c, tc, &mc, h->partials, advance, h->stream);
    if (e != hipSuccess) return e;
    if (advance && h->timing) {
        e = hipEventRecord(h->ev[h->ev_used + 1], h->stream);
        if (e != hipSuccess) return e;
        h->ev_used += 2;
        h->measured_launches += 1;
        h->ev_measured.push_back(1);
        h->ev_steps.push_back(1);
    }
    e = launch_measure_final(h->partials, nb, dst, h->stream);
    if (e != hipSuccess) return e;
    if (advance) {
        h->cur ^= 1;
        h->curm ^= 1;
        h->step += 1;
    }
    return hipSuccess;
}

// Brackets a step launch with an event pair while timing is on.
struct TimedLaunch {
    ah_handle* h;
    int steps;
    hipError_t begin()
    {
        if (!h->timing) return hipSuccess;
        if (h->ev_used + 2 > h->ev.size()) {
            for (int k = 0; k < 2; ++k) {
                hipEvent_t ev;
                const hipError_t e = hipEventCreate(&ev);
                if (e != hipSuccess) return e;
                h->ev.push_back(ev);
            }
        }
        return hipEventRecord(h->ev[h->ev_used], h->stream);
    }
    hipError_t end()
    {
        if (!h->timing) return hipSuccess;
        const hipError_t e = hipEventRecord(h->ev[h->ev_used + 1], h->stream);
        if (e != hipSuccess) return e;
        h->ev_used += 2;
        h->ev_measured.push_back(0);
        h->ev_steps.push_back((char)steps);
        return hipSuccess;
    }
};

template <typename R>
hipError_t do_step(ah_handle* h)
{
    const Fields<R> in = fields_of<R>(h, h->cur);
    const Fields<R> out = fields_of<R>(h, h->cur ^ 1);
    const StepCoef c = coef_at(h->p, h->step);
    TimedLaunch t{h, 1};
    hipError_t e = t.begin();
    if (e != hipSuccess) return e;
    if (h->cfg.kernel == AH_KERNEL_TILE || h->cfg.kernel == AH_KERNEL_TILE2) {
        TileConfig tc{h->cfg.tile_x, h->cfg.tile_y, h->cfg.zchunk};
        if (h->cfg.kernel == AH_KERNEL_TILE2) {
            // a single step between two-step passes runs the default one-step
            // tiling (every tiling gives the same fields)
            if (default_tile(h->p.precision, h->p.N, &tc.tx, &tc.ty))
                tc.zchunk = auto_zchunk(AH_KERNEL_TILE, h->p.precision, h->p.N, tc.tx, tc.ty, false);
        }
        e = launch_step_tile<R>(in, out, lconst(h->p), c, tc, nullptr, nullptr, true, h->stream);
    } else {
        e = launch_step<R>(in, out.phr, out.phi, out.a0, out.a1, out.a2, lconst(h->p), c, h->stream);
    }
    if (e != hipSuccess) return e;
    e = t.end();
    if (e != hipSuccess) return e;
    h->cur ^= 1;
    h->step += 1;
    return hipSuccess;
}

// A graph holds the addresses of the buffers that its steps read and wrote
// when they were recorded.  Whoever replays it between calls counts on an even
// number of plain steps to leave the snapshot in those buffers, and on ah_init
// and ah_set_state to put a new one there.  Single steps do; a two-step pass
// exchanges both pairs.  So a handle remembers that work of it was recorded:
// from then on the passes of an automatic configuration come in twos
// (plain_steps), and a new snapshot goes to the pair that single steps in the
// place of the passes before would have it in (first_pair).
void note_capture(ah_handle* h)
{
    if (h->captured) return;
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(h->stream, &st) != hipSuccess) {
        (void)hipGetLastError();  // the launch will say what is wrong
        return;
    }
    h->captured = st != hipStreamCaptureStatusNone;
}
// The buffers that a new snapshot goes to.
void first_pair(ah_handle* h)
{
    if (!h->captured) h->swapped = 0;
    h->cur = h->curm = h->swapped;
}

// Two steps in one pass on tiling tc: reads snapshot n from the
// current buffers and writes snapshot n+2 into the other phi/A and Pi/E ones.
template <typename R>
hipError_t do_step2(ah_handle* h, const TileConfig& tc)
{
    Fields<R> in = fields_of<R>(h, h->cur);
    Fields<R> out = fields_of<R>(h, h->cur ^ 1);
    const int om = h->curm ^ 1;
    out.pir = (R*)h->mom[om][0];
    out.pii = (R*)h->mom[om][1];
    out.e0 = (R*)h->mom[om][2];
    out.e1 = (R*)h->mom[om][3];
    out.e2 = (R*)h->mom[om][4];
    const StepCoef c0 = coef_at(h->p, h->step), c1 = coef_at(h->p, h->step + 1);
    TimedLaunch t{h, 2};
    hipError_t e = t.begin();
    if (e != hipSuccess) return e;
    e = launch_step2_tile<R>(in, out, lconst(h->p), c0, c1, tc, h->stream);
    if (e != hipSuccess) return e;
    e = t.end();
    if (e != hipSuccess) return e;
    h->cur ^= 1;
    h->curm ^= 1;
    h->step += 2;
    return hipSuccess;
}

// nsteps plain steps: two-step passes while at least two remain when the
// handle's kernel is AH_KERNEL_TILE2 or its automatic configuration takes
// them, single steps otherwise.  An automatic configuration takes an even
// number of passes a call once work of the handle has been recorded into a
// graph: every buffer is then where single steps would have left it.
hipError_t plain_steps(ah_handle* h, int64_t nsteps)
{
    note_capture(h);
    const bool automatic = h->two.zchunk > 0;
    TileConfig tc = h->two;
    if (!automatic && h->cfg.kernel == AH_KERNEL_TILE2) tc = TileConfig{h->cfg.tile_x, h->cfg.tile_y, h->cfg.zchunk};
    int64_t passes = tc.zchunk > 0 ? nsteps / 2 : 0;
    if (automatic && h->captured) passes -= passes % 2;
    const int64_t singles = nsteps - 2 * passes;
    for (int64_t k = 0; k < passes; ++k) {
        const hipError_t e = h->p.precision == AH_FP64 ? do_step2<double>(h, tc) : do_step2<float>(h, tc);
        if (e != hipSuccess) return e;
        if (automatic) h->swapped ^= 1;
    }
    for (int64_t k = 0; k < singles; ++k) {
        const hipError_t e = h->p.precision == AH_FP64 ? do_step<double>(h) : do_step<float>(h);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace

extern "C" {

int ah_params_default(ah_params* p)
{
    if (!p) return AH_E_INVAL;
    std::memset(p, 0, sizeof(*p));
    p->N = 64;
    p->precision = AH_FP64;
    p->gauge_action = AH_COMPACT;
    p->dx = 0.5;
    p->deta = 0.1;
    p->lambda0 = 2.0;
    p->e0 = 1.0;
    p->sigma = 1.0;
    p->m = 1.0;
    p->alpha = 2.0;
    p->s_early = 0.0;
    p->s_late = 0.0;
    p->eta_switch = HUGE_VAL;
    p->eta0 = 1.0;
    p->eta_ref = 0.0;
    p->damp_gamma = 0.0;  // no artificial damping phase
    p->eta_damp = 0.0;
    return AH_OK;
}

int ah_stability_margin(const ah_params* p, int64_t step, double* mu)
{
    return no_throw([&]() -> int {
        std::string why;
        if (validate(p, &why) != AH_OK || step < 0 || !mu) return AH_E_INVAL;
        *mu = stability_margin(*p, step);
        return AH_OK;
    });
}

int ah_required_bytes(const ah_params* p, size_t* bytes)
{
    return no_throw([&]() -> int {
        std::string why;
        int rc = validate(p, &why);
        if (rc != AH_OK) return rc;
        if (!bytes) return AH_E_INVAL;
        *bytes = required_bytes(*p);
        return AH_OK;
    });
}

int ah_create(const ah_params* p, void* dev_arena, size_t arena_bytes, void* hip_stream, ah_handle** out)
{
    return no_throw([&]() -> int {
        if (!out) return AH_E_INVAL;
        *out = nullptr;
        std::string why;
        int rc = validate(p, &why);
        if (rc != AH_OK) {
            std::fprintf(stderr, "ah_create: %s\n", why.c_str());
            return rc;
        }
        ah_handle* h = new (std::nothrow) ah_handle;
        if (!h) return AH_E_NOMEM;
        h->p = *p;
        h->stream = (hipStream_t)hip_stream;
        h->V = (int64_t)p->N * p->N * p->N;
        h->P = row_pitch(p->N, p->precision);
        h->real_bytes = p->precision == AH_FP64 ? 8 : 4;
        hipError_t e = hipGetDevice(&h->device);
        if (e != hipSuccess) {
            delete h;
            return AH_E_DEVICE;
        }
        const size_t need = required_bytes(*p);
        if (dev_arena) {
            if (arena_bytes < need || ((uintptr_t)dev_arena % kAlign) != 0) {
                delete h;
                return AH_E_NOMEM;
            }
            h->arena = dev_arena;
            h->arena_bytes = arena_bytes;
        } else {
            e = hipMalloc(&h->arena, need);
            if (e != hipSuccess) {
                (void)hipGetLastError();
                delete h;
                return AH_E_NOMEM;
            }
            h->owns_arena = true;
            h->arena_bytes = need;
        }
        char* base = (char*)h->arena;
        const size_t fb = field_bytes(*p);
        for (int b = 0; b < 2; ++b)
            for (int c = 0; c < 5; ++c) {
                h->pp[b][c] = base;
                base += fb;
            }
        for (int b = 0; b < 2; ++b)
            for (int c = 0; c < 5; ++c) {
                h->mom[b][c] = base;
                base += fb;
            }
        h->partials = (double*)base;
        e = hipHostMalloc((void**)&h->host_series, (size_t)kSeriesCap * kMeasStride * sizeof(double),
                          hipHostMallocDefault);
        if (e == hipSuccess) e = hipHostGetDevicePointer((void**)&h->series, h->host_series, 0);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            if (h->host_series) (void)hipHostFree(h->host_series);
            if (h->owns_arena) (void)hipFree(h->arena);
            delete h;
            return AH_E_NOMEM;
        }
        {
            std::string why2;
            const ah_step_config dflt{AH_KERNEL_AUTO, 0, 0, 0};
            if (resolve_config(h->p, dflt, &h->cfg, &h->two, &why2) != AH_OK) {
                (void)hipHostFree(h->host_series);
                if (h->owns_arena) (void)hipFree(h->arena);
                delete h;
                return AH_E_INVAL;
            }
        }
        *out = h;
        return AH_OK;
    });
}

int ah_set_step_config(ah_handle* h, const ah_step_config* c)
{
    return no_throw([&]() -> int {
        if (!h || !c) return fail(h, AH_E_INVAL, "ah_set_step_config: bad argument");
        std::string why;
        ah_step_config r;
        TileConfig two;
        int rc = resolve_config(h->p, *c, &r, &two, &why);
        if (rc != AH_OK) return fail(h, rc, "ah_set_step_config: " + why);
        h->cfg = r;
        h->two = two;
        return AH_OK;
    });
}

int ah_get_step_config(const ah_handle* h, ah_step_config* c)
{
    if (!h || !c) return AH_E_INVAL;
    *c = h->cfg;
    return AH_OK;
}

int ah_init(ah_handle* h, uint64_t seed)
{
    return no_throw([&]() -> int {
        if (!h) return AH_E_INVAL;
        DeviceGuard g(h->device);
        note_capture(h);
        first_pair(h);
        h->step = 0;
        hipError_t e = h->p.precision == AH_FP64
                           ? launch_init<double>(fields_of<double>(h, h->cur), h->p.N, h->P, h->p.sigma, seed, h->stream)
                           : launch_init<float>(fields_of<float>(h, h->cur), h->p.N, h->P, h->p.sigma, seed, h->stream);
        if (e != hipSuccess) return hip_fail(h, e, "ah_init launch");
        h->ready = true;
        return AH_OK;
    });
}

int ah_set_state(ah_handle* h, const double* host_soa, int64_t step)
{
    return no_throw([&]() -> int {
        if (!h || !host_soa || step < 0) return fail(h, AH_E_INVAL, "ah_set_state: bad argument");
        DeviceGuard g(h->device);
        hipError_t e = hipStreamSynchronize(h->stream);
        if (e != hipSuccess) return hip_fail(h, e, "ah_set_state sync");
        first_pair(h);
        IoStage* st = nullptr;
        e = io_stage(h, 10 * (size_t)h->V * h->real_bytes, &st);
        const size_t fb = field_bytes(h->p);
        void *pp = h->pp[h->cur][0], *mom = h->mom[h->curm][0];
        if (e == hipSuccess)
            e = h->real_bytes == 8 ? state_upload<double>(pp, mom, fb, host_soa, h->p.N, h->P, *st, h->stream)
                                   : state_upload<float>(pp, mom, fb, host_soa, h->p.N, h->P, *st, h->stream);
        if (e != hipSuccess) return hip_fail(h, e, "ah_set_state copy");
        h->step = step;
        h->ready = true;
        return AH_OK;
    });
}

int ah_get_state(ah_handle* h, double* host_soa, int64_t* step)
{
    return no_throw([&]() -> int {
        if (!h || !host_soa) return fail(h, AH_E_INVAL, "ah_get_state: bad argument");
        if (!h->ready) return fail(h, AH_E_STATE, "ah_get_state before ah_init/ah_set_state");
        DeviceGuard g(h->device);
        hipError_t e = hipStreamSynchronize(h->stream);
        if (e != hipSuccess) return hip_fail(h, e, "ah_get_state sync");
        IoStage* st = nullptr;
        e = io_stage(h, 10 * (size_t)h->V * h->real_bytes, &st);
        const size_t fb = field_bytes(h->p);
        void *pp = h->pp[h->cur][0], *mom = h->mom[h->curm][0];
        if (e == hipSuccess)
            e = h->real_bytes == 8 ? state_download<double>(pp, mom, fb, host_soa, h->p.N, h->P, *st, h->stream)
                                   : state_download<float>(pp, mom, fb, host_soa, h->p.N, h->P, *st, h->stream);
        if (e != hipSuccess) return hip_fail(h, e, "ah_get_state copy");
        if (step) *step = h->step;
        return AH_OK;
    });
}

int ah_gather(ah_handle* h, const int64_t* sites, int64_t count, double* host_out)
{
    return no_throw([&]() -> int {
        if (!h || count < 0 || (count > 0 && (!sites || !host_out))) return fail(h, AH_E_INVAL, "ah_gather: bad argument");
        if (!h->ready) return fail(h, AH_E_STATE, "ah_gather before ah_init/ah_set_state");
        for (int64_t k = 0; k < count; ++k)
            if (sites[k] < 0 || sites[k] >= h->V) return fail(h, AH_E_INVAL, "ah_gather: site index out of range");
        if (count == 0) return AH_OK;
        DeviceGuard g(h->device);
        // through the staging memory, which the kernel reads the indices from
        // and writes the values to: in one piece if they fit, else in pieces,
        // so that the host packs and unpacks some while others are gathered
        // (MI355X, 1e5 sites of 8^3 FP64: 505 us, 595 one after the other)
        const size_t rb = h->real_bytes, each = sizeof(int64_t) + 10 * rb;
        IoStage* st = nullptr;
        hipError_t e = io_stage(h, (size_t)count * each, &st);
        void* dev = nullptr;
        if (e == hipSuccess) e = hipHostGetDevicePointer(&dev, st->host, 0);
        if (e != hipSuccess) return hip_fail(h, e, "ah_gather");
        auto fits = [&](size_t bytes) { return (int64_t)(bytes / each) / 32 * 32; };  // values start on a cache line
        const bool whole = count <= fits(st->bytes);
        const IoLane l{st->host, (char*)dev, whole ? st->bytes : st->bytes / kIoSlots / 256 * 256, st->ev};
        const int64_t per = fits(l.slot);
        const size_t off = per * sizeof(int64_t);
        e = pieces_out(
            l, 0, count, per, h->stream,
            [&](char* slot, int64_t k, int64_t n) {
                std::memcpy(l.host + (slot - l.dev), sites + k, n * sizeof(int64_t));
                const int64_t* in = (const int64_t*)slot;
                return rb == 8 ? launch_gather<double>(fields_of<double>(h, h->cur), in, n, h->p.N, h->P,
                                                       (double*)(slot + off), h->stream)
                               : launch_gather<float>(fields_of<float>(h, h->cur), in, n, h->p.N, h->P,
                                                      (float*)(slot + off), h->stream);
            },
            [&](const char* slot, int64_t k, int64_t n) {
                double* dst = host_out + 10 * k;
                if (rb == 8) {
                    std::memcpy(dst, slot + off, 10 * n * 8);
                } else {
                    const float* src = (const float*)(slot + off);
                    for (int64_t q = 0; q < 10 * n; ++q) dst[q] = (double)src[q];
                }
            });
        if (e != hipSuccess) {
            (void)hipStreamSynchronize(h->stream);  // nothing uses the staging memory once the call has failed
            return hip_fail(h, e, "ah_gather");
        }
        return AH_OK;
    });
}

int ah_gather_noalloc(ah_handle* h, const int64_t* sites, int64_t count, double* host_out)
{
    return no_throw([&]() -> int {
        if (!h || count < 0 || (count > 0 && (!sites || !host_out)))
            return fail(h, AH_E_INVAL, "ah_gather_noalloc: bad argument");
        if (count > kGatherMax)
            return fail(h, AH_E_INVAL, "ah_gather_noalloc: more than 65536 sites in one call");
        if (!h->ready) return fail(h, AH_E_STATE, "ah_gather_noalloc before ah_init/ah_set_state");
        for (int64_t k = 0; k < count; ++k)
            if (sites[k] < 0 || sites[k] >= h->V)
                return fail(h, AH_E_INVAL, "ah_gather_noalloc: site index out of range");
        if (count == 0) return AH_OK;
        DeviceGuard g(h->device);
        void* base = nullptr;
        hipError_t e = scratch_ptr(h->device, &base);
        if (e != hipSuccess) return hip_fail(h, e, "ah_gather_noalloc: scratch lookup");
        // scratch layout: kGatherMax site indices, then the gathered values
        int64_t* d_sites = (int64_t*)base;
        void* d_out = (char*)base + (size_t)kGatherMax * sizeof(int64_t);
        const size_t rb = h->real_bytes;
        e = hipMemcpyAsync(d_sites, sites, count * sizeof(int64_t), hipMemcpyHostToDevice, h->stream);
        if (e == hipSuccess)
            e = rb == 8 ? launch_gather<double>(fields_of<double>(h, h->cur), d_sites, count, h->p.N, h->P, (double*)d_out,
                                                h->stream)
                        : launch_gather<float>(fields_of<float>(h, h->cur), d_sites, count, h->p.N, h->P, (float*)d_out,
                                               h->stream);
        // FP32 values land in the first half of host_out and are widened in
        // place, last first, so no host staging buffer is needed either
        if (e == hipSuccess)
            e = hipMemcpyAsync(host_out, d_out, count * 10 * rb, hipMemcpyDeviceToHost, h->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
        if (e != hipSuccess) return hip_fail(h, e, "ah_gather_noalloc");
        if (rb == 4) {
            const float* src = (const float*)host_out;
            for (int64_t q = count * 10 - 1; q >= 0; --q) host_out[q] = (double)src[q];
        }
        return AH_OK;
    });
}

int ah_get_step(const ah_handle* h, int64_t* step)
{
    if (!h || !step) return AH_E_INVAL;
    *step = h->step;
    return AH_OK;
}

int ah_step(ah_handle* h, int64_t nsteps)
{
    return no_throw([&]() -> int {
        if (!h || nsteps < 0) return fail(h, AH_E_INVAL, "ah_step: bad argument");
        if (!h->ready) return fail(h, AH_E_STATE, "ah_step before ah_init/ah_set_state");
        DeviceGuard g(h->device);
        const hipError_t e = plain_steps(h, nsteps);
        if (e != hipSuccess) return hip_fail(h, e, "ah_step launch");
        return AH_OK;
    });
}

int ah_step_measured(ah_handle* h, int64_t nsteps, int32_t measure_every, ah_measurement* series, int32_t cap,
                     int32_t* n)
{
    return no_throw([&]() -> int {
        if (!h || nsteps < 0 || measure_every <= 0 || !n || (cap > 0 && !series))
            return fail(h, AH_E_INVAL, "ah_step_measured: bad argument");
        if (!h->ready) return fail(h, AH_E_STATE, "ah_step_measured before ah_init/ah_set_state");
        if (h->p.gauge_action != AH_COMPACT)
            return fail(h, AH_E_INVAL, "ah_step_measured: fused diagnostics need the compact action");
        int64_t due = 0;
        for (int64_t k = 0; k < nsteps; ++k)
            if ((h->step + k) % measure_every == 0) ++due;
        if (due > cap) return fail(h, AH_E_INVAL, "ah_step_measured: more due snapshots than cap");
        DeviceGuard g(h->device);
        int32_t written = 0;
        std::vector<int64_t> steps;
        auto flush = [&]() -> hipError_t {
            if (steps.empty()) return hipSuccess;
            hipError_t e = hipStreamSynchronize(h->stream);
            if (e != hipSuccess) return e;
            for (size_t j = 0; j < steps.size(); ++j)
                to_measurement(h->p, steps[j], h->host_series + j * kMeasStride, h->V, &series[written++]);
            steps.clear();
            return hipSuccess;
        };
        const int64_t end = h->step + nsteps;
        while (h->step < end) {
            hipError_t e;
            if (h->step % measure_every == 0) {
                if ((int)steps.size() == kSeriesCap) {
                    e = flush();
                    if (e != hipSuccess) return hip_fail(h, e, "ah_step_measured sync");
                }
                steps.push_back(h->step);
                double* dst = h->series + (steps.size() - 1) * kMeasStride;
                e = h->p.precision == AH_FP64 ? measured_pass<double>(h, dst, true) : measured_pass<float>(h, dst, true);
            } else {
                // the plain steps up to the next due snapshot (or the end)
                const int64_t next = (h->step / measure_every + 1) * measure_every;
                e = plain_steps(h, (next < end ? next : end) - h->step);
            }
            if (e != hipSuccess) return hip_fail(h, e, "ah_step_measured launch");
        }
        hipError_t e = flush();
        if (e != hipSuccess) return hip_fail(h, e, "ah_step_measured sync");
        *n = written;
        return AH_OK;
    });
}

int ah_get_timing_split(ah_handle* h, double* measured_ms, int64_t* measured_launches)
{
    return no_throw([&]() -> int {
        if (!h || !measured_ms || !measured_launches) return fail(h, AH_E_INVAL, "ah_get_timing_split: bad argument");
        DeviceGuard g(h->device);
        hipError_t e = hipStreamSynchronize(h->stream);
        if (e != hipSuccess) return hip_fail(h, e, "ah_get_timing_split sync");
        double tot = 0.0;
        for (size_t k = 0; k + 1 < h->ev_used; k += 2) {
            if (!h->ev_measured[k / 2]) continue;
            float ms = 0.0f;
            e = hipEventElapsedTime(&ms, h->ev[k], h->ev[k + 1]);
            if (e != hipSuccess) return hip_fail(h, e, "ah_get_timing_split elapsed");
            tot += ms;
        }
        *measured_ms = tot;
        *measured_launches = h->measured_launches;
        return AH_OK;
    });
}

int ah_measure(ah_handle* h, ah_measurement* out)
{
    return no_throw([&]() -> int {
        if (!h || !out) return fail(h, AH_E_INVAL, "ah_measure: bad argument");
        if (!h->ready) return fail(h, AH_E_STATE, "ah_measure before ah_init/ah_set_state");
        DeviceGuard g(h->device);
        const ah_params& p = h->p;
        hipError_t e;
        if (p.gauge_action == AH_COMPACT) {
            e = p.precision == AH_FP64 ? measured_pass<double>(h, h->series, false)
                                       : measured_pass<float>(h, h->series, false);
        } else {
            const StepCoef c = coef_at(p, h->step);
            const MeasConst mc = meas_const(p, h->step);
            e = p.precision == AH_FP64 ? launch_measure<double>(fields_of<double>(h, h->cur), lconst(p), c, mc,
                                                                h->partials, h->series, h->stream)
                                       : launch_measure<float>(fields_of<float>(h, h->cur), lconst(p), c, mc,
                                                               h->partials, h->series, h->stream);
        }
        if (e != hipSuccess) return hip_fail(h, e, "ah_measure launch");
        e = hipStreamSynchronize(h->stream);
        if (e != hipSuccess) return hip_fail(h, e, "ah_measure sync");
        to_measurement(p, h->step, h->host_series, h->V, out);
        return AH_OK;
    });
}

int ah_get_winding(ah_handle* h, int8_t* host_w)
{
    return no_throw([&]() -> int {
        if (!h || !host_w) return fail(h, AH_E_INVAL, "ah_get_winding: bad argument");
        if (!h->ready) return fail(h, AH_E_STATE, "ah_get_winding before ah_init/ah_set_state");
        DeviceGuard g(h->device);
        // the Pi and E buffers that no snapshot is in hold them (3 bytes a
        // site of their 20 or 40): the next step writes those anew
        int8_t* d = (int8_t*)h->mom[h->curm ^ 1][0];
        const size_t bytes = 3 * (size_t)h->V;
        hipError_t e = hipStreamSynchronize(h->stream);
        if (e == hipSuccess)
            e = h->p.precision == AH_FP64 ? launch_winding<double>(fields_of<double>(h, h->cur), lconst(h->p), d, h->stream)
                                          : launch_winding<float>(fields_of<float>(h, h->cur), lconst(h->p), d, h->stream);
        IoStage* st = nullptr;
        if (e == hipSuccess) e = io_stage(h, bytes, &st);
        if (e == hipSuccess) e = bytes_download(d, host_w, bytes, *st, h->stream);
        if (e != hipSuccess) return hip_fail(h, e, "ah_get_winding");
        return AH_OK;
    });
}

int ah_synchronize(ah_handle* h)
{
    return no_throw([&]() -> int {
        if (!h) return AH_E_INVAL;
        DeviceGuard g(h->device);
        hipError_t e = hipStreamSynchronize(h->stream);
        if (e != hipSuccess) return hip_fail(h, e, "ah_synchronize");
        return AH_OK;
    });
}

int ah_set_timing(ah_handle* h, int enable)
{
    return no_throw([&]() -> int {
        if (!h) return AH_E_INVAL;
        h->timing = enable != 0;
        h->ev_used = 0;
        h->measured_launches = 0;
        h->ev_measured.clear();
        h->ev_steps.clear();
        return AH_OK;
    });
}

int ah_get_timing(ah_handle* h, double* total_ms, int64_t* launches)
{
    return no_throw([&]() -> int {
        if (!h || !total_ms || !launches) return fail(h, AH_E_INVAL, "ah_get_timing: bad argument");
        DeviceGuard g(h->device);
        hipError_t e = hipStreamSynchronize(h->stream);
        if (e != hipSuccess) return hip_fail(h, e, "ah_get_timing sync");
        double tot = 0.0;
        for (size_t k = 0; k + 1 < h->ev_used; k += 2) {
            float ms = 0.0f;
            e = hipEventElapsedTime(&ms, h->ev[k], h->ev[k + 1]);
            if (e != hipSuccess) return hip_fail(h, e, "ah_get_timing elapsed");
            tot += ms;
        }
        int64_t steps = 0;
        for (size_t k = 0; k < h->ev_used / 2; ++k) steps += h->ev_steps[k];
        *total_ms = tot;
        *launches = steps;
        return AH_OK;
    });
}

int ah_destroy(ah_handle* h)
{
    if (!h) return AH_E_INVAL;
    DeviceGuard g(h->device);
    (void)hipStreamSynchronize(h->stream);
    for (hipEvent_t ev : h->ev) (void)hipEventDestroy(ev);
    io_close(&h->io);
    if (h->io_mem) (void)hipHostFree(h->io_mem);
    if (h->host_series) (void)hipHostFree(h->host_series);
    if (h->owns_arena && h->arena) (void)hipFree(h->arena);
    delete h;
    return AH_OK;
}

const char* ah_strerror(int code)
{
    switch (code) {
    case AH_OK: return "ok";
    case AH_E_INVAL: return "invalid argument";
    case AH_E_NOMEM: return "out of device memory or arena too small";
    case AH_E_DEVICE: return "HIP device error";
    case AH_E_STATE: return "call out of order";
    case AH_E_AGAIN: return "resource busy; retry later";
    default: return "unknown error";
    }
}

const char* ah_last_error(const ah_handle* h)
{
    if (!h) return "";
    return h->err.c_str();
}

}  // extern "C"
