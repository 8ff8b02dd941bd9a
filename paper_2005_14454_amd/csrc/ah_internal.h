// Internal declarations shared by the host runtime and the HIP kernels of libah.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "ah.h"

namespace ah {

// Runs the body of a C-ABI entry point: an exception from the host containers
// it uses (host memory exhausted, a size past what a container can hold)
// becomes AH_E_NOMEM instead of crossing the ABI.
template <typename F>
inline int no_throw(F&& body) noexcept
{
    try {
        return body();
    } catch (...) {
        return AH_E_NOMEM;
    }
}

// Structure-of-arrays field pointers of one lattice snapshot.  phi and A come
// from the current ping-pong buffer, Pi and E are single buffers updated in
// place; the drift writes phi and A into the other ping-pong buffer.
template <typename R>
struct Fields {
    R* phr;
    R* phi;
    R* pir;
    R* pii;
    R* a0;
    R* a1;
    R* a2;
    R* e0;
    R* e1;
    R* e2;
};

// The same fields as the marches take them: phi_re, phi_im, A0, A1, A2 and
// Pi_re, Pi_im, E0, E1, E2 of the snapshot read and of the one written, each
// five in one block with `fs` values from field to field, as every arena lays
// them out.  Four pointers and a stride stay in a kernel's scalar registers
// where twenty pointers spill.
template <typename R>
struct Blocks {
    const R *ip, *im;
    R *op, *om;
    int64_t fs;
};
// The ten fields of two blocks with stride fs (in bytes).
template <typename R>
inline Fields<R> fields_at(void* pp, void* mom, size_t fs)
{
    char *p = (char*)pp, *m = (char*)mom;
    return Fields<R>{(R*)p,            (R*)(p + fs),     (R*)m,            (R*)(m + fs),     (R*)(p + 2 * fs),
                     (R*)(p + 3 * fs), (R*)(p + 4 * fs), (R*)(m + 2 * fs), (R*)(m + 3 * fs), (R*)(m + 4 * fs)};
}
// The blocks of a snapshot read and one written; false if the fields are not
// so laid out.
template <typename R>
inline bool blocks_of(const Fields<R>& in, const Fields<R>& out, Blocks<R>* b)
{
    const size_t fs = (size_t)((char*)in.phi - (char*)in.phr);
    for (const Fields<R>* f : {&in, &out}) {
        const Fields<R> g = fields_at<R>(f->phr, f->pir, fs);
        if (g.phi != f->phi || g.a0 != f->a0 || g.a1 != f->a1 || g.a2 != f->a2 || g.pii != f->pii || g.e0 != f->e0 ||
            g.e1 != f->e1 || g.e2 != f->e2)
            return false;
    }
    *b = Blocks<R>{in.phr, in.pir, out.phr, out.pir, (int64_t)(fs / sizeof(R))};
    return true;
}

// Per-step scalars of the update, formed on the host in FP64 and rounded to
// the storage type (kick: X^{n+1/2} = c1 X^{n-1/2} + c2 force).
struct StepCoef {
    double cP1, cP2;   // (1-delta)/(1+delta), deta/(1+delta)
    double cE1, cE2;   // (1-omega)/(1+omega), deta/(1+omega)
    double lam_half;   // lambda0 f / 2
    double kappa;      // 2 e0^2 f
};

// Stored layout of every field of a lattice: site (x, y, z) at element
// x + P (y + N z), with the row pitch P >= N a whole number of 128-byte cache
// lines.  Every row then starts on a line, and a tile's rows are read as
// whole lines whatever N is; the P - N elements that end a row are never
// read or written.
inline int row_pitch(int N, int precision)
{
    const int per_line = precision == AH_FP64 ? 16 : 32;
    return (N + per_line - 1) / per_line * per_line;
}

// Lattice-wide constants.
struct LatticeConst {
    int N;
    int P;  // row pitch (row_pitch(N, precision))
    int compact;
    double dx, deta, sigma2;
};

// Diagnostics reduction slots (FP64 sums over sites unless noted).  The
// Lagrangian sum is kin - grad - pot + el - mag of the first five, so it has
// no slot of its own.
enum MeasSlot {
    M_KIN = 0,   // |Pi_bar|^2
    M_GRAD,      // sum_i |D_i^+ phi|^2
    M_POT,       // lambda0 f/4 (|phi|^2 - sigma^2)^2
    M_EL,        // sum_i E_bar_i^2 / (2 e0^2 f)
    M_MAG,       // sum_{i<j} B_ij^2 / (2 e0^2 f)
    M_KINL,      // |Pi_bar|^2 L
    M_GRADL,     // sum_i |D_i^+ phi|^2 L
    M_PL,        // p L, with the pressure p = kin - grad/3 - pot + (el + mag)/3
    M_RHOL,      // rho L, with the energy density rho = kin + grad + pot + el + mag
    M_G2,        // G^2
    M_DIV2,      // (div E)^2
    M_CRHO2,     // (c rho)^2
    M_GMAX,      // max |G|   (max-reduced)
    M_WABS,      // sum_{i<j} |W_ij|  (exact integer in FP64)
    M_NONFIN,    // count of sites with a non-finite value
    M_COUNT
};
constexpr int kMarchSums = M_RHOL + 1;  // FP64 sums the measured march forms: slots 0 .. M_RHOL
constexpr int kMeasStride = 16;        // doubles per partial record
static_assert(M_COUNT <= kMeasStride, "a record holds every slot");
constexpr int kMeasBlocks = 2048;      // fixed grid of the measurement kernel
constexpr int kMeasThreads = 256;

struct MeasConst {
    double inv_2e2f;   // 1 / (2 e0^2 f)
    double lam_quarter;// lambda0 f / 4
    double gauss_c;    // coupling of the Gauss residual
};

// Tiled step kernel shape: TX x TY sites per workgroup, zchunk x2-planes per
// workgroup (0 = the whole lattice).
struct TileConfig {
    int tx, ty, zchunk;
};

// Tile shapes the tiled kernels are built for (the 1024-thread ones for FP32 only).
inline bool tile_supported(int precision, int tx, int ty)
{
    if (tx == 64 && (ty == 8 || ty == 4)) return true;
    if (tx == 32 && ty == 8) return true;
    if (tx == 128 && ty == 4) return true;
    if ((tx == 64 && ty == 16) || (tx == 128 && ty == 8)) return precision == AH_FP32;
    return false;
}

// Tile shapes of the two-step pass (its LDS holds two regions of links per
// workgroup, so the FP64 shapes are the smaller ones).
inline bool tile2_supported(int precision, int tx, int ty)
{
    if ((tx == 32 && ty == 8) || (tx == 64 && ty == 4)) return true;
    return tx == 64 && ty == 8 && precision == AH_FP32;
}

// Tile shapes of the pool's batched plain step (its measured step runs the
// measured march's shape, measured_tile).
inline bool batch_tile_supported(int precision, int tx, int ty)
{
    if ((tx == 64 && (ty == 8 || ty == 4)) || (tx == 32 && ty == 8)) return true;
    return precision == AH_FP32 && tx == 128 && (ty == 4 || ty == 8);
}

// Default one-step tile shape for side N; false if none applies.
bool default_tile(int precision, int N, int* tx, int* ty);
// Workgroups of a tiled launch one CU holds at once (measured: the march
// that also forms the diagnostics).
int resident_per_cu(int kernel, int precision, int tx, int ty, bool measured);
// Automatic z-chunk of a tiled launch.
int auto_zchunk(int kernel, int precision, int N, int tx, int ty, bool measured);
int start_planes(int kernel, int tx, int ty);
// Whether two-step passes are the faster way to take two plain steps of a
// lattice without a tuning entry, alone or in a pool: FP32 at every size, FP64
// from N = 65 on (MI355X, us per step, two-step / single: FP32 24^3 4.9 / 5.6,
// 48^3 5.8 / 6.2, 64^3 6.7 / 7.0, 192^3 78 / 116, 512^3 1283 / 1998; FP64 32^3
// 9.5 / 8.7, 64^3 13.2 / 12.0: its pass's longer start is not paid for by two
// planes a chunk; 75^3 25.8 / 27.2, 512^3 3610 / 4490).
inline bool two_step_pays(int precision, int N) { return precision == AH_FP32 || N > 64; }
// Tiling of the two-step passes of an automatic configuration (zchunk 0: none).
TileConfig default_two(int precision, int N);
// Tiling of the measured march of a lattice stepped with cfg (resolved).
TileConfig measured_tiling(const ah_params& p, const ah_step_config& cfg);

// Smallest z-chunk the tiled kernels accept for a lattice of side N.  Short
// chunks pay for themselves only on small lattices, which they give enough
// workgroups (64^3 FP32 on MI355X: 2-plane chunks step in 11.4 us, 8-plane
// ones in 22 us); larger lattices keep at least 8 planes, which bounds the
// diagnostics records a handle holds.
inline int min_zchunk(int N) { return N <= 128 ? 2 : 8; }

// Tile shape for the measured march of a lattice stepped on (tx, ty): 32 x 8.
// Its four waves leave room for two workgroups per CU, which fill the chip
// more evenly than one of eight waves (FP32 on MI355X, us per measured step
// on 32 x 8 / 64 x 8: 512^3 3645 / 3659, 337^3 1143 / 1649, 200^3 285 / 293),
// and the FP64 march would spill on larger ones.  Returns whether it changed.
inline bool measured_tile(int* tx, int* ty)
{
    const bool changed = *tx != 32 || *ty != 8;
    *tx = 32;
    *ty = 8;
    return changed;
}

// ---- lattice pool (many independent lattices advanced by one launch) ------
// Row layout of a lattice's per-step FP64 coefficient table.
enum CoefSlot { C_P1 = 0, C_P2, C_E1, C_E2, C_LAMH, C_KAPPA, C_INV2E2F, C_LAMQ, C_GAUSS, kCoefStride = 10 };

// Device-resident descriptor of one pool lattice (plain data; uploaded by the host).
struct PoolLattice {
    void* pp[2];           // ping-pong blocks of phi_re, phi_im, A0, A1, A2; counter[2] names the current one
    void* mom[2];          // blocks of Pi_re, Pi_im, E0, E1, E2; counter[3] names the current one (updated in place
                           // by a plain single step; a two-step pass and a measured step write the other)
    int64_t fs;            // values from one field of a block to the next
    const double* coef;    // (nsteps + 1) rows of kCoefStride doubles
    int64_t* counter;      // kCounterWords words: local step k, measurements taken, phi/A buffer, Pi/E buffer
    double* partials;      // diagnostics records of this lattice
    double* series;        // measurement records: kSeriesStride doubles each
    int64_t nsteps;        // steps to run; the lattice is finished when counter[0] == nsteps + 1
    int64_t series_cap;
    int N, tiles_x, tiles_y, zchunk;     // step tiling
    int meas_zchunk, meas_blocks, measure_every, precision;
    int P;                   // row pitch
    int mtiles_x, mtiles_y;  // tiling of the measured step (measured_tile), z-chunks of meas_zchunk
    int two_tiles_x, two_tiles_y, two_zchunk;  // tiling of the two-step pass; two_zchunk == 0: none
    int compact;
    double dx, deta, sigma2;
};

// Whether pool lattice L forms the diagnostics of its snapshot k (every
// measure_every-th and the last), and whether its step k is a two-step pass:
// it has a two-step tiling, neither k nor k+1 is due and both steps remain.
__host__ __device__ inline bool measure_due(const PoolLattice& L, int64_t k)
{
    if (k > L.nsteps) return false;
    if (k == L.nsteps) return true;
    return L.measure_every > 0 && (k % L.measure_every) == 0;
}
__host__ __device__ inline bool two_step_due(const PoolLattice& L, int64_t k)
{
    return L.two_zchunk > 0 && k + 1 < L.nsteps && !measure_due(L, k) && !measure_due(L, k + 1);
}
struct WorkItem {
    int lattice, tile;  // lattice < 0: an empty item (padding)
};
constexpr int kXcdCount = 8;           // XCDs of the device; block b runs on XCD b % 8
constexpr int kCounterWords = 4;       // int64 words of a pool lattice's counter
constexpr int kSeriesStride = 18;      // M_COUNT sums + step index + pad
static_assert(M_COUNT + 1 <= kSeriesStride, "a series record holds the sums and the step index");

// ---- fixed device scratch (ah_scratch.hip) ---------------------------------
// Sites one ah_gather_noalloc call may ask for, and the scratch that holds
// their indices and their FP64-sized values.
constexpr int64_t kGatherMax = 65536;
constexpr size_t kScratchBytes = (size_t)kGatherMax * sizeof(int64_t) + (size_t)kGatherMax * 10 * sizeof(double);
// Device address of `device`'s copy of the scratch (looked up on the first
// call for that device, with it current).
hipError_t scratch_ptr(int device, void** out);

// Pinned host memory that a snapshot passes through on its way between the
// fields and a caller's array: kIoSlots slots for each host thread that works
// on it, and an event for every slot.  At most kIoBytes: allocating it takes
// 0.25 ms per MB, which the first call pays.
constexpr int kIoThreads = 4, kIoSlots = 3;
constexpr size_t kIoBytes = 4u << 20;
struct IoStage {
    char* host = nullptr;
    size_t bytes = 0;
    hipEvent_t ev[kIoThreads * kIoSlots] = {};
};
hipError_t io_events(IoStage* st);   // creates those that are missing
void io_close(IoStage* st);          // destroys them
// A dense FP64 SoA state (state order, x fastest) into the fields at (pp, mom)
// (as fields_at takes them), and back; both return when it is done
// (ah_runtime.cpp).
template <typename R>
hipError_t state_upload(void* pp, void* mom, size_t fs, const double* host, int N, int P, const IoStage& st,
                        hipStream_t s);
template <typename R>
hipError_t state_download(void* pp, void* mom, size_t fs, double* host, int N, int P, const IoStage& st,
                          hipStream_t s);
// Device bytes (16-byte aligned) to the host in the same way.
hipError_t bytes_download(const void* dev, void* host, size_t bytes, const IoStage& st, hipStream_t s);

// ---- launchers (ah_kernels.hip, ah_step_tile.hip) -------------------------
template <typename R>
hipError_t launch_init(const Fields<R>& f, int N, int P, double sigma, uint64_t seed, hipStream_t s);

template <typename R>
hipError_t launch_step(const Fields<R>& in, R* ophr, R* ophi, R* oa0, R* oa1, R* oa2,
                       const LatticeConst& L, const StepCoef& c, hipStream_t s);

// Tiled step from `in` to `out`: phi and A into out's (other) buffers, Pi
// and E into out's, which may be in's (an update in place).  With mc !=
// nullptr also the diagnostics of the snapshot read, Gauss residual included
// (one record per workgroup into partials, in tile order); a measured step
// then needs Pi and E out of place (else hipErrorInvalidValue).  write =
// false leaves the fields untouched (diagnostics only).
template <typename R>
hipError_t launch_step_tile(const Fields<R>& in, const Fields<R>& out, const LatticeConst& L, const StepCoef& c,
                            const TileConfig& tc, const MeasConst* mc, double* partials, bool write, hipStream_t s);

// Two steps in one pass: snapshot n of `in` to snapshot n+2 of `out` (all
// ten fields in other buffers), with the coefficients of steps n and n+1.
template <typename R>
hipError_t launch_step2_tile(const Fields<R>& in, const Fields<R>& out, const LatticeConst& L, const StepCoef& c0,
                             const StepCoef& c1, const TileConfig& tc, hipStream_t s);

// workgroups (= diagnostics records) of one tiled launch
int step_tile_blocks(int N, const TileConfig& tc);


template <typename R>
hipError_t launch_step_batch(const PoolLattice* lat, const WorkItem* work, int nwork, int tx, int ty, int grid,
                             bool measured, hipStream_t s);
// the pool's two-step pass (ah_step2.hip): lattices whose step k takes one
template <typename R>
hipError_t launch_step2_batch(const PoolLattice* lat, const WorkItem* work, int nwork, int tx, int ty, int grid,
                              hipStream_t s);

template <typename R>
hipError_t launch_measure(const Fields<R>& f, const LatticeConst& L, const StepCoef& c,
                          const MeasConst& mc, double* partials, double* result, hipStream_t s);

// second-stage fold of nblocks per-workgroup records into result[M_COUNT]
hipError_t launch_measure_final(const double* partials, int nblocks, double* result, hipStream_t s);

hipError_t launch_fold_batch(const PoolLattice* lat, int nlat, hipStream_t s);
hipError_t launch_advance_batch(const PoolLattice* lat, int nlat, hipStream_t s);

template <typename R>
hipError_t launch_gather(const Fields<R>& f, const int64_t* sites, int64_t count, int N, int P, R* out, hipStream_t s);

// Rows row0 .. row0 + nrows - 1 of a state's 10 N^2 (component, then x2, then
// x1) between the fields at (pp, mom) and a dense buffer: out of the fields
// (pack) or into them.  `rows` may be pinned host memory.
template <typename R>
hipError_t launch_state_rows(void* pp, void* mom, size_t fs, int N, int P, int64_t row0, int64_t nrows, R* rows, bool pack,
                             hipStream_t s);

// n bytes from src to dst (pinned host memory).
hipError_t launch_bytes(const void* src, void* dst, int64_t n, hipStream_t s);

template <typename R>
hipError_t launch_winding(const Fields<R>& f, const LatticeConst& L, int8_t* w, hipStream_t s);

}  // namespace ah
