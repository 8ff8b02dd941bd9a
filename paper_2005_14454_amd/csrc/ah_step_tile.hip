// Tiled, z-marching leapfrog step and diagnostics for gfx950 (compact gauge
// action), for one lattice and for a pool of lattices.
//
// One workgroup owns a TX x TY tile of the (x0, x1) plane and a chunk of
// x2-planes ("z").  It walks the chunk in phases of one plane and one barrier:
// phase z turns A of plane z+2 (the tile plus a one-site halo ring, loaded
// during the phase before) into link variables U_j = exp(-i dx A_j), one sincos
// per link, shared by all users through LDS, and updates the own sites of
// plane z:
//   - covariant Laplacian and current from U and phi (section 2);
//   - lattice curl from plaquettes formed as products of four links,
//     F_ij = -Im(U_i^x U_j^{x+i} conj(U_i^{x+j}) conj(U_j^x)) / dx^2, which
//     equals sin(Theta_ij)/dx^2 for the compact action;
//   - Crank-Nicolson kick of Pi and E in place, drift of phi and A into the
//     other ping-pong buffer.
// Every site reads its 10 state values and writes 10 values once per step;
// the halo re-reads hit L2.  Own-column quantities of the planes below and
// above (phi, U_z, F_xz, F_yz) are carried in registers.  Workgroups are
// placed so that each XCD gets a contiguous band of tiles, which keeps halo
// reads inside one L2.
//
// What bounds it: memory for the plain march of a large lattice (512^3 on
// MI355X: FP32 128 x 4 2.00 ms a step, 5.4 TB/s of algorithmic bytes; FP64
// 64 x 8 4.49 ms, 4.8 TB/s; a copy reaches 5.5 TB/s); the latency of a chunk's
// first loads and barriers for a small one (64^3 FP64, 2-plane chunks: 12.0
// us); instruction issue and latency for the measured march (512^3: FP32 3.5
// ms, FP64 6.0 ms).  Links in three slots, so that one barrier a plane is
// enough, and every load of a chunk's start issued before its first barrier
// took the measured march from 3.74 and 7.3 ms and the 64^3 step from 16.4 us
// (two barriers a plane, three rounds of loads at the start of a chunk).
//
// Floating-point contraction is off in this file and every fused multiply-add
// is written out, so each site is computed by the same sequence of roundings
// whatever the tile shape, z-chunk or template instance: results are
// bitwise reproducible across launch configurations.
#include "ah_device.h"
#include "ah_internal.h"
#include "ah_stencil.h"

#pragma clang fp contract(off)

namespace ah {
namespace {


template <typename R, int TX, int TY>
struct TileGeom {
    static constexpr int RW = TX + 2;             // region width (tile + halo)
    static constexpr int RH = TY + 2;             // region height
    static constexpr int RS = RW * RH;            // region sites
    static constexpr int NT = TX * TY;            // threads
    static constexpr int H = 2 * RW + 2 * TY;     // halo ring sites
    static constexpr int HPT = (H + NT - 1) / NT; // halo sites per thread (upper bound)
};

// Per-launch constants of one lattice step (coefficients rounded to R).
template <typename R>
struct StepArgs {
    // phi and A go to other buffers; Pi and E may be written in place, but not
    // by the measured march
    Blocks<R> b;
    int N, P;  // side, row pitch: site (x, y, z) at x + P (y + N z)
    R dx, sigma2, cP1, cP2, cE1, cE2, lamh, kappa, deta;
};

// Constants of the diagnostics of the snapshot a measured march reads.
struct MeasArgs {
    double dx;          // lattice spacing (FP64, for plaquette angles and links)
    double inv_2e2f;    // 1 / (2 e0^2 f)
    double lam_quarter; // lambda0 f / 4
    double gauss_c;     // coupling of the Gauss residual
};

template <typename R, int TX, int TY>
struct TileShared {
    static constexpr int RS = TileGeom<R, TX, TY>::RS;
    // x and y links of planes z and z+1, which the update of plane z reads,
    // and of plane z+2, which the same phase writes; z links and phi of planes
    // z (read) and z+1 (written)
    Pair<R, RS> U[3], W[2];
};

template <typename R, int TX, int TY>
struct MeasShared {
    static constexpr int RS = (TX + 2) * (TY + 2);
    R A[2][3][RS];      // stored A of planes z (read) and z+1 (written)
    float Y[2][3][RS];  // link phases of planes z (written) and z-1 (read)
    // FP32 lattices: E_x, E_y of planes z (read) and z+1 (written; own sites,
    // and the -x / -y halo) for the Gauss residual
    R E[2][2][sizeof(R) == 4 ? RS : 1];
    double red[TX * TY / 64][M_COUNT];  // block reduction
};

// FP64 link for the windings of FP32 lattices (the stored value, exactly widened)
__device__ inline Cx<double> link64(double dx, double a)
{
    double s, c;
    sincos(dx * a, &s, &c);
    return {c, -s};
}

// atan2(y, x) in FP32 to within 1e-6 rad for max(|x|, |y|) in [1e-30, 1e30]:
// reduction to t = min(|x|, |y|) / max(|x|, |y|) in [0, 1], atan(t) ~ t P(t^2)
// with P of degree 6 fitted by weighted least squares on Chebyshev nodes
// (largest error 3.3e-7 in FP32 over [0, 1]), then the octant and the sign.
// Only the angle of a branch the caller has already made safe is taken from
// it; the cut itself is decided in FP64.
__device__ inline float atan2_fast(float y, float x)
{
    const float ax = fabsf(x), ay = fabsf(y);
    const float t = fminf(ax, ay) * __builtin_amdgcn_rcpf(fmaxf(ax, ay));
    const float s = t * t;
    float p = 0.00681175384670496f;
    p = fm(p, s, -0.033604107797145844f);
    p = fm(p, s, 0.07962355017662048f);
    p = fm(p, s, -0.13233335316181183f);
    p = fm(p, s, 0.19807814061641693f);
    p = fm(p, s, -0.3331736922264099f);
    p = fm(p, s, 0.9999961256980896f);
    float a = p * t;
    if (ay > ax) a = 1.57079632679489662f - a;
    if (x < 0.f) a = 3.14159265358979324f - a;
    return copysignf(a, y);
}

// Link phase arg(conj(phi^x) U phi^{x+j}) in (-pi, pi].  z is formed in FP64
// with plain products and sums; its sign decides the branch exactly as an
// FP64 atan2 would (-0 -> +0; atan2_fast keeps the sign of its first
// argument), and the angle itself is evaluated in FP32 on the exactly
// rescaled z: the windings only need it to well below pi.
__device__ inline float link_phase(double pr, double pim, Cx<double> U, double vr, double vi)
{
    const double wr = U.r * vr - U.i * vi;
    const double wi = U.r * vi + U.i * vr;
    const double zr = pr * wr + pim * wi;
    double zi = pr * wi - pim * wr;
    zi = (zi == 0.0) ? 0.0 : zi;
    const double mz = fmax(fabs(zr), fabs(zi));
    const int e = ilogb(mz);
    const float y = atan2_fast((float)ldexp(zi, -e), (float)ldexp(zr, -e));
    return mz == 0.0 ? (signbit(zr) ? 3.14159265358979f : 0.0f) : y;
}

// The FP64 evaluation for an FP32 lattice's link near the cut.  It runs for a
// few links in a million, so it is kept out of line: inlined, its FP64 sincos
// raises the register count of the whole measured march.
__device__ __attribute__((noinline)) float link_phase_near_cut(Cx<float> ph, Cx<float> pn, float a, double dx)
{
    return link_phase((double)ph.r, (double)ph.i, link64(dx, (double)a), (double)pn.r, (double)pn.i);
}

// Link phase of an FP32 lattice from z = conj(ph) (U pn), formed in FP32 from
// the link the step itself uses; its angle, taken in FP32, is within
//   |dx A| 2^-22 (rounding of dx A, in the link's phase)
//   + 1e-5        (the link's sine and cosine, within 3e-7; the two complex
//                  products; atan2_fast)
// of the FP64 value, so unless it lies that close to the cut at +-pi it is on
// the same side of it.  Near the cut, where |z| leaves the range in which
// FP32 keeps its relative precision (or is not finite), and where |dx A|
// exceeds 1e5 (so that four phases stay well within pi of the FP64 sum), the
// FP64 evaluation above decides from the stored A.
//
// The K phases of a site are taken side by side, with one test for all of
// them: a branch apiece would leave a chain of some forty dependent
// instructions at a time in flight, at two waves per SIMD.
template <int K>
__device__ inline void link_phases_f(const Cx<float> (&z)[K], Cx<float> ph, const Cx<float> (&pn)[K],
                                     const float (&a)[K], double dx, float (&y)[K])
{
    bool ok[K], all = true;
    for (int d = 0; d < K; ++d) {
        const float mz = fmaxf(fabsf(z[d].r), fabsf(z[d].i));
        const float dxa = fabsf((float)dx * a[d]);
        y[d] = atan2_fast(z[d].i, z[d].r);
        ok[d] = mz > 1e-30f && mz < 1e30f && dxa < 1e5f && 3.14159265f - fabsf(y[d]) > 1e-5f + 2.4e-7f * dxa;
        all = all && ok[d];
    }
    if (!all)
        for (int d = 0; d < K; ++d)
            if (!ok[d]) y[d] = link_phase_near_cut(ph, pn[d], a[d], dx);
}

// The multiple of 2 pi that wraps a plaquette angle to (-pi, pi]: the nearest
// one that the division th / 2 pi rounds to (a product with 1 / 2 pi gives the
// same multiple unless the quotient is close to a half turn, where the
// division itself is taken).
__device__ inline double turns_of(double th)
{
    const double two_pi = 6.283185307179586;
    const double q = th * (1.0 / two_pi);
    const double r = rint(q);
    return fabs(q - r) < 0.49 && fabs(q) < 1e12 ? r : rint(th / two_pi);
}

// Angles dx (((a + b) - c) - d) of a site's plaquettes, in FP64 from the stored
// A of either precision.  FP32 lattices could take most of them in FP32 (MI355X,
// measured step of 512^3 3.38 ms rather than 3.46), at fewer bits than the
// diagnostics promise.
template <typename R>
__device__ inline void plaq_angles(double dx, const R (&q)[3][4], double (&th)[3])
{
    for (int k = 0; k < 3; ++k)
        th[k] = dx * ((((double)q[k][0] + (double)q[k][1]) - (double)q[k][2]) - (double)q[k][3]);
}

// Winding of a plaquette from its four link phases and its angle (FP64): their
// sum, once the angle is wrapped, is within 4e-5 + 1e-6 |dx A| of a multiple of
// 2 pi (four phases, link_phases_f; |dx A| up to 1e5 in FP32, FP64 beyond).
__device__ inline int winding_of(float y1, float y2, float y3, float y4, double th)
{
    const double two_pi = 6.283185307179586;
    const double thw = th - two_pi * turns_of(th);
    const double sum = ((((double)y1 + (double)y2) - (double)y3) - (double)y4) + thw;
    return (int)rint(sum * (1.0 / two_pi));
}

// 1 - cos(Theta) of a plaquette from its four links, without cancellation
template <typename R>
__device__ inline R plaq_omc(Cx<R> ui_x, Cx<R> uj_xi, Cx<R> ui_xj, Cx<R> uj_x, R* sn)
{
    const Cx<R> p = cmul(ui_x, uj_xi);
    const Cx<R> q = cmul(ui_xj, uj_x);
    const R c = fm(p.r, q.r, p.i * q.i);
    const R s = fm(p.r, q.i, -(p.i * q.r));
    *sn = s;
    return c > R(0) ? (s * s) / (R(1) + c) : R(1) - c;
}

// v of the lane whose number differs in bit `off` (1, 2, 8: by DPP, without LDS)
template <int off>
__device__ inline double xor_lane(double v)
{
    if constexpr (off == 4) {
        return __shfl_xor(v, 4, 64);
    } else {
        constexpr int ctrl = off == 8 ? 0x128 : (off == 2 ? 0x4e : 0xb1);  // row_ror:8, quad_perm [2,3,0,1], [1,0,3,2]
        const int2 d = __builtin_bit_cast(int2, v);
        return __builtin_bit_cast(double, int2{__builtin_amdgcn_update_dpp(0, d.x, ctrl, 0xf, 0xf, true),
                                               __builtin_amdgcn_update_dpp(0, d.y, ctrl, 0xf, 0xf, true)});
    }
}
// Half-wave (off 32) or row (off 16) exchange: the lanes with that bit clear get
// a plus a's partner, the others b plus b's.
template <int off>
__device__ inline double swap_add(double a, double b)
{
    const uint2 x = __builtin_bit_cast(uint2, a), y = __builtin_bit_cast(uint2, b);
    using U = unsigned __attribute__((ext_vector_type(2)));
    U lo, hi;
    if constexpr (off == 32) {
        lo = __builtin_amdgcn_permlane32_swap(x.x, y.x, false, false);
        hi = __builtin_amdgcn_permlane32_swap(x.y, y.y, false, false);
    } else {
        lo = __builtin_amdgcn_permlane16_swap(x.x, y.x, false, false);
        hi = __builtin_amdgcn_permlane16_swap(x.y, y.y, false, false);
    }
    return __builtin_bit_cast(double, uint2{lo[0], hi[0]}) + __builtin_bit_cast(double, uint2{lo[1], hi[1]});
}
// Sums over the wave of 16 values; lane l returns that of value l / 4.  Each
// level halves the values a lane holds rather than summing all of them in
// every lane: 8 + 4 + 2 + 1 additions and two more, where 16 butterflies take
// 96 and, through LDS, 192 permutes, which on a short march are a tenth of
// its time (MI355X, 32^3 FP32: 15.0 us with the butterflies, 12.9 now; 64^3 FP64
// 25.3, 23.1).  Every sum goes through the lanes in the butterfly's order: 32,
// 16, 8, 4, 2, 1.
__device__ inline double wave_sums(const double (&v)[16])
{
    const int lane = threadIdx.x & 63;
    double a[8], b[4], c[2];
    for (int k = 0; k < 8; ++k) a[k] = swap_add<32>(v[k], v[k + 8]);
    for (int k = 0; k < 4; ++k) b[k] = swap_add<16>(a[k], a[k + 4]);
    const bool b8 = lane & 8, b4 = lane & 4;
    for (int k = 0; k < 2; ++k) c[k] = (b8 ? b[k + 2] : b[k]) + xor_lane<8>(b8 ? b[k] : b[k + 2]);
    double r = (b4 ? c[1] : c[0]) + xor_lane<4>(b4 ? c[0] : c[1]);
    r += xor_lane<2>(r);
    return r + xor_lane<1>(r);
}
__device__ inline double wave_max(double v)
{
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
    return v;
}

// Walk planes [z0, z1) of the tile whose lower corner is (x0, y0): kick and
// drift every own site (if `write`), and with MEAS also form the diagnostics of
// the snapshot being read (section 2 estimators, energy split, windings, the
// residual of the discrete Gauss law), writing the workgroup's fixed-order
// sums to `record`.  The Gauss residual
// reads E at the -x and -y neighbours, which a neighbouring workgroup of a
// pass that updated E in place could already have overwritten, so a measured
// march that steps writes Pi and E out of place (a.b.om).  E_z of the
// plane below is carried in a register; FP32 passes E_x and E_y of each plane
// through LDS, FP64 (whose LDS holds two workgroups per CU only without that
// exchange) loads the two neighbours with the plane's Pi and E.
// All threads of the workgroup call this with the same arguments; it
// synchronises the workgroup internally.
template <typename R, int TX, int TY, bool MEAS>
__device__ void march_step(TileShared<R, TX, TY>& sh, MeasShared<R, TX, TY>* mx, const StepArgs<R>& a,
                           const MeasArgs& ma, double* __restrict__ record, bool write, int x0, int y0, int z0,
                           int z1)
{
    using G = TileGeom<R, TX, TY>;
    constexpr int RW = G::RW, H = G::H, NT = G::NT;
    static_assert(G::HPT == 1, "halo must fit one extra site per thread");
    const int N = a.N;
    const R dx = a.dx, sigma2 = a.sigma2, cP1 = a.cP1, cP2 = a.cP2, cE1 = a.cE1, cE2 = a.cE2;
    const R lamh = a.lamh, kappa = a.kappa, deta = a.deta;
    constexpr bool GAUSS = MEAS;                  // Gauss residual in this march
    constexpr bool GLDS = GAUSS && sizeof(R) == 4;  // its -x / -y E through LDS (FP64: loads)
    constexpr bool EARLY = MEAS || (sizeof(R) == 8 && TX == 32);  // next phase's loads ahead of the barrier

    const R inv_dx = R(1) / dx;
    const R inv_dx2 = inv_dx * inv_dx;
    const int P = a.P;
    const int64_t NN = (int64_t)N * P;  // plane stride
    const uint32_t pb = (uint32_t)NN * (uint32_t)sizeof(R);  // bytes of a plane (N P < 2^28)

    const int tid = threadIdx.x;
    const int lx = tid % TX, ly = tid / TX;
    const int gx = x0 + lx, gy = y0 + ly;
    const bool active = gx < N && gy < N;
    const int gxw = wrapi(gx, N), gyw = wrapi(gy, N);
    // byte offsets in a plane: of the own site, and for the stores (kNoSite for
    // the lanes past a ragged edge and for a pass that only measures)
    const uint32_t ob = ((uint32_t)gxw + (uint32_t)P * (uint32_t)gyw) * (uint32_t)sizeof(R);
    const uint32_t so = write && active ? ob : kNoSite;
    int ro = (ly + 1) * RW + (lx + 1);  // own region slot

    // halo ring site of this thread (if any)
    const bool has_halo = tid < H;
    const bool halo_wave = uniform(tid & ~63) < H;  // a wave with halo sites
    int rh = 0, hrx = 0, hry = 0;
    uint32_t hb = kNoSite;
    if (has_halo) {
        if (tid < RW) {
            hrx = tid;
            hry = 0;
        } else if (tid < 2 * RW) {
            hrx = tid - RW;
            hry = TY + 1;
        } else if (tid < 2 * RW + TY) {
            hrx = 0;
            hry = 1 + (tid - 2 * RW);
        } else {
            hrx = TX + 1;
            hry = 1 + (tid - 2 * RW - TY);
        }
        rh = hry * RW + hrx;
        hb = ((uint32_t)wrapi(x0 - 1 + hrx, N) + (uint32_t)P * (uint32_t)wrapi(y0 - 1 + hry, N)) * (uint32_t)sizeof(R);
    }
    // Link phases on the halo that the windings of the tile read: Y_x and Y_z
    // of the +y row, Y_y and Y_z of the +x column.  Each is one evaluation of
    // some fifty instructions; a wave that made two of them on top of its halo
    // links would hold every barrier up, so they are dealt out one to a thread
    // from the last thread down, away from the waves with the halo sites.
    static_assert(2 * (TX + TY) <= NT, "a halo link phase per thread at most");
    const int ph_t = NT - 1 - tid;
    const bool has_ph = MEAS && ph_t < 2 * (TX + TY);
    const bool ph_wave = MEAS && uniform(NT - 1 - (tid | 63)) < 2 * (TX + TY);
    const bool ph_row = ph_t < 2 * TX;
    const bool ph_z = ph_row ? ph_t >= TX : ph_t >= 2 * TX + TY;        // Y_z
    const int ph_k = ph_row ? ph_t % TX : (ph_t - 2 * TX) % TY;         // place in the row / column
    const int ph_x = ph_row ? 1 + ph_k : TX + 1, ph_y = ph_row ? TY + 1 : 1 + ph_k;
    const int ph_d = ph_z ? 2 : (ph_row ? 0 : 1);
    const int ph_r = has_ph ? ph_y * RW + ph_x : 0;                     // region slot
    const int ph_n = ph_r + (ph_row ? 1 : RW);                          // that of the neighbour (not for Y_z)
    const uint32_t ph_b = has_ph && ph_z ? ((uint32_t)wrapi(x0 - 1 + ph_x, N) + (uint32_t)P * (uint32_t)wrapi(y0 - 1 + ph_y, N)) *
                                       (uint32_t)sizeof(R)
                                         : kNoSite;
    // halo sites whose E the Gauss residual of the tile reads: E_x on the -x
    // column, E_y on the -y row
    const bool halo_ex = has_halo && hrx == 0 && hry >= 1 && hry <= TY;
    const bool halo_ey = has_halo && hry == 0 && hrx >= 1 && hrx <= TX;
    const bool halo_e = GLDS && (halo_ex || halo_ey);
    const uint32_t hbx = halo_ex ? hb : kNoSite, hby = halo_ey ? hb : kNoSite;
    const int hEc = halo_ex ? 0 : 1;

    auto plane_of = [&](int z) -> int64_t { return (int64_t)wrapz(z, N) * NN; };
    auto in_p = [&](int64_t plane) { return plane_bufs(a.b.ip, a.b.fs, plane, pb); };
    auto in_m = [&](int64_t plane) { return plane_bufs(a.b.im, a.b.fs, plane, pb); };
    auto ld = [](Rsrc r, uint32_t off) -> R { return ld_plane<R>(r, off); };
    auto ld_nt = [](Rsrc r, uint32_t off) -> R { return ld_plane<R, true>(r, off); };

    // The FP64 marches read the site's own links of planes z and z+1 from LDS
    // where they use them rather than carrying them from plane to plane in
    // registers, but for U_z of plane z+1.
    constexpr bool ULDS = sizeof(R) == 8;
    Cx<R> Uc[3], Up[3];
    R Ac[3], Ap[3];
    Cx<R> phi_c, phi_p;
    R pr_c, pi_c, e_c[3];
    Cx<R> bz_m;  // conj(U_z) phi of the own site one plane below
    R fxz_m, fyz_m;
    // halo site: U_z and (MEAS) A of plane z+1, into LDS during phase z
    Cx<R> huz = {};
    R ha1[3] = {0, 0, 0};
    // diagnostics state (MEAS): the windings of plane z need its halo's link
    // phases, and those of the (x, z) and (y, z) plaquettes Y_x, Y_y of plane
    // z+1, so they are completed one plane later from the own link phases (_b)
    // and the plaquette angles of plane z
    float yx_b = 0.f, yy_b = 0.f, yz_b = 0.f;
    double th_b[3] = {0.0, 0.0, 0.0};  // (x, y), (x, z), (y, z)
    // link phase of a link U = exp(-i dx a) between phi values ph and pn
    auto phase = [&](Cx<R> ph, Cx<R> U, Cx<R> pn, R av) -> float {
        if constexpr (sizeof(R) == 8)
            return link_phase(ph.r, ph.i, U, pn.r, pn.i);
        else {
            float y[1];
            link_phases_f<1>({cmulc(ph, cmul(U, pn))}, ph, {pn}, {av}, ma.dx, y);
            return y[0];
        }
    };
    // sums of the march: M_KIN .. M_RHOL (kMarchSums slots, FP64) and the
    // exact counts M_WABS, M_NONFIN (integers); the Gauss sums follow
    double acc[kMarchSums];
    int wabs = 0, nonfin = 0;
    if constexpr (MEAS)
        for (int k = 0; k < kMarchSums; ++k) acc[k] = 0.0;
    // Gauss residual (GAUSS): sums of G^2, (div E)^2, (c rho)^2, max |G|, and
    // E_z of the own site one plane below
    double g2 = 0.0, d2 = 0.0, c2 = 0.0, gmax = 0.0;
    R ezm = R(0);
    // FP64: E_x at x - kx and E_y at x - ky of plane z, loaded with the plane's
    // Pi and E (Pi and E go to other buffers, so these are the snapshot's)
    R ex_xm = R(0), ey_ym = R(0);
    const uint32_t row = (uint32_t)P * (uint32_t)sizeof(R);
    const uint32_t ob_xm = gxw == 0 ? ob + (uint32_t)(N - 1) * (uint32_t)sizeof(R) : ob - (uint32_t)sizeof(R);
    const uint32_t ob_ym = gyw == 0 ? ob + (uint32_t)(N - 1) * row : ob - row;
    const double inv_dx64 = 1.0 / ma.dx;
    // Operands of phase t, loaded during the phase before it: A of plane t+2
    // (own and halo), phi of plane t+1 (halo) and t+2 (own), Pi and E of plane
    // t+1 (own).
    struct Pre {
        R a[3], ha[3];
        Cx<R> hphi, phi2;
        R pr, pi, e[3];
        Cx<R> he;      // GLDS: E_x, E_y of plane t+1 at the halo site (it needs one of them)
        Cx<R> pphi;    // phi of plane t+1 at the halo link phase's site
        R exm, eym;    // FP64 Gauss: E_x at x - kx, E_y at x - ky of plane t+1
    };
    // The halo loads come first: only some waves make them, and what follows
    // them is the same for every wave, so that the waits can count it.
    auto prefetch = [&](int t, Pre& q) {
        const int64_t p1 = plane_of(t + 1);
        const PlaneBufs f2 = in_p(plane_of(t + 2)), m1 = in_m(p1);
        if (halo_wave) {
            for (int d = 0; d < 3; ++d) q.ha[d] = ld(f2.f[B_A + d], hb);
            const PlaneBufs f1 = in_p(p1);
            q.hphi = {ld(f1.f[B_PHR], hb), ld(f1.f[B_PHI], hb)};
            if constexpr (GLDS) q.he = {ld(m1.f[B_E], hbx), ld(m1.f[B_E + 1], hby)};
        }
        if constexpr (MEAS)
            if (ph_wave) {
                const PlaneBufs f1 = in_p(p1);
                q.pphi = {ld(f1.f[B_PHR], ph_b), ld(f1.f[B_PHI], ph_b)};
            }
        for (int d = 0; d < 3; ++d) q.a[d] = ld(f2.f[B_A + d], ob);
        if constexpr (GAUSS && !GLDS) {
            q.exm = ld(m1.f[B_E], ob_xm);
            q.eym = ld(m1.f[B_E + 1], ob_ym);
        }
        q.phi2 = {ld(f2.f[B_PHR], ob), ld(f2.f[B_PHI], ob)};
        q.pr = ld_nt(m1.f[B_PIR], ob);
        q.pi = ld_nt(m1.f[B_PII], ob);
        for (int d = 0; d < 3; ++d) q.e[d] = ld_nt(m1.f[B_E + d], ob);
    };
    Pre q;
    {
        // Every load of the prologue, and those of the first phase, are issued
        // before its first barrier: a chunk then starts with one round of
        // memory latency.
        const int64_t pm = plane_of(z0 - 1), p0 = plane_of(z0), p1 = plane_of(z0 + 1);
        const PlaneBufs fm = in_p(pm), f0 = in_p(p0), f1 = in_p(p1), m0 = in_m(p0);
        R am[3], hm[1] = {0}, h0[3] = {0, 0, 0};
        Cx<R> hph0 = {}, he0 = {};
        if (halo_wave) {
            hm[0] = ld(fm.f[B_A + 2], hb);
            for (int d = 0; d < 3; ++d) h0[d] = ld(f0.f[B_A + d], hb);
            for (int d = 0; d < 3; ++d) ha1[d] = ld(f1.f[B_A + d], hb);
            hph0 = Cx<R>{ld(f0.f[B_PHR], hb), ld(f0.f[B_PHI], hb)};
            if constexpr (GLDS) he0 = {ld(m0.f[B_E], hbx), ld(m0.f[B_E + 1], hby)};
        }
        for (int d = 0; d < 3; ++d) am[d] = ld(fm.f[B_A + d], ob);
        for (int d = 0; d < 3; ++d) Ac[d] = ld(f0.f[B_A + d], ob);
        for (int d = 0; d < 3; ++d) Ap[d] = ld(f1.f[B_A + d], ob);
        const Cx<R> phi_m{ld(fm.f[B_PHR], ob), ld(fm.f[B_PHI], ob)};
        phi_c = {ld(f0.f[B_PHR], ob), ld(f0.f[B_PHI], ob)};
        phi_p = {ld(f1.f[B_PHR], ob), ld(f1.f[B_PHI], ob)};
        pr_c = ld_nt(m0.f[B_PIR], ob);
        pi_c = ld_nt(m0.f[B_PII], ob);
        for (int d = 0; d < 3; ++d) e_c[d] = ld_nt(m0.f[B_E + d], ob);
        if constexpr (GAUSS) ezm = ld(in_m(pm).f[B_E + 2], ob);
        if constexpr (GAUSS && !GLDS) {
            ex_xm = ld(m0.f[B_E], ob_xm);
            ey_ym = ld(m0.f[B_E + 1], ob_ym);
        }
        if (MEAS || z0 + 1 < z1) prefetch(z0, q);

        // planes z0 and z0+1: x, y links into slots 0 and 1; U_z of z0 into
        // slot 0, of z0-1 (for F there) into slot 1
        Cx<R> um[3], uh[3], uhm[1];
        links(dx, am, um);
        links(dx, Ac, Uc);
        links(dx, Ap, Up);
        sh.W[1].at(ro, 0) = um[2];
        sh.W[0].set(ro, Uc[2], phi_c);
        sh.U[0].set(ro, Uc[0], Uc[1]);
        sh.U[1].set(ro, Up[0], Up[1]);
        if constexpr (MEAS)
            for (int d = 0; d < 3; ++d) mx->A[0][d][ro] = Ac[d];
        if (has_halo) {
            links(dx, hm, uhm);
            sh.W[1].at(rh, 0) = uhm[0];
            links(dx, h0, uh);
            sh.W[0].set(rh, uh[2], hph0);
            sh.U[0].set(rh, uh[0], uh[1]);
            links(dx, ha1, uh);
            sh.U[1].set(rh, uh[0], uh[1]);
            huz = uh[2];
            if constexpr (MEAS)
                for (int d = 0; d < 3; ++d) mx->A[0][d][rh] = h0[d];
        }
        if constexpr (GLDS) {
            mx->E[0][0][ro] = e_c[0];
            mx->E[0][1][ro] = e_c[1];
            if (halo_e) mx->E[0][hEc][rh] = halo_ex ? he0.r : he0.i;
        }
        bz_m = cmulc(um[2], phi_m);
        __syncthreads();
        // F_xz, F_yz of the own column at plane z0-1
        fxz_m = plaq_sin(um[0], sh.W[1].get(ro + 1, 0), Uc[0], um[2]) * inv_dx2;
        fyz_m = plaq_sin(um[1], sh.W[1].get(ro + RW, 0), Uc[1], um[2]) * inv_dx2;
        __syncthreads();
        // wait here for the loads that the first plane takes from registers,
        // rather than on every pass through the loop that it enters
        asm volatile("" : "+v"(pr_c), "+v"(pi_c), "+v"(e_c[0]), "+v"(e_c[1]), "+v"(e_c[2]));
        if constexpr (GAUSS) asm volatile("" : "+v"(ezm));
        if constexpr (GAUSS && !GLDS) asm volatile("" : "+v"(ex_xm), "+v"(ey_ym));
    }

    // The march, a phase and a barrier per plane: phase z updates plane z and
    // forms the links of plane z+2.  What it writes to LDS, no wave reads
    // before the barrier that ends it.
    int s0 = 0, s1 = 1, s2 = 2;  // slots of the x, y links of planes z, z+1, z+2
    for (int z = z0, b = 0;; ++z, b ^= 1) {
        const bool more = z + 1 < z1;  // there is a next plane to update
        // neighbour slots in the region
        const int rxm = ro - 1, rxp = ro + 1, rym = ro - RW, ryp = ro + RW;
        const int rxm_yp = ro - 1 + RW, rxp_ym = ro + 1 - RW;
        const auto &su = sh.U[s0], &sup = sh.U[s1];  // x, y links of planes z and z+1
        const auto& sw = sh.W[b];                     // U_z and phi of plane z
        if constexpr (MEAS)
            if (has_ph) {
                const Cx<R> u = ph_z ? sw.get(ph_r, 0) : su.get(ph_r, ph_row ? 0 : 1), nb = sw.get(ph_n, 1), up = q.pphi;
                mx->Y[b][ph_d][ph_r] = phase(sw.get(ph_r, 1), u, ph_z ? up : nb, mx->A[b][ph_d][ph_r]);
            }

        // ---- 1. update of the own site at plane z
        {
            if constexpr (ULDS) {
                su.get(ro, &Uc[0], &Uc[1]);
                Uc[2] = sw.get(ro, 0);
                sup.get(ro, &Up[0], &Up[1]);
            }
            if constexpr (GAUSS && !GLDS) {
                // FP64: the Gauss residual of the site first, while few values
                // are live (FP32 forms it with the other diagnostics below)
                if (active) {
                    const double dv = (((double)e_c[0] - (double)ex_xm) * inv_dx64 +
                                       ((double)e_c[1] - (double)ey_ym) * inv_dx64) +
                                      ((double)e_c[2] - (double)ezm) * inv_dx64;
                    const double crho = ma.gauss_c * ((double)phi_c.r * (double)pi_c -
                                                      (double)phi_c.i * (double)pr_c);
                    const double G = dv - crho;
                    g2 += G * G;
                    d2 += dv * dv;
                    c2 += crho * crho;
                    gmax = fmax(gmax, fabs(G));
                }
            }
            Cx<R> ph_xm, ph_xp, ph_ym, ph_yp, uz_xm, uz_xp, uz_ym, uz_yp;
            Cx<R> ux_xm, uy_xm, ux_ym, uy_ym;  // U_x, U_y at x-kx and x-ky
            if constexpr (Pair<R, 1>::kBeside) {
                sw.get(rxm, &uz_xm, &ph_xm);
                sw.get(rxp, &uz_xp, &ph_xp);
                sw.get(rym, &uz_ym, &ph_ym);
                sw.get(ryp, &uz_yp, &ph_yp);
                su.get(rxm, &ux_xm, &uy_xm);
                su.get(rym, &ux_ym, &uy_ym);
            } else {  // the others where they are used
                ph_xm = sw.get(rxm, 1);
                ph_xp = sw.get(rxp, 1);
                ph_ym = sw.get(rym, 1);
                ph_yp = sw.get(ryp, 1);
                ux_xm = su.get(rxm, 0);
                uy_ym = su.get(rym, 1);
            }
            // covariant Laplacian: sum_j U_j^x phi^{x+j} + conj(U_j^{x-j}) phi^{x-j} - 2 phi^x
            const Cx<R> fx = cmul(Uc[0], ph_xp), fy = cmul(Uc[1], ph_yp), fz = cmul(Uc[2], phi_p);
            const Cx<R> bx = cmulc(ux_xm, ph_xm), by = cmulc(uy_ym, ph_ym), bz = bz_m;
            const R lr = ((fx.r + bx.r) + (fy.r + by.r)) + fm(R(-6), phi_c.r, fz.r + bz.r);
            const R li = ((fx.i + bx.i) + (fy.i + by.i)) + fm(R(-6), phi_c.i, fz.i + bz.i);
            // currents J_i = Im[conj(phi) U_i phi^{x+i}] / dx
            const R jx = fm(phi_c.r, fx.i, -(phi_c.i * fx.r)) * inv_dx;
            const R jy = fm(phi_c.r, fy.i, -(phi_c.i * fy.r)) * inv_dx;
            const R jz = fm(phi_c.r, fz.i, -(phi_c.i * fz.r)) * inv_dx;
            if constexpr (MEAS) {
                // own link phases of plane z (FP32 lattices: z = conj(phi) U phi^{x+j}
                // is the forward product of the Laplacian)
                float yx_c, yy_c, yz_c;
                if constexpr (sizeof(R) == 8) {
                    yx_c = link_phase(phi_c.r, phi_c.i, Uc[0], ph_xp.r, ph_xp.i);
                    yy_c = link_phase(phi_c.r, phi_c.i, Uc[1], ph_yp.r, ph_yp.i);
                    yz_c = link_phase(phi_c.r, phi_c.i, Uc[2], phi_p.r, phi_p.i);
                } else {
                    float y[3];
                    link_phases_f<3>({cmulc(phi_c, fx), cmulc(phi_c, fy), cmulc(phi_c, fz)}, phi_c,
                                     {ph_xp, ph_yp, phi_p}, Ac, ma.dx, y);
                    yx_c = y[0];
                    yy_c = y[1];
                    yz_c = y[2];
                }
                auto& sY = mx->Y[b];
                sY[0][ro] = yx_c;
                sY[1][ro] = yy_c;
                sY[2][ro] = yz_c;
                // the windings at x, plane z-1, now that its link phases are all
                // there and Y_x, Y_y of plane z are known
                const auto& sYb = mx->Y[b ^ 1];
                if (z > z0) {
                    const int w = abs(winding_of(yx_b, sYb[1][rxp], sYb[0][ryp], yy_b, th_b[0])) +
                                  abs(winding_of(yx_b, sYb[2][rxp], yx_c, yz_b, th_b[1])) +
                                  abs(winding_of(yy_b, sYb[2][ryp], yy_c, yz_b, th_b[2]));
                    wabs += active ? w : 0;
                }
                yx_b = yx_c;
                yy_b = yy_c;
                yz_b = yz_c;
                // plaquette angles at x, plane z, from the stored A
                const auto& sA = mx->A[b];
                const R q4[3][4] = {{Ac[0], sA[1][rxp], sA[0][ryp], Ac[1]},
                                    {Ac[0], sA[2][rxp], Ap[0], Ac[2]},
                                    {Ac[1], sA[2][ryp], Ap[1], Ac[2]}};
                plaq_angles(ma.dx, q4, th_b);
            }
            // plaquettes at x (F_ij^x, i<j)
            const Cx<R> uy_xp = su.get(rxp, 1), ux_yp = su.get(ryp, 0);
            if constexpr (!Pair<R, 1>::kBeside) {
                uz_xp = sw.get(rxp, 0);
                uz_yp = sw.get(ryp, 0);
            }
            R sxy, sxz, syz, oxy = 0, oxz = 0, oyz = 0;
            if constexpr (MEAS) {
                oxy = plaq_omc(Uc[0], uy_xp, ux_yp, Uc[1], &sxy);
                oxz = plaq_omc(Uc[0], uz_xp, Up[0], Uc[2], &sxz);
                oyz = plaq_omc(Uc[1], uz_yp, Up[1], Uc[2], &syz);
            } else {
                sxy = plaq_sin(Uc[0], uy_xp, ux_yp, Uc[1]);
                sxz = plaq_sin(Uc[0], uz_xp, Up[0], Uc[2]);
                syz = plaq_sin(Uc[1], uz_yp, Up[1], Uc[2]);
            }
            const R fxy = sxy * inv_dx2;
            const R fxz = sxz * inv_dx2;
            const R fyz = syz * inv_dx2;
            // plaquettes at x - kx and x - ky
            if constexpr (!Pair<R, 1>::kBeside) {
                uy_xm = su.get(rxm, 1);
                uz_xm = sw.get(rxm, 0);
                ux_ym = su.get(rym, 0);
                uz_ym = sw.get(rym, 0);
            }
            const Cx<R> ux_xm_yp = su.get(rxm_yp, 0), uy_xp_ym = su.get(rxp_ym, 1);
            const Cx<R> ux_xm_zp = sup.get(rxm, 0), uy_ym_zp = sup.get(rym, 1);
            const R fxy_xm = plaq_sin(ux_xm, Uc[1], ux_xm_yp, uy_xm) * inv_dx2;
            const R fxy_ym = plaq_sin(ux_ym, uy_xp_ym, Uc[0], uy_ym) * inv_dx2;
            const R fxz_xm = plaq_sin(ux_xm, Uc[2], ux_xm_zp, uz_xm) * inv_dx2;
            const R fyz_ym = plaq_sin(uy_ym, Uc[2], uy_ym_zp, uz_ym) * inv_dx2;
            // lattice curl C_i = sum_{j != i} (F_ij^x - F_ij^{x-j}) / dx, F_ji = -F_ij
            const R cx = ((fxy - fxy_ym) + (fxz - fxz_m)) * inv_dx;
            const R cy = ((fyz - fyz_m) - (fxy - fxy_xm)) * inv_dx;
            const R cz = -((fxz - fxz_xm) + (fyz - fyz_ym)) * inv_dx;
            // Crank-Nicolson kick, drift
            const R m2 = fm(phi_c.r, phi_c.r, fm(phi_c.i, phi_c.i, -sigma2));
            const R pot = lamh * m2;
            const R npr = fm(cP1, pr_c, cP2 * fm(lr, inv_dx2, -(pot * phi_c.r)));
            const R npi = fm(cP1, pi_c, cP2 * fm(li, inv_dx2, -(pot * phi_c.i)));
            const R ne0 = fm(cE1, e_c[0], cE2 * fm(kappa, jx, -cx));
            const R ne1 = fm(cE1, e_c[1], cE2 * fm(kappa, jy, -cy));
            const R ne2 = fm(cE1, e_c[2], cE2 * fm(kappa, jz, -cz));
            const int64_t o = (int64_t)z * NN;
            const PlaneBufs wm = plane_bufs(a.b.om, a.b.fs, o, pb), wp = plane_bufs(a.b.op, a.b.fs, o, pb);
            st_plane(wm.f[B_PIR], so, npr);
            st_plane(wm.f[B_PII], so, npi);
            st_plane(wm.f[B_E], so, ne0);
            st_plane(wm.f[B_E + 1], so, ne1);
            st_plane(wm.f[B_E + 2], so, ne2);
            st_plane(wp.f[B_PHR], so, fm(deta, npr, phi_c.r));
            st_plane(wp.f[B_PHI], so, fm(deta, npi, phi_c.i));
            st_plane(wp.f[B_A], so, fm(deta, ne0, Ac[0]));
            st_plane(wp.f[B_A + 1], so, fm(deta, ne1, Ac[1]));
            st_plane(wp.f[B_A + 2], so, fm(deta, ne2, Ac[2]));
            if constexpr (MEAS) {
                if (active) {
                    // site densities with centred momenta (average of the stored
                    // half step and the kick), summed in FP64
                    const R v[10] = {phi_c.r, phi_c.i, pr_c, pi_c, Ac[0], Ac[1], Ac[2], e_c[0], e_c[1], e_c[2]};
                    // 0 v is 0 for a finite v, else NaN
                    R bad0 = 0, bad1 = 0;
                    for (int k = 0; k < 5; ++k) {
                        bad0 = fm(v[k], R(0), bad0);
                        bad1 = fm(v[5 + k], R(0), bad1);
                    }
                    nonfin += bad0 + bad1 == R(0) ? 0 : 1;
                    const R pbr = R(0.5) * (pr_c + npr), pbi = R(0.5) * (pi_c + npi);
                    const double kin = (double)fm(pbr, pbr, pbi * pbi);
                    const R d0r = fx.r - phi_c.r, d0i = fx.i - phi_c.i;
                    const R d1r = fy.r - phi_c.r, d1i = fy.i - phi_c.i;
                    const R d2r = fz.r - phi_c.r, d2i = fz.i - phi_c.i;
                    const double grad =
                        (double)(((d0r * d0r + d0i * d0i) + (d1r * d1r + d1i * d1i) + (d2r * d2r + d2i * d2i)) *
                                 inv_dx2);
                    const double pot_e = ma.lam_quarter * (double)m2 * (double)m2;
                    const R eb0 = R(0.5) * (e_c[0] + ne0), eb1 = R(0.5) * (e_c[1] + ne1),
                            eb2 = R(0.5) * (e_c[2] + ne2);
                    const double el = (double)(eb0 * eb0 + eb1 * eb1 + eb2 * eb2) * ma.inv_2e2f;
                    const double mag = (double)(R(2) * (oxy + oxz + oyz) * (inv_dx2 * inv_dx2)) * ma.inv_2e2f;
                    const double L = kin - grad - pot_e + el - mag;
                    acc[M_KIN] += kin;
                    acc[M_GRAD] += grad;
                    acc[M_POT] += pot_e;
                    acc[M_EL] += el;
                    acc[M_MAG] += mag;
                    acc[M_KINL] += kin * L;
                    acc[M_GRADL] += grad * L;
                    // pressure and energy density for the equation-of-state estimator
                    const double pres = (kin - pot_e) + ((el + mag) - grad) * (1.0 / 3.0);
                    const double rho = ((kin + grad) + pot_e) + (el + mag);
                    acc[M_PL] += pres * L;
                    acc[M_RHOL] += rho * L;
                    if constexpr (GLDS) {
                        // G = sum_i (E_i^x - E_i^{x-i}) / dx - c Im[conj(phi) Pi] of the
                        // snapshot, in FP64 from the exactly widened stored values
                        const double dv = (((double)e_c[0] - (double)mx->E[b][0][rxm]) * inv_dx64 +
                                           ((double)e_c[1] - (double)mx->E[b][1][rym]) * inv_dx64) +
                                          ((double)e_c[2] - (double)ezm) * inv_dx64;
                        const double crho = ma.gauss_c * ((double)phi_c.r * (double)pi_c -
                                                          (double)phi_c.i * (double)pr_c);
                        const double G = dv - crho;
                        g2 += G * G;
                        d2 += dv * dv;
                        c2 += crho * crho;
                        gmax = fmax(gmax, fabs(G));
                    }
                }
            }
            fxz_m = fxz;
            fyz_m = fyz;
            bz_m = cmulc(Uc[2], phi_c);  // for plane z+1
        }

        if (!MEAS && !more) break;

        // ---- 2. planes z+1 and z+2 into LDS: phi and U_z of plane z+1 (U_z held
        //         since the phase before), x and y links of plane z+2
        sh.W[b ^ 1].set(ro, Up[2], phi_p);
        if (has_halo) sh.W[b ^ 1].set(rh, huz, q.hphi);
        if (!more) break;
        Cx<R> u2[3];
        if (has_halo) {
            links(dx, q.ha, u2);
            sh.U[s2].set(rh, u2[0], u2[1]);
            huz = u2[2];
            if constexpr (MEAS)
                for (int d = 0; d < 3; ++d) {
                    mx->A[b ^ 1][d][rh] = ha1[d];
                    ha1[d] = q.ha[d];
                }
            if constexpr (GLDS)
                if (halo_e) mx->E[b ^ 1][hEc][rh] = halo_ex ? q.he.r : q.he.i;
        }
        links(dx, q.a, u2);
        sh.U[s2].set(ro, u2[0], u2[1]);
        if constexpr (MEAS)
            for (int d = 0; d < 3; ++d) mx->A[b ^ 1][d][ro] = Ap[d];
        if constexpr (GLDS) {
            mx->E[b ^ 1][0][ro] = q.e[0];
            mx->E[b ^ 1][1][ro] = q.e[1];
        }

        // ---- 3. rotate the own-column registers, and issue the loads of the
        //         next phase
        if constexpr (GAUSS) ezm = e_c[2];
        if constexpr (GAUSS && !GLDS) {
            ex_xm = q.exm;
            ey_ym = q.eym;
        }
        for (int d = 0; d < 3; ++d) {
            if constexpr (!ULDS) Uc[d] = Up[d];
            if (!ULDS || d == 2) Up[d] = u2[d];
            Ac[d] = Ap[d];
            Ap[d] = q.a[d];
            e_c[d] = q.e[d];
        }
        phi_c = phi_p;
        phi_p = q.phi2;
        pr_c = q.pr;
        pi_c = q.pi;
        // Measured march: issued before the barrier, which hides more of their
        // latency.  Plain march, which memory bounds: after it, and with the
        // plane's stores complete, so that the workgroups that share an L2 stay
        // within a plane of each other and their halo reads hit it.  (FP64 32 x
        // 8, whose narrow tiles read the most halo, gains 1 to 3% from early
        // loads all the same: MI355X 256^3 593 us after the barrier, 580
        // before it, 512^3 4750 and 4670; the other shapes lose.)
        if constexpr (EARLY)
            if (MEAS || z + 2 < z1) prefetch(z + 1, q);
        if constexpr (!MEAS) __builtin_amdgcn_s_waitcnt(kWaitVm0);
        __syncthreads();
        if constexpr (!EARLY)
            if (z + 2 < z1) prefetch(z + 1, q);
        const int t = s0;
        s0 = s1;
        s1 = s2;
        s2 = t;
    }
    if constexpr (MEAS) {
        // own Y_x, Y_y of plane z1 complete the windings of the chunk's last plane
        __syncthreads();
        const int b = (z1 - 1 - z0) & 1, rxp = ro + 1, ryp = ro + RW;
        const auto& sw = sh.W[b ^ 1];
        const float yx_n = phase(phi_p, Up[0], sw.get(rxp, 1), Ap[0]);
        const float yy_n = phase(phi_p, Up[1], sw.get(ryp, 1), Ap[1]);
        if (active) {
            const auto& sYb = mx->Y[b];
            wabs += abs(winding_of(yx_b, sYb[1][rxp], sYb[0][ryp], yy_b, th_b[0])) +
                    abs(winding_of(yx_b, sYb[2][rxp], yx_n, yz_b, th_b[1])) +
                    abs(winding_of(yy_b, sYb[2][ryp], yy_n, yz_b, th_b[2]));
        }
    }

    if constexpr (MEAS) {
        // fixed-order block reduction of the diagnostics into one record
        static_assert(M_KIN == 0 && kMarchSums == M_RHOL + 1, "march sums occupy slots 0 .. M_RHOL");
        auto& red = mx->red;
        const int lane = tid & 63, wv = tid >> 6;
        double v[16] = {};
        static_assert(kMeasStride == 16, "a record's slots are reduced together");
        for (int k = 0; k < kMarchSums; ++k) v[k] = acc[k];
        v[M_WABS] = (double)wabs;
        v[M_NONFIN] = (double)nonfin;
        if constexpr (GAUSS) {
            v[M_G2] = g2;
            v[M_DIV2] = d2;
            v[M_CRHO2] = c2;
        }
        const double r = wave_sums(v);
        if ((lane & 3) == 0 && lane >> 2 < M_COUNT && lane >> 2 != M_GMAX) red[wv][lane >> 2] = r;
        if constexpr (GAUSS) {
            const double m = wave_max(gmax);
            if (lane == 0) red[wv][M_GMAX] = m;
        }
        __syncthreads();
        if (tid < kMeasStride) {
            const bool gslot = tid == M_G2 || tid == M_DIV2 || tid == M_CRHO2 || tid == M_GMAX;
            double r = 0.0;
            if (tid < kMarchSums || tid == M_WABS || tid == M_NONFIN || (GAUSS && gslot)) {
                r = red[0][tid];
                for (int w = 1; w < NT / 64; ++w) r = tid == M_GMAX ? fmax(r, red[w][tid]) : r + red[w][tid];
            }
            record[tid] = r;
        }
    }
}

// Waves per SIMD the compiler must leave room for.  The plain FP32 march
// fits in 128 registers, i.e. four waves per SIMD: two 512-thread workgroups
// per CU, so one can load while the other waits at a barrier.  FP64 fits two
// (its measured march takes 255 registers).  The FP32 measured march takes 198
// and runs two; held to 168 for three it spills 8, and runs slower (512^3 3583
// us against 3400, 128^3 73 against 65).
template <typename R, bool MEAS>
constexpr int kMinWaves = sizeof(R) == 8 ? 2 : (MEAS ? 1 : 4);

// The tile shape of the measured march (measured_tile).
constexpr bool has_measured(int tx, int ty) { return tx == 32 && ty == 8; }

// One lattice: block b owns tile t = xcd_tile(b) (tx fastest, then ty, then
// z-chunk); with MEAS it writes diagnostics record t, so the records are in
// tile order whatever the launch geometry.
template <typename R, int TX, int TY, bool MEAS>
__global__ void __launch_bounds__(TX* TY, (kMinWaves<R, MEAS>)) k_step_tile(StepArgs<R> a, MeasArgs ma, double* partials, int write,
                                                      int zchunk, int tiles_x, int tiles_y)
{
    __shared__ TileShared<R, TX, TY> sh;
    __shared__ MeasShared<R, TX, MEAS ? TY : 8> mxs;
    const int t0 = xcd_tile(blockIdx.x, gridDim.x);
    int t = t0;
    const int tx = t % tiles_x;
    t /= tiles_x;
    const int ty = t % tiles_y;
    const int tz = t / tiles_y;
    const int z0 = tz * zchunk;
    const int z1 = (z0 + zchunk < a.N) ? z0 + zchunk : a.N;
    if constexpr (MEAS)
        march_step<R, TX, TY, true>(sh, &mxs, a, ma, partials + (int64_t)t0 * kMeasStride, write != 0, tx * TX,
                                    ty * TY, z0, z1);
    else
        march_step<R, TX, TY, false>(sh, nullptr, a, ma, nullptr, true, tx * TX, ty * TY, z0, z1);
}


// Many lattices in one launch: blocks stride over a work list of
// (lattice, tile) items; each lattice reads its own step counter k, takes the
// coefficients of step k from its own FP64 table, and is skipped once it has
// run its steps.  MEAS: only lattices whose snapshot k is due for diagnostics
// (measured step, or measurement alone for the final snapshot); otherwise
// only lattices that are not due.

template <typename R, int TX, int TY, bool MEAS>
__global__ void __launch_bounds__(TX* TY, (kMinWaves<R, MEAS>)) k_step_batch(const PoolLattice* __restrict__ lat,
                                                       const WorkItem* __restrict__ work, int nwork)
{
    __shared__ TileShared<R, TX, TY> sh;
    __shared__ MeasShared<R, TX, MEAS ? TY : 8> mxs;
    // one work item per block; XCD x gets the x-th eighth of the list (the
    // host lays the list out so that this is an equal share of every lattice)
    const int w = xcd_tile(blockIdx.x, nwork);
    const WorkItem it = work[w];
    if (it.lattice < 0) return;
    const PoolLattice& L = lat[it.lattice];
    const int64_t k = L.counter[0];
    const bool due = measure_due(L, k);
    if (MEAS != due) return;                     // uniform across the block
    if (!MEAS && (k >= L.nsteps || two_step_due(L, k))) return;
    const double* row = L.coef + k * kCoefStride;
    const int cur = (int)L.counter[2], curm = (int)L.counter[3];
    StepArgs<R> a;
    // Pi and E in place, but out of place for the measured march
    a.b = Blocks<R>{(const R*)L.pp[cur], (const R*)L.mom[curm], (R*)L.pp[cur ^ 1],
                    (R*)L.mom[MEAS ? curm ^ 1 : curm], L.fs};
    a.N = L.N;
    a.P = L.P;
    a.dx = (R)L.dx;
    a.sigma2 = (R)L.sigma2;
    a.cP1 = (R)row[C_P1];
    a.cP2 = (R)row[C_P2];
    a.cE1 = (R)row[C_E1];
    a.cE2 = (R)row[C_E2];
    a.lamh = (R)row[C_LAMH];
    a.kappa = (R)row[C_KAPPA];
    a.deta = (R)L.deta;
    a = uniform(a);
    const MeasArgs ma = uniform(MeasArgs{L.dx, row[C_INV2E2F], row[C_LAMQ], row[C_GAUSS]});
    // the measured node runs the lattice's measured tiling, the plain node its step tiling
    const int tiles_x = MEAS ? L.mtiles_x : L.tiles_x, tiles_y = MEAS ? L.mtiles_y : L.tiles_y;
    const int zchunk = MEAS ? L.meas_zchunk : L.zchunk;
    int t = it.tile;
    const int tx = t % tiles_x;
    t /= tiles_x;
    const int ty = t % tiles_y;
    const int tz = t / tiles_y;
    const int z0 = uniform(tz * zchunk);
    const int z1 = uniform((z0 + zchunk < L.N) ? z0 + zchunk : L.N);
    const int x0 = uniform(tx * TX), y0 = uniform(ty * TY);
    if constexpr (MEAS)
        march_step<R, TX, TY, true>(sh, &mxs, a, ma, uniform(L.partials + (int64_t)it.tile * kMeasStride),
                                    k < L.nsteps, x0, y0, z0, z1);
    else
        march_step<R, TX, TY, false>(sh, nullptr, a, ma, nullptr, true, x0, y0, z0, z1);
}


// Fold the records of every due lattice into its measurement series (one
// block per lattice, the same fixed order as the single-lattice fold).
__global__ void __launch_bounds__(kFoldThreads) k_fold_batch(const PoolLattice* __restrict__ lat, int nlat)
{
    __shared__ double red[kFoldRed];
    const PoolLattice& L = lat[blockIdx.x];
    const int64_t k = L.counter[0];
    if (!measure_due(L, k)) return;
    const int64_t slot = L.counter[1];
    if (slot >= L.series_cap) return;
    double* out = L.series + slot * kSeriesStride;
    fold_records(L.partials, L.meas_blocks, out, red);
    if (threadIdx.x == 0) {
        out[M_COUNT] = (double)k;
        L.counter[1] = slot + 1;
    }
}

// Advance the counter of every pool lattice that is not finished by what
// this replay did to it: the final measurement one step; a single step one
// step and the phi/A buffer, and the Pi/E buffer too if it was a measured
// step; a two-step pass two steps and both buffers.
__global__ void k_advance_batch(const PoolLattice* __restrict__ lat, int nlat)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nlat) return;
    const PoolLattice& L = lat[i];
    int64_t* c = L.counter;
    const int64_t k = c[0];
    if (k > L.nsteps) return;
    if (k == L.nsteps) {
        c[0] = k + 1;  // the final measurement: finished
    } else if (two_step_due(L, k)) {
        c[0] = k + 2;
        c[2] ^= 1;
        c[3] ^= 1;
    } else {
        c[0] = k + 1;
        c[2] ^= 1;
        if (measure_due(L, k)) c[3] ^= 1;
    }
}

}  // namespace

template <typename R>
hipError_t launch_step_tile(const Fields<R>& in, const Fields<R>& out, const LatticeConst& L, const StepCoef& c,
                            const TileConfig& tc, const MeasConst* mc, double* partials, bool write, hipStream_t s)
{
    const int N = L.N;
    // a measured step reads E of neighbours that other workgroups update:
    // its Pi and E go to other buffers
    if (mc && write && (out.pir == in.pir || out.pii == in.pii || out.e0 == in.e0 || out.e1 == in.e1 ||
                        out.e2 == in.e2))
        return hipErrorInvalidValue;
    StepArgs<R> a;
    if (!blocks_of(in, out, &a.b)) return hipErrorInvalidValue;
    a.N = N;
    a.P = L.P;
    a.dx = (R)L.dx;
    a.sigma2 = (R)L.sigma2;
    a.cP1 = (R)c.cP1;
    a.cP2 = (R)c.cP2;
    a.cE1 = (R)c.cE1;
    a.cE2 = (R)c.cE2;
    a.lamh = (R)c.lam_half;
    a.kappa = (R)c.kappa;
    a.deta = (R)L.deta;
    MeasArgs ma{L.dx, 0.0, 0.0, 0.0};
    if (mc) {
        ma.inv_2e2f = mc->inv_2e2f;
        ma.lam_quarter = mc->lam_quarter;
        ma.gauss_c = mc->gauss_c;
    }
    const int zc = tc.zchunk > 0 ? tc.zchunk : N;
    // MEASv: whether the shape has a measured instance
#define AH_TILE_CASE(TXv, TYv, MEASv)                                                                              \
    if (tc.tx == TXv && tc.ty == TYv) {                                                                            \
        const int tiles_x = (N + TXv - 1) / TXv, tiles_y = (N + TYv - 1) / TYv;                                   \
        const int nb = tiles_x * tiles_y * ((N + zc - 1) / zc);                                                   \
        if (mc) {                                                                                                  \
            if constexpr (!MEASv) return hipErrorInvalidValue;                                                     \
            else                                                                                                   \
                hipLaunchKernelGGL((k_step_tile<R, TXv, TYv, MEASv>), dim3(nb), dim3(TXv * TYv), 0, s, a, ma,      \
                                   partials, write ? 1 : 0, zc, tiles_x, tiles_y);                                \
        } else {                                                                                                   \
            hipLaunchKernelGGL((k_step_tile<R, TXv, TYv, false>), dim3(nb), dim3(TXv * TYv), 0, s, a, ma, partials, \
                               1, zc, tiles_x, tiles_y);                                                          \
        }                                                                                                          \
        return hipGetLastError();                                                                                 \
    }
    AH_TILE_CASE(64, 8, has_measured(64, 8))
    AH_TILE_CASE(64, 4, has_measured(64, 4))
    AH_TILE_CASE(32, 8, has_measured(32, 8))
    AH_TILE_CASE(128, 4, has_measured(128, 4))
    if constexpr (sizeof(R) == 4) {
        AH_TILE_CASE(64, 16, false)
        AH_TILE_CASE(128, 8, false)
    }
#undef AH_TILE_CASE
    return hipErrorInvalidValue;
}

int step_tile_blocks(int N, const TileConfig& tc)
{
    const int zc = tc.zchunk > 0 ? tc.zchunk : N;
    return ((N + tc.tx - 1) / tc.tx) * ((N + tc.ty - 1) / tc.ty) * ((N + zc - 1) / zc);
}

template <typename R>
hipError_t launch_step_batch(const PoolLattice* lat, const WorkItem* work, int nwork, int tx, int ty, int grid,
                             bool measured, hipStream_t s)
{
    // plain node: the shapes of batch_tile_supported; measured node: the
    // measured march's shape (measured_tile)
    if (measured) {
        if (!has_measured(tx, ty)) return hipErrorInvalidValue;
        hipLaunchKernelGGL((k_step_batch<R, 32, 8, true>), dim3(grid), dim3(256), 0, s, lat, work, nwork);
        return hipGetLastError();
    }
    if (!batch_tile_supported(sizeof(R) == 8 ? AH_FP64 : AH_FP32, tx, ty)) return hipErrorInvalidValue;
#define AH_BATCH_CASE(TXv, TYv)                                                                                   \
    if (tx == TXv && ty == TYv) {                                                                                 \
        hipLaunchKernelGGL((k_step_batch<R, TXv, TYv, false>), dim3(grid), dim3(TXv * TYv), 0, s, lat, work, nwork); \
        return hipGetLastError();                                                                                 \
    }
    AH_BATCH_CASE(64, 8)
    AH_BATCH_CASE(64, 4)
    AH_BATCH_CASE(32, 8)
    if constexpr (sizeof(R) == 4) {
        AH_BATCH_CASE(128, 4)
        AH_BATCH_CASE(128, 8)
    }
#undef AH_BATCH_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_fold_batch(const PoolLattice* lat, int nlat, hipStream_t s)
{
    hipLaunchKernelGGL(k_fold_batch, dim3(nlat), dim3(kFoldThreads), 0, s, lat, nlat);
    return hipGetLastError();
}

hipError_t launch_advance_batch(const PoolLattice* lat, int nlat, hipStream_t s)
{
    hipLaunchKernelGGL(k_advance_batch, dim3((nlat + 63) / 64), dim3(64), 0, s, lat, nlat);
    return hipGetLastError();
}

template hipError_t launch_step_batch<double>(const PoolLattice*, const WorkItem*, int, int, int, int, bool,
                                              hipStream_t);
template hipError_t launch_step_batch<float>(const PoolLattice*, const WorkItem*, int, int, int, int, bool,
                                             hipStream_t);

template hipError_t launch_step_tile<double>(const Fields<double>&, const Fields<double>&, const LatticeConst&,
                                             const StepCoef&, const TileConfig&, const MeasConst*, double*, bool,
                                             hipStream_t);
template hipError_t launch_step_tile<float>(const Fields<float>&, const Fields<float>&, const LatticeConst&,
                                            const StepCoef&, const TileConfig&, const MeasConst*, double*, bool,
                                            hipStream_t);

}  // namespace ah
