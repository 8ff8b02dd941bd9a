// Device helpers of the stencil shared by the tiled step kernels: complex
// arithmetic with every fused multiply-add written out, the link variable,
// the plaquette field strength, periodic wrap, XCD-aware tile placement and
// the kick and drift of one site.
//
// Floating-point contraction is off wherever this is included, so each site
// is computed by the same sequence of roundings in every kernel.
#pragma once

#include "ah_internal.h"

#define AH_SINCOS_QUAL __device__
#include "ah_sincos.h"

#pragma clang fp contract(off)

namespace ah {

// A buffer descriptor (raw buffer, stride 0) and the buffer instructions on
// it.  The descriptor is written out word by word: a device address has no
// bits above 47, so its words are the address, the length and the format, and
// stepping to the next field is one 64-bit scalar addition.
typedef int Rsrc __attribute__((ext_vector_type(4)));
typedef float Float2 __attribute__((ext_vector_type(2)));
extern __device__ float buf_load_f32(Rsrc r, int voff, int soff, int aux) __asm("llvm.amdgcn.raw.buffer.load.f32");
extern __device__ Float2 buf_load_2f32(Rsrc r, int voff, int soff, int aux) __asm("llvm.amdgcn.raw.buffer.load.v2f32");
extern __device__ void buf_store_f32(float v, Rsrc r, int voff, int soff, int aux) __asm("llvm.amdgcn.raw.buffer.store.f32");
extern __device__ void buf_store_2f32(Float2 v, Rsrc r, int voff, int soff, int aux) __asm("llvm.amdgcn.raw.buffer.store.v2f32");
constexpr int kBufNt = 2;  // aux: non-temporal

namespace {

__device__ inline float fm(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// A block-uniform value moved into scalar registers.  What a kernel loads
// from a descriptor or a coefficient row in memory, or converts from it, the
// compiler keeps in vector registers (one copy per lane), which would cost a
// march a wave per SIMD of occupancy.
template <typename T>
__device__ inline T uniform(T v)
{
    static_assert(sizeof(T) % 4 == 0, "32-bit words");
    int w[sizeof(T) / 4];
    __builtin_memcpy(w, &v, sizeof(T));
    for (unsigned k = 0; k < sizeof(T) / 4; ++k) w[k] = __builtin_amdgcn_readfirstlane(w[k]);
    __builtin_memcpy(&v, w, sizeof(T));
    return v;
}
__device__ inline double fm(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Access to one plane of a field through a buffer descriptor of exactly that
// plane: its base in scalar registers and a 32-bit byte offset per lane, so an
// access costs no vector address arithmetic and holds no 64-bit vector
// addresses (the FP64 step march takes 150 registers rather than 186).  An
// offset of kNoSite is past the plane's end: the store is dropped.  That keeps
// lanes without a site from storing with no branch, which matters for the
// waits: loads and stores share one in-order counter, and behind a store that
// may have been skipped the compiler can only wait for everything, i.e. each
// plane of a march would wait for its own streaming stores to reach memory.
//
// Pi and E are read and written once per step at their own site, phi and A
// are written once into the other ping-pong buffer; none of it is reused from
// cache within a step, so those accesses (STREAM) are non-temporal and leave
// L2 to the phi / A halo lines that neighbouring tiles read again.
constexpr uint32_t kNoSite = 0xffffffffu;

// s_waitcnt operand (gfx9 encoding): vmcnt(0), the other counters unconstrained
constexpr int kWaitVm0 = 0x0f70;

enum { B_PHR = 0, B_PHI = 1, B_PIR = 0, B_PII = 1, B_A = 2, B_E = 2 };

// Descriptors of one plane of the five fields of a block; `bytes`: the
// plane's length, at most 4096 x 4096 x 8.
struct PlaneBufs {
    Rsrc f[5];
};
template <typename R>
__device__ inline PlaneBufs plane_bufs(const R* block, int64_t fs, int64_t plane, uint32_t bytes)
{
    PlaneBufs b;
    uint64_t q = (uint64_t)(block + plane);
    for (int k = 0; k < 5; ++k, q += (uint64_t)fs * sizeof(R))
        b.f[k] = Rsrc{(int)(uint32_t)q, (int)(uint32_t)(q >> 32), (int)bytes, 0x00020000};  // 32-bit data
    return b;
}
template <typename R, bool STREAM = false>
__device__ inline R ld_plane(Rsrc r, uint32_t off)
{
    if constexpr (sizeof(R) == 4)
        return buf_load_f32(r, (int)off, 0, STREAM ? kBufNt : 0);
    else
        return __builtin_bit_cast(R, buf_load_2f32(r, (int)off, 0, STREAM ? kBufNt : 0));
}
__device__ inline void st_plane(Rsrc r, uint32_t off, float v) { buf_store_f32(v, r, (int)off, 0, kBufNt); }
__device__ inline void st_plane(Rsrc r, uint32_t off, double v)
{
    buf_store_2f32(__builtin_bit_cast(Float2, v), r, (int)off, 0, kBufNt);
}

template <typename R>
struct Cx {
    R r, i;
};
template <typename R>
__device__ inline Cx<R> cmul(Cx<R> a, Cx<R> b)
{
    return {fm(a.r, b.r, -(a.i * b.i)), fm(a.r, b.i, a.i * b.r)};
}
template <typename R>
__device__ inline Cx<R> cmulc(Cx<R> a, Cx<R> b)  // conj(a) * b
{
    return {fm(a.r, b.r, a.i * b.i), fm(a.r, b.i, -(a.i * b.r))};
}

// Two values of each of S sites in LDS (the x and y links, or the z link and
// phi) in one array: FP32 ones side by side, so that one 16-byte access has
// both, FP64 ones in two rows (at 32 bytes from site to site the lanes of a row
// would meet in the same banks).  With an array and 8-byte reads for each value
// LDS reads bound the two-step pass (MI355X, us per step: 512^3 FP32 1495, 1283
// now, FP64 3828, 3610 now; 96^3 FP32 17.2, 14.8); the marches gain little at
// 512^3, 7% on 64^3 FP64 (12.9 to 12.0).  A single value of a pair is read as 8
// bytes (as 16, half of it unused: 1328).
template <typename R, int S>
struct alignas(16) Pair {
    Cx<R> v[2 * S];
    static constexpr bool kBeside = sizeof(R) == 4;
    __device__ __forceinline__ Cx<R>& at(int c, int k) { return v[kBeside ? 2 * c + k : c + k * S]; }
    __device__ __forceinline__ Cx<R> get(int c, int k) const
    {
        return v[kBeside ? 2 * c + k : c + k * S];
    }
    __device__ __forceinline__ void get(int c, Cx<R>* a, Cx<R>* b) const
    {
        if constexpr (kBeside) {
            const float4 q = *(const float4*)&v[2 * c];
            *a = {q.x, q.y};
            *b = {q.z, q.w};
        } else {
            *a = v[c];
            *b = v[c + S];
        }
    }
    __device__ __forceinline__ void set(int c, Cx<R> a, Cx<R> b)
    {
        if constexpr (kBeside) {
            *(float4*)&v[2 * c] = float4{a.r, a.i, b.r, b.i};
        } else {
            v[c] = a;
            v[c + S] = b;
        }
    }
};

// Links U_j = exp(-i dx A_j) = (cos(dx A_j), -sin(dx A_j)) of K values of A.
//
// FP64: the reduced-range sincos (accurate to ~2 ulp for |x| <= 1e9), the
// library routine beyond that (out of line, with the in-range ones of the K
// left as they are: a link phase past 1e9 is a lattice long blown up, and
// inlined it would cost the march registers).
__device__ __noinline__ double2 sincos_far(double x)
{
    double2 v;
    sincos(x, &v.x, &v.y);
    return v;
}
template <int K>
__device__ inline void links(double dx, const double (&a)[K], Cx<double> (&u)[K])
{
    double x[K], far = 0.0;
    for (int d = 0; d < K; ++d) {
        x[d] = dx * a[d];
        double s, c;
        sincos_reduced(x[d], &s, &c);
        u[d] = {c, -s};
        far = fmax(far, fabs(x[d]));
    }
    // one test for all of them (a NaN, which either way gives NaN, passes)
    if (far > 1e9)
        for (int d = 0; d < K; ++d)
            if (fabs(x[d]) > 1e9) {
                const double2 v = sincos_far(x[d]);
                u[d] = {v.y, -v.x};
            }
}
// FP32: the argument is reduced by whole turns with 2 pi split in three parts
// (Cody and Waite; the first two, 6.28125 and 1.9378662109375e-3, have at
// most 8 significant bits, so k times them is exact for |k| < 2^16 turns),
// the remainder in [-pi, pi] is converted to turns and given to the hardware
// sine and cosine of one turn.  Within about 3e-7 of the FP64 sine and cosine
// of the same FP32 argument for |x| < 4e5 (the library sincosf is within 7e-8
// but costs three times the instructions).  Beyond that (a link phase that
// large is a lattice long blown up) the turns are split off in FP64.
template <int K>
__device__ inline void links(float dx, const float (&a)[K], Cx<float> (&u)[K])
{
    float x[K], t[K], far = 0.f;
    for (int d = 0; d < K; ++d) {
        x[d] = dx * a[d];
        const float k = __builtin_rintf(x[d] * 0.15915494309189535f);
        float r = fm(-k, 6.28125f, x[d]);
        r = fm(-k, 1.9378662109375e-3f, r);
        r = fm(-k, -2.5590314e-6f, r);
        t[d] = r * 0.15915494309189535f;
        far = fmaxf(far, fabsf(x[d]));
    }
    if (far >= 4.0e5f)
        for (int d = 0; d < K; ++d)
            if (fabsf(x[d]) >= 4.0e5f) {
                const double w = (double)x[d] * 0.15915494309189535;
                t[d] = (float)(w - __builtin_rint(w));
            }
    for (int d = 0; d < K; ++d) u[d] = {__builtin_amdgcn_cosf(t[d]), -__builtin_amdgcn_sinf(t[d])};
}

// -Im(p conj(q)) with p = U_i^x U_j^{x+i}, q = U_i^{x+j} U_j^x: sin(Theta_ij)
template <typename R>
__device__ inline R plaq_sin(Cx<R> ui_x, Cx<R> uj_xi, Cx<R> ui_xj, Cx<R> uj_x)
{
    const Cx<R> p = cmul(ui_x, uj_xi);
    const Cx<R> q = cmul(ui_xj, uj_x);
    return fm(p.r, q.i, -(p.i * q.r));
}

// Periodic image in [0, N) of a plane within N of that range.
__device__ inline int wrapz(int z, int N)
{
    if (z < 0) return z + N;
    return z < N ? z : z - N;
}
__device__ inline int wrapi(int v, int N)
{
    // v in [-2, 2N + TX]: periodic image in [0, N)
    if (v < 0) return v + N;
    return v < N ? v : v % N;
}

// Place tiles so that the blocks the hardware sends to one XCD (block b goes
// to XCD b % 8) cover a contiguous range of tile indices.
__device__ inline int xcd_tile(int b, int nb)
{
    const int per = nb / kXcdCount, rem = nb % kXcdCount;
    const int xcd = b % kXcdCount, k = b / kXcdCount;
    return xcd * per + (xcd < rem ? xcd : rem) + k;
}

// Kick and drift of one site from the values its stencil reads (section 2):
// covariant Laplacian and potential for Pi, lattice curl of the plaquette
// field strength and current for E, Crank-Nicolson damping, then the drift.
// Own column: phi at planes z-1, z, z+1, the site's links U_j^x, the x and y
// links of the site above (x+kz), U_z^{x-kz}, and F_xz, F_yz of the site
// below (carried down the z-march).  Every kernel that steps a site calls
// this, so each site is computed by one sequence of roundings whatever the
// kernel, tile shape or schedule.
template <typename R>
struct SiteNbr {
    Cx<R> ph_xm, ph_xp, ph_ym, ph_yp;  // phi at x -/+ kx, x -/+ ky (plane z)
    Cx<R> ux_xm, uy_ym;                // U_x^{x-kx}, U_y^{x-ky}
    Cx<R> uy_xp, ux_yp, uz_xp, uz_yp;  // U_y^{x+kx}, U_x^{x+ky}, U_z^{x+kx}, U_z^{x+ky}
    Cx<R> ux_xm_yp, uy_xm, uz_xm;      // U_x^{x-kx+ky}, U_y^{x-kx}, U_z^{x-kx}
    Cx<R> ux_ym, uy_xp_ym, uz_ym;      // U_x^{x-ky}, U_y^{x+kx-ky}, U_z^{x-ky}
    Cx<R> ux_xm_zp, uy_ym_zp;          // U_x^{x-kx+kz}, U_y^{x-ky+kz}
};

template <typename R>
struct SiteCoef {
    R inv_dx, inv_dx2, sigma2, cP1, cP2, cE1, cE2, lamh, kappa, deta;
};

template <typename R>
struct SiteOut {
    R pr, pi, e[3];  // Pi^{n+1/2}, E^{n+1/2}
    Cx<R> phi;       // phi^{n+1}
    R a[3];          // A^{n+1}
    R fxz, fyz;      // F_xz, F_yz at x (the carry of the plane above)
};

// Plaquette fields of one site update (each F_ij = sin(Theta_ij) / dx^2):
// those at x, and at x - kx and x - ky, which are the neighbours' own ones.
template <typename R>
struct SiteF {
    R xy, xz, yz;           // at x
    R xy_xm, xz_xm;         // at x - kx
    R xy_ym, yz_ym;         // at x - ky
};

// The plaquettes a site forms at itself (links of planes z and z+1).
template <typename R>
__device__ __forceinline__ void own_plaquettes(const Cx<R> (&Uc)[3], Cx<R> uy_xp, Cx<R> ux_yp, Cx<R> uz_xp,
                                               Cx<R> uz_yp, Cx<R> ux_zp, Cx<R> uy_zp, R inv_dx2, R* fxy, R* fxz,
                                               R* fyz)
{
    *fxy = plaq_sin(Uc[0], uy_xp, ux_yp, Uc[1]) * inv_dx2;
    *fxz = plaq_sin(Uc[0], uz_xp, ux_zp, Uc[2]) * inv_dx2;
    *fyz = plaq_sin(Uc[1], uz_yp, uy_zp, Uc[2]) * inv_dx2;
}

// Kick and drift of one site from its neighbourhood's phi, the links of the
// Laplacian and the plaquette fields.
template <typename R>
__device__ __forceinline__ SiteOut<R> site_update_f(const SiteCoef<R>& k, Cx<R> ph_xm, Cx<R> ph_xp, Cx<R> ph_ym,
                                                    Cx<R> ph_yp, Cx<R> ux_xm, Cx<R> uy_ym, Cx<R> phi_m, Cx<R> phi_c,
                                                    Cx<R> phi_p, const Cx<R> (&Uc)[3], Cx<R> uz_m, const SiteF<R>& F,
                                                    R fxz_m, R fyz_m, R pr_c, R pi_c, const R (&e_c)[3],
                                                    const R (&a_c)[3])
{
    const R inv_dx = k.inv_dx, inv_dx2 = k.inv_dx2;
    // covariant Laplacian: sum_j U_j^x phi^{x+j} + conj(U_j^{x-j}) phi^{x-j} - 2 phi^x
    const Cx<R> fx = cmul(Uc[0], ph_xp), fy = cmul(Uc[1], ph_yp), fz = cmul(Uc[2], phi_p);
    const Cx<R> bx = cmulc(ux_xm, ph_xm), by = cmulc(uy_ym, ph_ym), bz = cmulc(uz_m, phi_m);
    const R lr = ((fx.r + bx.r) + (fy.r + by.r)) + fm(R(-6), phi_c.r, fz.r + bz.r);
    const R li = ((fx.i + bx.i) + (fy.i + by.i)) + fm(R(-6), phi_c.i, fz.i + bz.i);
    // currents J_i = Im[conj(phi) U_i phi^{x+i}] / dx
    const R jx = fm(phi_c.r, fx.i, -(phi_c.i * fx.r)) * inv_dx;
    const R jy = fm(phi_c.r, fy.i, -(phi_c.i * fy.r)) * inv_dx;
    const R jz = fm(phi_c.r, fz.i, -(phi_c.i * fz.r)) * inv_dx;
    // lattice curl C_i = sum_{j != i} (F_ij^x - F_ij^{x-j}) / dx, F_ji = -F_ij
    const R cx = ((F.xy - F.xy_ym) + (F.xz - fxz_m)) * inv_dx;
    const R cy = ((F.yz - fyz_m) - (F.xy - F.xy_xm)) * inv_dx;
    const R cz = -((F.xz - F.xz_xm) + (F.yz - F.yz_ym)) * inv_dx;
    // Crank-Nicolson kick, drift
    const R m2 = fm(phi_c.r, phi_c.r, fm(phi_c.i, phi_c.i, -k.sigma2));
    const R pot = k.lamh * m2;
    SiteOut<R> o;
    o.pr = fm(k.cP1, pr_c, k.cP2 * fm(lr, inv_dx2, -(pot * phi_c.r)));
    o.pi = fm(k.cP1, pi_c, k.cP2 * fm(li, inv_dx2, -(pot * phi_c.i)));
    o.e[0] = fm(k.cE1, e_c[0], k.cE2 * fm(k.kappa, jx, -cx));
    o.e[1] = fm(k.cE1, e_c[1], k.cE2 * fm(k.kappa, jy, -cy));
    o.e[2] = fm(k.cE1, e_c[2], k.cE2 * fm(k.kappa, jz, -cz));
    o.phi = {fm(k.deta, o.pr, phi_c.r), fm(k.deta, o.pi, phi_c.i)};
    o.a[0] = fm(k.deta, o.e[0], a_c[0]);
    o.a[1] = fm(k.deta, o.e[1], a_c[1]);
    o.a[2] = fm(k.deta, o.e[2], a_c[2]);
    o.fxz = F.xz;
    o.fyz = F.yz;
    return o;
}

// The same update forming all seven plaquettes from the neighbourhood's links.
template <typename R>
__device__ __forceinline__ SiteOut<R> site_update(const SiteCoef<R>& k, const SiteNbr<R>& n, Cx<R> phi_m, Cx<R> phi_c,
                                                  Cx<R> phi_p, const Cx<R> (&Uc)[3], Cx<R> ux_zp, Cx<R> uy_zp,
                                                  Cx<R> uz_m, R fxz_m, R fyz_m, R pr_c, R pi_c, const R (&e_c)[3],
                                                  const R (&a_c)[3])
{
    const R inv_dx2 = k.inv_dx2;
    SiteF<R> F;
    own_plaquettes(Uc, n.uy_xp, n.ux_yp, n.uz_xp, n.uz_yp, ux_zp, uy_zp, inv_dx2, &F.xy, &F.xz, &F.yz);
    F.xy_xm = plaq_sin(n.ux_xm, Uc[1], n.ux_xm_yp, n.uy_xm) * inv_dx2;
    F.xy_ym = plaq_sin(n.ux_ym, n.uy_xp_ym, Uc[0], n.uy_ym) * inv_dx2;
    F.xz_xm = plaq_sin(n.ux_xm, Uc[2], n.ux_xm_zp, n.uz_xm) * inv_dx2;
    F.yz_ym = plaq_sin(n.uy_ym, Uc[2], n.uy_ym_zp, n.uz_ym) * inv_dx2;
    return site_update_f(k, n.ph_xm, n.ph_xp, n.ph_ym, n.ph_yp, n.ux_xm, n.uy_ym, phi_m, phi_c, phi_p, Uc, uz_m, F,
                         fxz_m, fyz_m, pr_c, pi_c, e_c, a_c);
}

}  // namespace
}  // namespace ah
