// Two leapfrog steps per pass over HBM: a temporally blocked z-march for
// gfx950 (compact gauge action).
//
// The step is a memory-bound stencil (section 5 of the paper): one step
// reads 10 and writes 10 reals per site.  Here a workgroup advances its
// TX x TY tile by two steps while reading the snapshot n once and writing
// snapshot n+2 once, so HBM moves half the bytes of two single steps.
//
// Step n -> n+1 ("stage 1") is computed on the tile plus a one-site ring
// (region R1, (TX+2) x (TY+2)), which needs links and phi of snapshot n on a
// two-site ring (region R2, (TX+4) x (TY+4)).  Step n+1 -> n+2 ("stage 2")
// is computed on the tile from stage 1's values in LDS.  The workgroup walks
// its z-chunk in phases of one plane and one barrier.  Phase p is
//   - stage 1 at plane p on R1 (tile waves and ring waves);
//   - stage 2 at plane p-2 on the tile, stores of snapshot n+2;
//   - links of plane p+2 and phi of plane p+1 of snapshot n into LDS,
// with enough slots in LDS that nothing a phase writes is read before its
// barrier.  The two stages of a phase are then independent instructions of
// one wave.
//
// What bounds it: instruction issue and latency (512^3 FP32 on 64 x 8 tiles,
// one 11-wave workgroup per CU: vector ALU busy 77%; HBM 4.8 TB/s).  MI355X,
// us per step in runs of a few steps, as all comparisons here: 512^3 FP32 64 x 8
// 1283, FP64 32 x 8 3610 (1400 and 3800 over 200 steps).  Stage 2 one plane
// behind stage 1 with a barrier behind each of them (half the LDS, two
// barriers a plane) took 1677 and 4420 where this form took 1468 and 3774,
// before the values in LDS were paired (Pair, ah_stencil.h); stage 2 before stage 1 within a
// phase 1513 and 4103.
//
// Stage 1 reads Pi and E of snapshot n on the ring too, which the
// neighbouring workgroups' stage 2 would overwrite in place, so Pi and E are
// double-buffered: the pass reads (phi, A, Pi, E) from one set of buffers
// and writes all ten to the other.
//
// Each site of either stage is computed by site_update, the same sequence of
// roundings as the single-step march, so two steps here are bitwise equal
// to two single steps.
#include "ah_internal.h"
#include "ah_stencil.h"

#include <type_traits>

#pragma clang fp contract(off)

namespace ah {
namespace {

template <int TX, int TY>
struct Geom2 {
    static constexpr int W1 = TX + 2, H1 = TY + 2, S1 = W1 * H1;  // R1: tile + 1-site ring
    static constexpr int W2 = TX + 4, H2 = TY + 4, S2 = W2 * H2;  // R2: tile + 2-site ring
    static constexpr int NT = TX * TY;                            // tile threads
    static constexpr int NRING = S1 - NT;                         // R1 ring sites
    static constexpr int NTH = NT + (NRING + 63) / 64 * 64;       // threads (ring in whole waves)
    static constexpr int NOUT = S2 - S1;                          // R2 outer ring sites
    static_assert(NOUT <= NTH - NT, "one outer-ring site per ring thread at most");
};

// LDS of one workgroup.  Stage-1 links and phi live on R2, stage-2 ones on
// R1.  x and y links are kept for three planes (a phase reads two, as the
// plaquettes at x-kx and x-ky reach one plane up, and writes the third), z
// links and phi for two.
template <typename R, int TX, int TY>
struct Shared2 {
    using G = Geom2<TX, TY>;
    Pair<R, G::S2> u0[3], w0[2];  // links x, y; link z and phi
    Pair<R, G::S1> u1[3], w1[2];
    // FP64, as many as fit: stage 1's Pi, E and A of a tile site for stage 2 two
    // planes later (the rest, and FP32's, in registers)
    static constexpr int kFit = (160 * 1024 - (int)sizeof(Cx<R>) * 10 * (G::S1 + G::S2)) / (2 * (int)sizeof(R) * G::NT);
    static constexpr int HELD = sizeof(R) == 8 ? (kFit < 8 ? kFit : 8) : 0;
    R h[2][HELD > 0 ? HELD : 8][HELD > 0 ? G::NT : 1];
    // FP64 where not all of them fit (64 x 4): U_z and phi of the own column are
    // read back from the slots that the phase is about to write, where they are
    // until then, and not carried in registers.  With Pi, E and A in registers
    // and the column carried as well the pass spilled ten values a plane (MI355X,
    // us per step: 512^3 6490, 5310 now; 256^3 784, 645; 128^3 105, 86).
    static constexpr bool LEAN = sizeof(R) == 8 && HELD < 8;
};

template <typename R>
struct Step2Args {
    Blocks<R> b;  // snapshots n (read) and n+2 (written)
    int N, P;  // side, row pitch: site (x, y, z) at x + P (y + N z)
    SiteCoef<R> k0, k1;  // coefficients of steps n and n+1
    R dx;
};

// Neighbourhood of the site at index c of a region of width W whose links
// (x, y, z of plane z; x, y of plane z+1) and phi (plane z) are in LDS.
template <int W, typename R, int S>
__device__ __forceinline__ SiteNbr<R> gather_nbr(int c, const Pair<R, S>& u, const Pair<R, S>& w, const Pair<R, S>& up)
{
    SiteNbr<R> n;
    w.get(c - 1, &n.uz_xm, &n.ph_xm);
    w.get(c + 1, &n.uz_xp, &n.ph_xp);
    w.get(c - W, &n.uz_ym, &n.ph_ym);
    w.get(c + W, &n.uz_yp, &n.ph_yp);
    u.get(c - 1, &n.ux_xm, &n.uy_xm);
    u.get(c - W, &n.ux_ym, &n.uy_ym);
    n.uy_xp = u.get(c + 1, 1);
    n.ux_yp = u.get(c + W, 0);
    n.ux_xm_yp = u.get(c - 1 + W, 0);
    n.uy_xp_ym = u.get(c + 1 - W, 1);
    n.ux_xm_zp = up.get(c - 1, 0);
    n.uy_ym_zp = up.get(c - W, 1);
    return n;
}

template <int TX, int TY>
constexpr int kStep2Threads = Geom2<TX, TY>::NTH;
// Waves per SIMD the register allocation leaves room for: FP64 two (it takes
// 255 registers on 32 x 8); FP32 three (149 registers: one 11-wave 64 x 8 or
// 7-wave 64 x 4, or two 6-wave 32 x 8 workgroups per CU).
template <typename R, int TX, int TY>
constexpr int kStep2MinWaves = sizeof(R) == 8 ? 2 : 3;

// Two steps of planes [z0, z1) of the tile whose lower corner is (x0, y0), as
// the waves that own tile sites (TILE) or ring sites run them.  All threads of
// the workgroup call this with the same arguments but TILE, which is the same
// for every lane of a wave; both kinds pass the same barriers.
template <typename R, int TX, int TY, bool TILE>
__device__ __forceinline__ void march2_role(Shared2<R, TX, TY>& sh, const Step2Args<R>& a, int x0, int y0, int z0,
                                            int z1)
{
    using G = Geom2<TX, TY>;
    constexpr int W1 = G::W1, H1 = G::H1, W2 = G::W2, H2 = G::H2, NT = G::NT;

    const int N = a.N, P = a.P;
    const int64_t NN = (int64_t)N * P;  // plane stride
    const uint32_t pb = (uint32_t)NN * (uint32_t)sizeof(R);  // bytes of a plane (N P < 2^28)
    const R dx = a.dx;
    // 1/dx and 1/dx^2 formed on the device as the single-step march forms them
    SiteCoef<R> k0 = a.k0, k1 = a.k1;
    k0.inv_dx = k1.inv_dx = R(1) / dx;
    k0.inv_dx2 = k1.inv_dx2 = k0.inv_dx * k0.inv_dx;

    // ---- roles: every thread has an R1 position (stage 1); a tile thread
    //      also owns the stage-2 site there, a ring thread also one R2 outer
    //      site.  The lanes left over in the last ring wave repeat its last
    //      sites (the same values into the same slots).
    const int tid = threadIdx.x;
    int rx, ry, ox = 0, oy = 0;
    if constexpr (TILE) {
        rx = tid % TX + 1;
        ry = tid / TX + 1;
    } else {
        const int r = min(tid - NT, G::NRING - 1);
        if (r < W1) {
            rx = r;
            ry = 0;
        } else if (r < 2 * W1) {
            rx = r - W1;
            ry = H1 - 1;
        } else if (r < 2 * W1 + TY) {
            rx = 0;
            ry = 1 + (r - 2 * W1);
        } else {
            rx = W1 - 1;
            ry = 1 + (r - 2 * W1 - TY);
        }
        const int o = min(tid - NT, G::NOUT - 1);
        if (o < W2) {
            ox = o;
            oy = 0;
        } else if (o < 2 * W2) {
            ox = o - W2;
            oy = H2 - 1;
        } else if (o < 2 * W2 + (H2 - 2)) {
            ox = 0;
            oy = 1 + (o - 2 * W2);
        } else {
            ox = W2 - 1;
            oy = 1 + (o - 2 * W2 - (H2 - 2));
        }
    }
    int c1 = rx + W1 * ry;                    // R1 index of the stage-1 site
    int c2 = (rx + 1) + W2 * (ry + 1);        // its R2 index
    const int co = ox + W2 * oy;              // R2 index of the outer site
    // byte offsets in a plane: of the stage-1 site, of the outer site, and for
    // the stores (kNoSite for lanes past a ragged edge)
    const uint32_t ob = ((uint32_t)wrapi(x0 - 1 + rx, N) + (uint32_t)P * (uint32_t)wrapi(y0 - 1 + ry, N)) *
                        (uint32_t)sizeof(R);
    const uint32_t oo = ((uint32_t)wrapi(x0 - 2 + ox, N) + (uint32_t)P * (uint32_t)wrapi(y0 - 2 + oy, N)) *
                        (uint32_t)sizeof(R);
    const uint32_t so = x0 + rx - 1 < N && y0 + ry - 1 < N ? ob : kNoSite;

    auto plane_of = [&](int z) -> int64_t { return (int64_t)wrapz(z, N) * NN; };
    auto in_p = [&](int64_t plane) { return plane_bufs(a.b.ip, a.b.fs, plane, pb); };
    auto in_m = [&](int64_t plane) { return plane_bufs(a.b.im, a.b.fs, plane, pb); };
    auto ld = [](Rsrc r, uint32_t off) -> R { return ld_plane<R>(r, off); };

    // ---- stage-1 column state (snapshot n at the stage-1 site).  The
    //      site's own links of planes p and p+1 are read back from LDS.
    R ac[3], ap[3];      // A at planes p, p+1
    Cx<R> upz;           // U_z at plane p+1 (into LDS during phase p)
    Cx<R> uz_m;          // U_z at plane p-1
    R fxz_m, fyz_m;      // F_xz, F_yz at plane p-1
    Cx<R> phm, phc, php; // phi at planes p-1, p, p+1
    R pr, pi, e[3];      // Pi, E at plane p
    Cx<R> uo_z = {};     // outer site: U_z of plane p+1
    // ---- stage-2 column state (snapshot n+1 at the tile site)
    constexpr int HELD = Shared2<R, TX, TY>::HELD;
    constexpr bool LEAN = Shared2<R, TX, TY>::LEAN;
    R hr[2][8];              // Pi, E, A of planes p-1, p-2, by parity: those not held in LDS
    auto h = [&](int b, int k) -> R& {
        if (k >= 8 - HELD)
            return sh.h[b][HELD > 0 ? k - (8 - HELD) : 0][TILE && HELD > 0 ? tid : 0];
        else
            return hr[b][k];
    };
    Cx<R> vz_m = {};         // U_z^{n+1} at q-1
    R gxz_m = 0, gyz_m = 0;  // F^{n+1}_xz, F^{n+1}_yz at q-1
    Cx<R> chm = {};          // phi^{n+1} at q-1
    // stage-1 phi and U_z of plane p-1, into LDS during phase p
    Cx<R> s1phi = {}, s1z = {};

    // Operands loaded one iteration ahead: A of plane p+2 (stage-1 site and
    // outer site), phi of plane p+2 (stage-1 site) and p+1 (outer site), Pi
    // and E of plane p+1 (stage-1 site).
    R na[3], noa[3] = {0, 0, 0}, npr, npi, ne[3];
    Cx<R> nph, noph = {};
    auto prefetch = [&](int p) {
        const int64_t p1 = plane_of(p + 1);
        const PlaneBufs f2 = in_p(plane_of(p + 2));
        for (int d = 0; d < 3; ++d) na[d] = ld(f2.f[B_A + d], ob);
        if constexpr (!TILE) {
            for (int d = 0; d < 3; ++d) noa[d] = ld(f2.f[B_A + d], oo);
            const PlaneBufs f1 = in_p(p1);
            noph = Cx<R>{ld(f1.f[B_PHR], oo), ld(f1.f[B_PHI], oo)};
        }
        nph = Cx<R>{ld(f2.f[B_PHR], ob), ld(f2.f[B_PHI], ob)};
        const PlaneBufs m1 = in_m(p1);
        npr = ld(m1.f[B_PIR], ob);
        npi = ld(m1.f[B_PII], ob);
        for (int d = 0; d < 3; ++d) ne[d] = ld(m1.f[B_E + d], ob);
    };

    // ------------------------------------------------------------ prologue
    // Every load of the prologue, and those of the first iteration, are
    // issued before its first barrier: a chunk then starts with one round of
    // memory latency.
    {
        const int64_t pm2 = plane_of(z0 - 2), pm1 = plane_of(z0 - 1), p0 = plane_of(z0);
        R am2[3], om[7] = {0, 0, 0, 0, 0, 0, 0};  // om: A_z at z0-2, A at z0-1, A at z0 of the outer site
        Cx<R> oph = {};
        const PlaneBufs fm2 = in_p(pm2), fm1 = in_p(pm1), f0 = in_p(p0), mm1 = in_m(pm1);
        for (int d = 0; d < 3; ++d) am2[d] = ld(fm2.f[B_A + d], ob);
        for (int d = 0; d < 3; ++d) ac[d] = ld(fm1.f[B_A + d], ob);
        for (int d = 0; d < 3; ++d) ap[d] = ld(f0.f[B_A + d], ob);
        if constexpr (!TILE) {
            om[0] = ld(fm2.f[B_A + 2], oo);
            for (int d = 0; d < 3; ++d) om[1 + d] = ld(fm1.f[B_A + d], oo);
            for (int d = 0; d < 3; ++d) om[4 + d] = ld(f0.f[B_A + d], oo);
            oph = Cx<R>{ld(fm1.f[B_PHR], oo), ld(fm1.f[B_PHI], oo)};
        }
        phm = Cx<R>{ld(fm2.f[B_PHR], ob), ld(fm2.f[B_PHI], ob)};
        phc = Cx<R>{ld(fm1.f[B_PHR], ob), ld(fm1.f[B_PHI], ob)};
        php = Cx<R>{ld(f0.f[B_PHR], ob), ld(f0.f[B_PHI], ob)};
        pr = ld(mm1.f[B_PIR], ob);
        pi = ld(mm1.f[B_PII], ob);
        for (int d = 0; d < 3; ++d) e[d] = ld(mm1.f[B_E + d], ob);
        prefetch(z0 - 1);

        // planes z0-1 and z0: x, y links into slots 0 and 1; U_z and phi of
        // z0-1 into slot 0, U_z of z0-2 (for F^n there) into slot 1
        Cx<R> um2[3], uc[3], up[3];
        links(dx, am2, um2);
        if constexpr (LEAN)
            sh.w0[1].set(c2, um2[2], phm);
        else
            sh.w0[1].at(c2, 0) = um2[2];
        uz_m = um2[2];
        links(dx, ac, uc);
        sh.u0[0].set(c2, uc[0], uc[1]);
        sh.w0[0].set(c2, uc[2], phc);
        links(dx, ap, up);
        sh.u0[1].set(c2, up[0], up[1]);
        upz = up[2];
        if constexpr (!TILE) {
            Cx<R> uo[7];
            links(dx, om, uo);
            sh.w0[1].at(co, 0) = uo[0];
            sh.u0[0].set(co, uo[1], uo[2]);
            sh.w0[0].set(co, uo[3], oph);
            sh.u0[1].set(co, uo[4], uo[5]);
            uo_z = uo[6];
        }
        __syncthreads();
        // F^n_xz, F^n_yz at z0-2 of the stage-1 site
        fxz_m = plaq_sin(um2[0], sh.w0[1].get(c2 + 1, 0), uc[0], um2[2]) * k0.inv_dx2;
        fyz_m = plaq_sin(um2[1], sh.w0[1].get(c2 + W2, 0), uc[1], um2[2]) * k0.inv_dx2;
        __syncthreads();
    }

    // Slots of the x and y links: planes p, p+1 and p+2 of snapshot n, and
    // planes p, p-2 and p-1 of snapshot n+1.
    int sa = 0, sb = 1, sc = 2;

    // Phase p: stage 1 at plane p (S1), stage 2 at plane q = p-2 (S2).  What
    // it writes to LDS, no wave reads before the barrier that ends it.
    // `par`: the parity of p - (z0-1), the slot of planes p and p-2 where
    // there are two.
    auto phase = [&](auto par, auto s1, auto s2, int p) __attribute__((always_inline)) {
        constexpr int b = decltype(par)::value;
        constexpr bool S1 = decltype(s1)::value, S2 = decltype(s2)::value && TILE;
        const bool more = p < z1;  // there is a stage 1 in the next phase
        // the LDS addresses anew in each phase, rather than some thirty of
        // them held in registers through the march (149 registers, not spills)
        asm volatile("" : "+v"(c1), "+v"(c2));
        if (S1 && more && p > z0 - 1) prefetch(p);

        const Cx<R> phq = s1phi;  // phi^{n+1} of plane p-1 = q+1
        if constexpr (LEAN && S2) sh.w1[b ^ 1].get(c1, &vz_m, &chm);
        sh.w1[b ^ 1].set(c1, s1z, s1phi);
        SiteOut<R> o1 = {}, o2 = {};
        Cx<R> u1[3];
        if constexpr (S1) {
            Cx<R> uc[3], upx, upy;
            sh.u0[sa].get(c2, &uc[0], &uc[1]);
            if constexpr (LEAN) {
                sh.w0[b ^ 1].get(c2, &uz_m, &phm);
                sh.w0[b].get(c2, &uc[2], &phc);
            } else {
                uc[2] = sh.w0[b].get(c2, 0);
            }
            sh.u0[sb].get(c2, &upx, &upy);
            const SiteNbr<R> nb = gather_nbr<W2>(c2, sh.u0[sa], sh.w0[b], sh.u0[sb]);
            o1 = site_update(k0, nb, phm, phc, php, uc, upx, upy, uz_m, fxz_m, fyz_m, pr, pi, e, ac);
            fxz_m = o1.fxz;
            fyz_m = o1.fyz;
            uz_m = uc[2];
            links(dx, o1.a, u1);
            sh.u1[sa].set(c1, u1[0], u1[1]);
            s1phi = o1.phi;
            s1z = u1[2];
        }
        if constexpr (S2) {
            Cx<R> vc[3], chc, vpx, vpy;
            sh.u1[sb].get(c1, &vc[0], &vc[1]);
            sh.w1[b].get(c1, &vc[2], &chc);
            sh.u1[sc].get(c1, &vpx, &vpy);
            const R qe[3] = {h(b, 2), h(b, 3), h(b, 4)}, qa[3] = {h(b, 5), h(b, 6), h(b, 7)};
            const SiteNbr<R> nb = gather_nbr<W1>(c1, sh.u1[sb], sh.w1[b], sh.u1[sc]);
            o2 = site_update(k1, nb, chm, chc, phq, vc, vpx, vpy, vz_m, gxz_m, gyz_m, h(b, 0), h(b, 1), qe, qa);
            gxz_m = o2.fxz;
            gyz_m = o2.fyz;
            vz_m = vc[2];
            chm = chc;
            // plane z0-1 only starts the carry (F^{n+1}_xz, F^{n+1}_yz, U_z,
            // phi): its stores are dropped
            const int q = p - 2 < z0 ? z0 : p - 2;
            const uint32_t off = p - 2 < z0 ? kNoSite : so;
            const int64_t oq = (int64_t)q * NN;
            const PlaneBufs wm = plane_bufs(a.b.om, a.b.fs, oq, pb), wp = plane_bufs(a.b.op, a.b.fs, oq, pb);
            st_plane(wm.f[B_PIR], off, o2.pr);
            st_plane(wm.f[B_PII], off, o2.pi);
            for (int d = 0; d < 3; ++d) st_plane(wm.f[B_E + d], off, o2.e[d]);
            st_plane(wp.f[B_PHR], off, o2.phi.r);
            st_plane(wp.f[B_PHI], off, o2.phi.i);
            for (int d = 0; d < 3; ++d) st_plane(wp.f[B_A + d], off, o2.a[d]);
        }
        if constexpr (S1) {
            if constexpr (TILE) {
                h(b, 0) = o1.pr;
                h(b, 1) = o1.pi;
                for (int d = 0; d < 3; ++d) {
                    h(b, 2 + d) = o1.e[d];
                    h(b, 5 + d) = o1.a[d];
                }
            }
            if (more) {
                // stage-1 operands of the next phase: U_z and phi of plane
                // p+1, links of plane p+2 (U_z held)
                sh.w0[b ^ 1].set(c2, upz, php);
                Cx<R> un[3];
                links(dx, na, un);
                sh.u0[sc].set(c2, un[0], un[1]);
                upz = un[2];
                if constexpr (!TILE) {
                    sh.w0[b ^ 1].set(co, uo_z, noph);
                    links(dx, noa, un);
                    sh.u0[sc].set(co, un[0], un[1]);
                    uo_z = un[2];
                }
                for (int d = 0; d < 3; ++d) {
                    ac[d] = ap[d];
                    ap[d] = na[d];
                    e[d] = ne[d];
                }
                phm = phc;
                phc = php;
                php = nph;
                pr = npr;
                pi = npi;
            }
            __syncthreads();
            const int t = sa;
            sa = sb;
            sb = sc;
            sc = t;
        }
    };
    const std::integral_constant<int, 0> even;
    const std::integral_constant<int, 1> odd;
    const std::true_type yes;
    const std::false_type no;
    phase(even, yes, no, z0 - 1);
    phase(odd, yes, no, z0);
    for (int p = z0 + 1;; p += 2) {
        phase(even, yes, yes, p);
        if (p == z1) {
            phase(odd, no, yes, p + 1);
            break;
        }
        phase(odd, yes, yes, p + 1);
        if (p + 1 == z1) {
            phase(even, no, yes, p + 2);
            break;
        }
    }
}

template <typename R, int TX, int TY>
__device__ __forceinline__ void march2(Shared2<R, TX, TY>& sh, const Step2Args<R>& a, int x0, int y0, int z0, int z1)
{
    static_assert(Geom2<TX, TY>::NT % 64 == 0, "a wave is of one kind");
    if (uniform((int)threadIdx.x) < Geom2<TX, TY>::NT)
        march2_role<R, TX, TY, true>(sh, a, x0, y0, z0, z1);
    else
        march2_role<R, TX, TY, false>(sh, a, x0, y0, z0, z1);
}

// One lattice: tile t = xcd_tile(b) (tx fastest, then ty, then z-chunk).
template <typename R, int TX, int TY>
__global__ void __launch_bounds__((kStep2Threads<TX, TY>), (kStep2MinWaves<R, TX, TY>))
    k_step2_tile(Step2Args<R> a, int zchunk, int tiles_x, int tiles_y)
{
    __shared__ Shared2<R, TX, TY> sh;
    int t = xcd_tile(blockIdx.x, gridDim.x);
    const int x0 = (t % tiles_x) * TX;
    t /= tiles_x;
    const int y0 = (t % tiles_y) * TY;
    const int z0 = (t / tiles_y) * zchunk;
    const int z1 = (z0 + zchunk < a.N) ? z0 + zchunk : a.N;
    march2<R, TX, TY>(sh, a, x0, y0, z0, z1);
}

// Pool lattices that take a two-step pass at their step k (two_step_due):
// one block per (lattice, tile) work item, XCD x the x-th eighth of the list
// as in the single-step batch kernel; snapshot k of the current buffers to
// snapshot k+2 in the other ones, with the coefficients of rows k and k+1 of
// the lattice's table.
template <typename R, int TX, int TY>
__global__ void __launch_bounds__((kStep2Threads<TX, TY>), (kStep2MinWaves<R, TX, TY>))
    k_step2_batch(const PoolLattice* __restrict__ lat, const WorkItem* __restrict__ work, int nwork)
{
    __shared__ Shared2<R, TX, TY> sh;
    const WorkItem it = work[xcd_tile(blockIdx.x, nwork)];
    if (it.lattice < 0) return;
    const PoolLattice& L = lat[it.lattice];
    const int64_t k = L.counter[0];
    if (!two_step_due(L, k)) return;  // uniform across the block
    const int cur = (int)L.counter[2], curm = (int)L.counter[3];
    Step2Args<R> a;
    a.b = Blocks<R>{(const R*)L.pp[cur], (const R*)L.mom[curm], (R*)L.pp[cur ^ 1], (R*)L.mom[curm ^ 1], L.fs};
    a.N = L.N;
    a.P = L.P;
    a.dx = (R)L.dx;
    const double* row = L.coef + k * kCoefStride;
    for (int j = 0; j < 2; ++j, row += kCoefStride) {
        SiteCoef<R>& c = j ? a.k1 : a.k0;
        c.inv_dx = c.inv_dx2 = R(0);  // formed in the march
        c.sigma2 = (R)L.sigma2;
        c.cP1 = (R)row[C_P1];
        c.cP2 = (R)row[C_P2];
        c.cE1 = (R)row[C_E1];
        c.cE2 = (R)row[C_E2];
        c.lamh = (R)row[C_LAMH];
        c.kappa = (R)row[C_KAPPA];
        c.deta = (R)L.deta;
    }
    a = uniform(a);
    int t = it.tile;
    const int x0 = uniform((t % L.two_tiles_x) * TX);
    t /= L.two_tiles_x;
    const int y0 = uniform((t % L.two_tiles_y) * TY);
    const int z0 = uniform((t / L.two_tiles_y) * L.two_zchunk);
    const int z1 = uniform((z0 + L.two_zchunk < L.N) ? z0 + L.two_zchunk : L.N);
    march2<R, TX, TY>(sh, a, x0, y0, z0, z1);
}

}  // namespace

template <typename R>
hipError_t launch_step2_tile(const Fields<R>& in, const Fields<R>& out, const LatticeConst& L, const StepCoef& c0,
                             const StepCoef& c1, const TileConfig& tc, hipStream_t s)
{
    const int N = L.N;
    Step2Args<R> a;
    if (!blocks_of(in, out, &a.b)) return hipErrorInvalidValue;
    a.N = N;
    a.P = L.P;
    a.dx = (R)L.dx;
    for (int j = 0; j < 2; ++j) {
        const StepCoef& c = j ? c1 : c0;
        SiteCoef<R>& k = j ? a.k1 : a.k0;
        k.inv_dx = k.inv_dx2 = R(0);  // formed in the kernel
        k.sigma2 = (R)L.sigma2;
        k.cP1 = (R)c.cP1;
        k.cP2 = (R)c.cP2;
        k.cE1 = (R)c.cE1;
        k.cE2 = (R)c.cE2;
        k.lamh = (R)c.lam_half;
        k.kappa = (R)c.kappa;
        k.deta = (R)L.deta;
    }
    const int zc = tc.zchunk > 0 ? tc.zchunk : N;
#define AH_STEP2_CASE(TXv, TYv)                                                                                   \
    if (tc.tx == TXv && tc.ty == TYv) {                                                                           \
        const int tiles_x = (N + TXv - 1) / TXv, tiles_y = (N + TYv - 1) / TYv;                                  \
        const int nb = tiles_x * tiles_y * ((N + zc - 1) / zc);                                                  \
        hipLaunchKernelGGL((k_step2_tile<R, TXv, TYv>), dim3(nb), dim3(Geom2<TXv, TYv>::NTH), 0, s, a, zc,       \
                           tiles_x, tiles_y);                                                                     \
        return hipGetLastError();                                                                                \
    }
    AH_STEP2_CASE(32, 8)
    AH_STEP2_CASE(64, 4)
    if constexpr (sizeof(R) == 4) {
        AH_STEP2_CASE(64, 8)  // FP64 would need more LDS than a CU has
    }
#undef AH_STEP2_CASE
    return hipErrorInvalidValue;
}

template <typename R>
hipError_t launch_step2_batch(const PoolLattice* lat, const WorkItem* work, int nwork, int tx, int ty, int grid,
                              hipStream_t s)
{
    if (!tile2_supported(sizeof(R) == 8 ? AH_FP64 : AH_FP32, tx, ty)) return hipErrorInvalidValue;
#define AH_STEP2_BATCH_CASE(TXv, TYv)                                                                             \
    if (tx == TXv && ty == TYv) {                                                                                 \
        hipLaunchKernelGGL((k_step2_batch<R, TXv, TYv>), dim3(grid), dim3(Geom2<TXv, TYv>::NTH), 0, s, lat, work, \
                           nwork);                                                                                \
        return hipGetLastError();                                                                                 \
    }
    AH_STEP2_BATCH_CASE(32, 8)
    AH_STEP2_BATCH_CASE(64, 4)
    if constexpr (sizeof(R) == 4) {
        AH_STEP2_BATCH_CASE(64, 8)
    }
#undef AH_STEP2_BATCH_CASE
    return hipErrorInvalidValue;
}
template hipError_t launch_step2_batch<double>(const PoolLattice*, const WorkItem*, int, int, int, int, hipStream_t);
template hipError_t launch_step2_batch<float>(const PoolLattice*, const WorkItem*, int, int, int, int, hipStream_t);

template hipError_t launch_step2_tile<double>(const Fields<double>&, const Fields<double>&, const LatticeConst&,
                                              const StepCoef&, const StepCoef&, const TileConfig&, hipStream_t);
template hipError_t launch_step2_tile<float>(const Fields<float>&, const Fields<float>&, const LatticeConst&,
                                             const StepCoef&, const StepCoef&, const TileConfig&, hipStream_t);

}  // namespace ah
