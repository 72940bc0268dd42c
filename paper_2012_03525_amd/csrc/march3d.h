// 3D single-phase SMAME step as a register march along z: a wave owns a
// window of 64 VX columns of RY neighbouring x rows and marches them through a
// chunk of planes; no LDS and no barrier.  FP32, rho0 = 1, any faces, with
// (FST) or without the two-phase force.
//
// What bounds it and why this layout.  On grids that stay in the caches
// (below about 200^3) the LDS-staged column march spends its time in
// barriers and LDS latency: with two to four workgroups per CU each plane is
// a chain of load, barrier, drho', barrier, momentum.  Here every wave runs
// on its own: x neighbours come from the adjacent lane (DPP), the planes
// below and above are registers, and the rows beside its own are loaded by
// the wave itself (they are in L2: RY + 4 rows of drho and v, RY + 2 of u and w
// for RY rows out), so the price of having no exchange is (RY + 2) / RY times
// the drho' work, about a fifth of the momentum's.  The values are formed by
// the expressions of step3d.h in the same order.  It is bound by instruction
// issue: 160 VALU instructions per node for RY = 2, 145 for RY = 4, and the
// four planes of lead-in of every chunk.  Against the column march, per step:
// 200 x 99 x 70 duct 26.7 -> 20.4 us, 256 x 100 x 80 cavity 33.6 -> 27, 100^3
// periodic 21.2 -> 15.2, 200 x 200 x 160 periodic 75 -> 54.
//
// Ghosts: a row or plane beyond a walled face is its mirror with the face's
// velocity rule, drho' there is the mirror's; beyond an x face the neighbour
// of the outermost node is formed from that node.  Only ghosts beyond one
// face are ever read.
#pragma once

#include "march2d.h"
#include "step3d.h"

namespace acm {
namespace march {

template <typename T, int VX, int RY>
struct Planes {
    // by plane modulo 6; rows y0 - 2 .. y0 + RY + 1 of drho and v, y0 - 1 .. y0 + RY of u and w
    T r[6][RY + 4][VX], u[6][RY + 2][VX], v[6][RY + 4][VX], w[6][RY + 2][VX];
    // by plane modulo 3, rows y0 - 1 .. y0 + RY: drho'
    T rn[3][RY + 2][VX];
    T gr[3][RY][VX];        // drho_E - drho_W of the own rows
    T fs[2][3][RY][VX];     // surface-tension force phi G_iso mu, by plane modulo 2
};

// RY rows from y0 of planes z0 .. z1 - 1 on the window starting at column xs;
// lanes l0 .. l1 - 1 store.
template <typename T, int VX, int RY, bool WX, bool WYZ, bool FST>
__device__ __forceinline__ void run3(const Coef<T>& c, const State<T>& in, const State<T>& out, int xs, int l0, int l1,
                                     int y0, int z0, int z1)
{
    const int nx = c.nx, ny = c.ny, nz = c.nz, lane = threadIdx.x & 63;
    const bool wallx = WX && c.bc[0] != BC_PERIODIC, wally = WYZ && c.bc[2] != BC_PERIODIC,
               wallz = WYZ && c.bc[4] != BC_PERIODIC;
    const unsigned pitch = (unsigned)nx * (unsigned)sizeof(T), pbytes = pitch * (unsigned)ny,
                   fbytes = pbytes * (unsigned)nz;
    int x = xs + VX * lane;
    if (wallx) {
        x = min(x, nx - VX);  // lanes past a short row repeat its last nodes
    } else {
        x = x < 0 ? x + nx : (x >= nx ? x - nx : x);
        if (x < 0 || x >= nx) x = ((x % nx) + nx) % nx;
    }
    const unsigned loff = (unsigned)x * (unsigned)sizeof(T);
    const bool st = lane >= l0 && lane < l1;
    Edge<T> eg;
    eg.l = wallx && xs == 0 && lane == 0;
    eg.r = wallx && xs + VX * (lane + 1) == nx;
    eg.any = wallx && (xs == 0 || xs + 64 * VX >= nx);
    T egw[2] = {T(0), T(0)};  // the x face's rule for w
    if (WX) {
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            eg.s[a] = eg.l ? c.fs[0][a] : c.fs[1][a];
            eg.o[a] = eg.l ? c.fo[0][a] : c.fo[1][a];
        }
        egw[0] = eg.l ? c.fs[0][2] : c.fs[1][2];
        egw[1] = eg.l ? c.fo[0][2] : c.fo[1][2];
    }
    // byte offsets within a plane of the rows y0 - 2 .. y0 + RY + 1, taken inside the grid
    unsigned yoff[RY + 4];
#pragma unroll
    for (int i = 0; i < RY + 4; ++i) {
        int y = y0 - 2 + i;
        if (wally) {
            y = y < 0 ? -1 - y : (y >= ny ? 2 * ny - 1 - y : y);  // the mirror row
            y = min(max(y, 0), ny - 1);                           // (rows further out are not used)
        } else {
            y = y < 0 ? y + ny : (y >= ny ? y - ny : y);
            if (y < 0 || y >= ny) y = ((y % ny) + ny) % ny;
        }
        yoff[i] = (unsigned)y * pitch;
    }
    T gx[RY];
#pragma unroll
    for (int i = 0; i < RY; ++i) {
        gx[i] = c.gdt[0];
        if (c.fx) gx[i] = fmaT(c.dt, c.fx[min(y0 + i, ny - 1)], gx[i]);
    }

    const __amdgpu_buffer_rsrc_t ir = field_rsrc(in.r, fbytes), iu = field_rsrc(in.u, fbytes),
                                 iv = field_rsrc(in.v, fbytes), iw = field_rsrc(in.w, fbytes);
    const __amdgpu_buffer_rsrc_t qr = field_rsrc(out.r, fbytes), qu = field_rsrc(out.u, fbytes),
                                 qv = field_rsrc(out.v, fbytes), qw = field_rsrc(out.w, fbytes);
    Planes<T, VX, RY> P;
    // plane p (possibly one outside the grid) into ring slot sl
    auto plane_in = [&](int p) {
        if (wallz) return min(max(p, 0), nz - 1);
        p = p < 0 ? p + nz : (p >= nz ? p - nz : p);
        return (p < 0 || p >= nz) ? ((p % nz) + nz) % nz : p;
    };
    auto fetch = [&](int p, auto slot) {
        constexpr int sl = decltype(slot)::value;
        const unsigned pz = (unsigned)plane_in(p) * pbytes;
#pragma unroll
        for (int i = 0; i < RY + 4; ++i) {
            row_load<T, VX>(P.r[sl][i], ir, loff, pz + yoff[i]);
            row_load<T, VX>(P.v[sl][i], iv, loff, pz + yoff[i]);
        }
#pragma unroll
        for (int i = 0; i < RY + 2; ++i) {
            row_load<T, VX>(P.u[sl][i], iu, loff, pz + yoff[i + 1]);
            row_load<T, VX>(P.w[sl][i], iw, loff, pz + yoff[i + 1]);
        }
    };
    // the force of plane p, used when plane p + 2 has arrived
    auto fetch_force = [&](int p, auto slot) {
        if constexpr (FST) {
            constexpr int sl = decltype(slot)::value;
            const unsigned pz = (unsigned)plane_in(p) * pbytes;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const __amdgpu_buffer_rsrc_t f = field_rsrc(c.fst[a], fbytes);
#pragma unroll
                for (int i = 0; i < RY; ++i) row_load<T, VX>(P.fs[sl][a][i], f, loff, pz + yoff[i + 2]);
            }
        }
    };
    // the velocity rule of face f on row i of plane slot sl (u, w rows shifted by one)
    auto rule = [&](int f, auto slot, int i) {
        constexpr int sl = decltype(slot)::value;
#pragma unroll
        for (int j = 0; j < VX; ++j) {
            P.v[sl][i][j] = fmaT(c.fs[f][1], P.v[sl][i][j], c.fo[f][1]);
            if (i >= 1 && i < RY + 3) {
                P.u[sl][i - 1][j] = fmaT(c.fs[f][0], P.u[sl][i - 1][j], c.fo[f][0]);
                P.w[sl][i - 1][j] = fmaT(c.fs[f][2], P.w[sl][i - 1][j], c.fo[f][2]);
            }
        }
    };

    const int nb = wallz ? max(z0 - 2, -1) : z0 - 2;  // first plane pushed
    const int ne = z1 + 1;                            // last
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int i = 0; i < RY + 4; ++i)
#pragma unroll
            for (int j = 0; j < VX; ++j) {
                P.r[q][i][j] = P.v[q][i][j] = T(0);
                if (i < RY + 2) P.u[q][i][j] = P.w[q][i][j] = T(0);
                if (q < 3 && i < RY + 2) P.rn[q][i][j] = T(0);
                if (q < 3 && i < RY) P.gr[q][i][j] = T(0);
            }
    fetch(nb, std::integral_constant<int, 0>{});
    fetch_force(nb - 2, std::integral_constant<int, 0>{});

    // plane n = nb + i has arrived (slot J = i mod 6): drho' of plane n - 1, the new state of plane n - 2
    auto iterate = [&](int nn, auto jc) {
        constexpr int J = decltype(jc)::value;
        constexpr int n = J % 6, k = (J + 5) % 6, m = (J + 4) % 6, s = (J + 3) % 6;
        constexpr int dk = (J + 2) % 3, dm = (J + 1) % 3, ds = J % 3;
        fetch(nn + 1, std::integral_constant<int, (J + 1) % 6>{});  // (two planes ahead measured the same)
        fetch_force(nn - 1, std::integral_constant<int, (J + 1) % 2>{});
        if (WYZ) {
            if (wally) {
#pragma unroll
                for (int i = 0; i < RY + 4; ++i) {
                    if (y0 - 2 + i == -1) rule(2, std::integral_constant<int, n>{}, i);
                    if (y0 - 2 + i == ny) rule(3, std::integral_constant<int, n>{}, i);
                }
            }
            if (wallz && (nn == -1 || nn == nz)) {
                const int f = nn == -1 ? 4 : 5;
#pragma unroll
                for (int i = 0; i < RY + 4; ++i) rule(f, std::integral_constant<int, n>{}, i);
            }
        }
        const bool mom = nn - 2 >= z0;
        T ro[RY][VX], uo[RY][VX], vo[RY][VX], wo[RY][VX];
        if (nn - 1 >= z0 - 1) {
            // drho' of plane n - 1 on rows y0 - 1 .. y0 + RY
#pragma unroll
            for (int i = 0; i < RY + 2; ++i) {
                T rE[VX], rW[VX], uE[VX], uW[VX];
                const T(&r)[VX] = P.r[k][i + 1];
                const T(&u)[VX] = P.u[k][i];
                east_west(r, rE, rW);
                east_west(u, uE, uW);
                if (WX && eg.any) {
                    const T gr = eg.l ? r[0] : r[VX - 1];
                    const T gu = fmaT(eg.s[0], eg.l ? u[0] : u[VX - 1], eg.o[0]);
                    rW[0] = eg.l ? gr : rW[0];
                    uW[0] = eg.l ? gu : uW[0];
                    rE[VX - 1] = eg.r ? gr : rE[VX - 1];
                    uE[VX - 1] = eg.r ? gu : uE[VX - 1];
                }
#pragma unroll
                for (int j = 0; j < VX; ++j) {
                    P.rn[dk][i][j] = rho_new_pt<false, T>(c, r[j], rE[j], uE[j], rW[j], uW[j], P.r[k][i + 2][j],
                                                          P.v[k][i + 2][j], P.r[k][i][j], P.v[k][i][j],
                                                          P.r[n][i + 1][j], P.w[n][i][j], P.r[m][i + 1][j],
                                                          P.w[m][i][j]);
                    if (i >= 1 && i < RY + 1) P.gr[dk][i - 1][j] = rE[j] - rW[j];
                }
            }
            if (WYZ) {  // drho' beyond a face is the mirror's
                if (wally) {
#pragma unroll
                    for (int j = 0; j < VX; ++j) {
                        if (y0 == 0) P.rn[dk][0][j] = P.rn[dk][1][j];
#pragma unroll
                        for (int i = 1; i < RY + 2; ++i)
                            if (y0 - 1 + i == ny) P.rn[dk][i][j] = P.rn[dk][i - 1][j];
                    }
                }
                if (wallz) {
#pragma unroll
                    for (int i = 0; i < RY + 2; ++i)
#pragma unroll
                        for (int j = 0; j < VX; ++j) {
                            if (nn == 1) P.rn[dm][i][j] = P.rn[dk][i][j];
                            if (nn - 1 == nz) P.rn[dk][i][j] = P.rn[dm][i][j];
                        }
                }
            }
        }
        if (mom) {
            const T cs2 = c.cs2;
            // y fluxes m v of rows y0 - 1 .. y0 + RY of plane n - 2
            T mx[RY + 2][VX], my[RY + 2][VX], mz[RY + 2][VX];
#pragma unroll
            for (int i = 0; i < RY + 2; ++i)
#pragma unroll
                for (int j = 0; j < VX; ++j) {
                    const T r = P.r[m][i + 1][j];
                    mx[i][j] = mom1(r, P.u[m][i][j]);
                    my[i][j] = mom1(r, P.v[m][i + 1][j]);
                    mz[i][j] = mom1(r, P.w[m][i][j]);
                }
#pragma unroll
            for (int i = 0; i < RY; ++i) {
                const T(&r)[VX] = P.r[m][i + 2];
                const T(&u)[VX] = P.u[m][i + 1];
                const T(&v)[VX] = P.v[m][i + 2];
                const T(&w)[VX] = P.w[m][i + 1];
                const T(&a)[VX] = mx[i + 1];
                const T(&b)[VX] = my[i + 1];
                const T(&d)[VX] = mz[i + 1];
                const T(&q)[VX] = P.rn[dm][i + 1];
                T xu[VX], yu[VX], zu[VX];
#pragma unroll
                for (int j = 0; j < VX; ++j) {
                    xu[j] = a[j] * u[j];
                    yu[j] = b[j] * u[j];
                    zu[j] = d[j] * u[j];
                }
                T xuE[VX], xuW[VX], yuE[VX], yuW[VX], zuE[VX], zuW[VX], aE[VX], aW[VX], bE[VX], bW[VX], dE[VX], dW[VX],
                    qE[VX], qW[VX];
                east_west(xu, xuE, xuW);
                east_west(yu, yuE, yuW);
                east_west(zu, zuE, zuW);
                east_west(a, aE, aW);
                east_west(b, bE, bW);
                east_west(d, dE, dW);
                east_west(q, qE, qW);
                if (WX && eg.any) {
                    const T gr = eg.l ? r[0] : r[VX - 1];
                    const T gu = fmaT(eg.s[0], eg.l ? u[0] : u[VX - 1], eg.o[0]);
                    const T gv = fmaT(eg.s[1], eg.l ? v[0] : v[VX - 1], eg.o[1]);
                    const T gw = fmaT(egw[0], eg.l ? w[0] : w[VX - 1], egw[1]);
                    const T ga = mom1(gr, gu), gb = mom1(gr, gv), gd = mom1(gr, gw);
                    const T gxu = ga * gu, gyu = gb * gu, gzu = gd * gu;
                    xuW[0] = eg.l ? gxu : xuW[0];
                    yuW[0] = eg.l ? gyu : yuW[0];
                    zuW[0] = eg.l ? gzu : zuW[0];
                    aW[0] = eg.l ? ga : aW[0];
                    bW[0] = eg.l ? gb : bW[0];
                    dW[0] = eg.l ? gd : dW[0];
                    qW[0] = eg.l ? q[0] : qW[0];
                    xuE[VX - 1] = eg.r ? gxu : xuE[VX - 1];
                    yuE[VX - 1] = eg.r ? gyu : yuE[VX - 1];
                    zuE[VX - 1] = eg.r ? gzu : zuE[VX - 1];
                    aE[VX - 1] = eg.r ? ga : aE[VX - 1];
                    bE[VX - 1] = eg.r ? gb : bE[VX - 1];
                    dE[VX - 1] = eg.r ? gd : dE[VX - 1];
                    qE[VX - 1] = eg.r ? q[VX - 1] : qE[VX - 1];
                }
#pragma unroll
                for (int j = 0; j < VX; ++j) {
                    // the expressions of momentum3d (step3d.h) on shared products
                    const T rc = r[j], uc = u[j], vc = v[j], wc = w[j];
                    const T rN = P.r[m][i + 3][j], rS = P.r[m][i + 1][j];
                    const T vN = P.v[m][i + 3][j], vS = P.v[m][i + 1][j];
                    const T mxN = mx[i + 2][j], mxS = mx[i][j], myN = my[i + 2][j], myS = my[i][j];
                    const T mzN = mz[i + 2][j], mzS = mz[i][j];
                    const T rU = P.r[k][i + 2][j], wU = P.w[k][i + 1][j];
                    const T mxU = mom1(rU, P.u[k][i + 1][j]), myU = mom1(rU, P.v[k][i + 2][j]), mzU = mom1(rU, wU);
                    const T rD = P.r[s][i + 2][j], wD = P.w[s][i + 1][j];
                    const T mxD = mom1(rD, P.u[s][i + 1][j]), myD = mom1(rD, P.v[s][i + 2][j]), mzD = mom1(rD, wD);
                    const T gxr = P.gr[dm][i][j], gyr = rN - rS, gzr = rU - rD;
                    const T fxx = fmaT(cs2, gxr, ((xuE[j] - xuW[j]) + (mxN * vN - mxS * vS)) + (mxU * wU - mxD * wD));
                    const T fyy = fmaT(cs2, gyr, ((yuE[j] - yuW[j]) + (myN * vN - myS * vS)) + (myU * wU - myD * wD));
                    const T fzz = fmaT(cs2, gzr, ((zuE[j] - zuW[j]) + (mzN * vN - mzS * vS)) + (mzU * wU - mzD * wD));
                    const T lpx = fmaT(T(-6), a[j], ((aE[j] + aW[j]) + (mxN + mxS)) + (mxU + mxD));
                    const T lpy = fmaT(T(-6), b[j], ((bE[j] + bW[j]) + (myN + myS)) + (myU + myD));
                    const T lpz = fmaT(T(-6), d[j], ((dE[j] + dW[j]) + (mzN + mzS)) + (mzU + mzD));
                    const T rnC = q[j];
                    const T sx = (qE[j] - qW[j]) - gxr;
                    const T sy = (P.rn[dm][i + 2][j] - P.rn[dm][i][j]) - gyr;
                    const T sz = (P.rn[dk][i + 1][j] - P.rn[ds][i + 1][j]) - gzr;
                    const T rho_n = T(1) + rnC;
                    T dmx = fmaT(rho_n, gx[i], fmaT(-c.ks, sx, fmaT(c.kv, lpx, -c.cg * fxx)));
                    T dmy = fmaT(rho_n, c.gdt[1], fmaT(-c.ks, sy, fmaT(c.kv, lpy, -c.cg * fyy)));
                    T dmz = fmaT(rho_n, c.gdt[2], fmaT(-c.ks, sz, fmaT(c.kv, lpz, -c.cg * fzz)));
                    if constexpr (FST) {  // -dt phi G_iso mu
                        dmx = fmaT(-c.dt, P.fs[J % 2][0][i][j], dmx);
                        dmy = fmaT(-c.dt, P.fs[J % 2][1][i][j], dmy);
                        dmz = fmaT(-c.dt, P.fs[J % 2][2][i][j], dmz);
                    }
                    const T drn = rnC - rc;
                    const T inv = recipT(rho_n);
                    ro[i][j] = rnC;
                    uo[i][j] = fmaT(fmaT(-uc, drn, dmx), inv, uc);
                    vo[i][j] = fmaT(fmaT(-vc, drn, dmy), inv, vc);
                    wo[i][j] = fmaT(fmaT(-wc, drn, dmz), inv, wc);
                }
            }
        }
        // stores stand outside the branch (see march2d.h); rows not formed or past the grid are dropped
        const unsigned pz = mom ? (unsigned)(nn - 2) * pbytes : 0u;
#pragma unroll
        for (int i = 0; i < RY; ++i) {
            const unsigned so = (mom && st && y0 + i < ny) ? loff : fbytes;
            row_store<T, VX>(ro[i], qr, so, pz + yoff[i + 2]);
            row_store<T, VX>(uo[i], qu, so, pz + yoff[i + 2]);
            row_store<T, VX>(vo[i], qv, so, pz + yoff[i + 2]);
            row_store<T, VX>(wo[i], qw, so, pz + yoff[i + 2]);
        }
    };
    int n = nb;
    for (;;) {
        iterate(n, std::integral_constant<int, 0>{});
        if (n++ == ne) break;
        iterate(n, std::integral_constant<int, 1>{});
        if (n++ == ne) break;
        iterate(n, std::integral_constant<int, 2>{});
        if (n++ == ne) break;
        iterate(n, std::integral_constant<int, 3>{});
        if (n++ == ne) break;
        iterate(n, std::integral_constant<int, 4>{});
        if (n++ == ne) break;
        iterate(n, std::integral_constant<int, 5>{});
        if (n++ == ne) break;
    }
}

}  // namespace march
}  // namespace acm
