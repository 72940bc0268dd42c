// Fused two-phase SMAME step (2D) for gfx950: flow update with the
// surface-tension force, and the Cahn-Hilliard equation (Eq. 2.14) advanced
// by Heun's second-order Runge-Kutta method, all in one launch.
//
// Per step and node (Sec. 2, two-phase paragraphs):
//   mu     = 4 a phi (phi^2 - 1) - kappa L_iso phi
//   flow   = single-phase update (Eqs. 2.10-2.11) + force -dt phi G_iso mu
//   R(f,m) = M L_iso m - (u G_iso,x f + v G_iso,y f)        (u = u^n)
//   phi*   = phi + dt R(phi, mu)
//   phi^{n+1} = (phi + phi* + dt R(phi*, mu*)) / 2,   mu* = mu(phi*)
// with the D2Q9-weighted isotropic stencils
//   G_iso,x f = [4 (f_E - f_W) + (f_NE + f_SE - f_NW - f_SW)] / (12 dx)
//   L_iso f   = [4 (f_E + f_W + f_N + f_S) + (f_NE + f_NW + f_SE + f_SW) - 20 f] / (6 dx^2).
// AXI = true is the axisymmetric form (x axial, y radial, axis on the -y
// face, row j at r = (j + 1/2) dx): L_iso gains (1/r) G_iso,r in mu and in
// the Cahn-Hilliard diffusion, continuity and momentum take the
// cylindrical flux forms of the single-phase axisymmetric step
// (kern_axisym.h); the advection and the surface-tension force are
// unchanged.
// Dependency radii: phi needs a 4-node halo (mu on tile+3, phi* on tile+2,
// mu* on tile+1), the flow fields a 2-node halo.  Ghost positions of every
// intermediate take the value at their mirror node for walls and symmetry
// planes, so they are computed there; phi and phi* ghosts across a wall
// then take the wetting rule of Sec. 2 (identity for a 90 degree angle).
// LDS: phi^n and mu^n are last read in the phi* phase (which also takes
// each output node's phi^n and surface-tension force into registers), so
// mu* and drho' are written over them afterwards; 18.7 KB per 32 x 16 tile
// lets eight workgroups share a CU.  The default where walls have no wetting
// rule is the register march further below.
#include <algorithm>
#include <cmath>

#include "acm_internal.h"
#include "kern_axisym.h"
#include "march2d.h"
#include "tile2d.h"

namespace acm {

template <typename T>
__device__ __forceinline__ T momc2(T r, T u, T rho0) { return fmaT(r, u, rho0 * u); }

template <int TX, int TY>
struct Shape2P {
    static constexpr int PX = TX + 8, PY = TY + 8, PXY = PX * PY;   // phi, halo 4
    static constexpr int MX = TX + 6, MY = TY + 6, MXY = MX * MY;   // mu, halo 3
    static constexpr int RX = TX + 4, RY = TY + 4, RXY = RX * RY;   // flow fields / phi*, halo 2
    static constexpr int DX = TX + 2, DY = TY + 2, DXY = DX * DY;   // mu*, drho', halo 1
    static_assert(DXY <= PXY && DXY <= MXY, "mu* and drho' fit in the phi and mu regions");
};

// isotropic Laplacian numerator: 4 (E+W+N+S) + (NE+NW+SE+SW) - 20 C
template <typename T, int W>
__device__ __forceinline__ T liso_num(const T* f, int e)
{
    const T ax = (f[e + 1] + f[e - 1]) + (f[e + W] + f[e - W]);
    const T dg = (f[e + 1 + W] + f[e - 1 + W]) + (f[e + 1 - W] + f[e - 1 - W]);
    return fmaT(T(4), ax, dg) - T(20) * f[e];
}
template <typename T, int W>
__device__ __forceinline__ T gisox_num(const T* f, int e)
{
    return fmaT(T(4), f[e + 1] - f[e - 1], (f[e + 1 + W] + f[e + 1 - W]) - (f[e - 1 + W] + f[e - 1 - W]));
}
template <typename T, int W>
__device__ __forceinline__ T gisoy_num(const T* f, int e)
{
    return fmaT(T(4), f[e + W] - f[e - W], (f[e + 1 + W] + f[e - 1 + W]) - (f[e + 1 - W] + f[e - 1 - W]));
}

// chemical potential from a phi array of row width W at index e
template <typename T, int W>
__device__ __forceinline__ T chem(const Coef<T>& c, const T* f, int e)
{
    const T p = f[e];
    return fmaT(c.a4 * p, fmaT(p, p, T(-1)), -c.kap6 * liso_num<T, W>(f, e));
}

// chemical potential with the cylindrical Laplacian when AXI (irc =
// 1 / (row + 1/2)): -kappa (1/r) G_iso,r phi = -(kappa / 6 dx^2) irc gy / 2
template <typename T, int W, bool AXI>
__device__ __forceinline__ T chem_a(const Coef<T>& c, const T* f, int e, T irc)
{
    const T m = chem<T, W>(c, f, e);
    if constexpr (AXI) return fmaT(T(-0.5) * c.kap6 * irc, gisoy_num<T, W>(f, e), m);
    else return m;
}

// numerator of the (cylindrical when AXI) isotropic Laplacian in units of
// 1 / (6 dx^2): L_iso + (1/r) G_iso,r = [liso_num + irc gy_num / 2] / (6 dx^2)
template <typename T, int W, bool AXI>
__device__ __forceinline__ T lap_a(const T* f, int e, T irc)
{
    if constexpr (AXI) return fmaT(T(0.5) * irc, gisoy_num<T, W>(f, e), liso_num<T, W>(f, e));
    else return liso_num<T, W>(f, e);
}

template <bool AXI, typename T>
__device__ __forceinline__ T inv_radius(int row)
{
    if constexpr (AXI) return T(1) / (T(row) + T(0.5));
    else return T(0);
}

// local coordinate (in a region with halo h) whose value stands in for the
// position l: the mirror node for wall / symmetry ghosts, else l itself
__device__ __forceinline__ int ghost_src(int l, int h, int o0, int n, int bc_lo, int lo, int hi)
{
    const int g = mirror_coord(o0 + l - h, n, bc_lo);
    return min(max(g - o0 + h, lo), hi);
}

template <typename T, int TX, int TY, int NT, bool AXI>
__global__ __launch_bounds__(NT) void twophase2d_kernel(Coef<T> c, State<T> in, State<T> out, int nbx)
{
    using S = Shape2P<TX, TY>;
    constexpr int PX = S::PX, MX = S::MX, RX = S::RX, DX = S::DX;
    __shared__ T sp[S::PXY];                          // phi^n, then mu*
    __shared__ T smu[S::MXY];                         // mu^n, then drho'
    __shared__ T sr[S::RXY], su[S::RXY], sv[S::RXY];  // drho, u, v
    __shared__ T sps[S::RXY];                         // phi*
    T* const sms = sp;
    T* const srn = smu;
    constexpr int NQ = (TX * TY + NT - 1) / NT;       // output nodes per thread
    T pcq[NQ], fsx[NQ], fsy[NQ];                      // phi^n and surface-tension force there

    const int lb = [&] {
        constexpr int NX = 8;
        const int nb = gridDim.x, b = blockIdx.x;
        const int per = nb / NX, rem = nb % NX;
        const int x = b % NX, i = b / NX;
        return x * per + min(x, rem) + i;
    }();
    const int by = lb / nbx, bx = lb - by * nbx;
    const int x0 = bx * TX, y0 = by * TY;
    const int nx = c.nx, ny = c.ny;
    const bool interior = (x0 >= 4) && (x0 + TX + 4 <= nx) && (y0 >= 4) && (y0 + TY + 4 <= ny);
    const bool mirror = !interior && c.nonperiodic;
    const int tid = threadIdx.x;

    // ---- stage phi (halo 4) and drho, u, v (halo 2); every load of the
    // thread is issued before its first LDS store so the latencies overlap
    {
        constexpr int NP = (S::PXY + NT - 1) / NT, NR = (S::RXY + NT - 1) / NT;
        T pv[NP], rv[NR], uv[NR], vv[NR];
        int fxs[NR], fys[NR];
        if (interior) {  // no ghost in either region: plain offsets
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const int q = min(tid + i * NT, S::PXY - 1);
                const int ly = q / PX, lx = q - ly * PX;
                pv[i] = in.phi[(size_t)(y0 + ly - 4) * nx + (x0 + lx - 4)];
            }
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                const int q = min(tid + i * NT, S::RXY - 1);
                const int ly = q / RX, lx = q - ly * RX;
                const size_t s = (size_t)(y0 + ly - 2) * nx + (x0 + lx - 2);
                rv[i] = in.r[s];
                uv[i] = in.u[s];
                vv[i] = in.v[s];
                fxs[i] = fys[i] = -1;
            }
        } else {
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const int q = min(tid + i * NT, S::PXY - 1);
                const int ly = q / PX, lx = q - ly * PX;
                int fx, fy;
                const int sx = map_coord(x0 + lx - 4, nx, c.bc[0], 0, fx);
                const int sy = map_coord(y0 + ly - 4, ny, c.bc[2], 2, fy);
                pv[i] = in.phi[(size_t)sy * nx + sx];
                if (c.wet) {  // wetting rule across wall faces, x then y
                    if (fx >= 0) pv[i] = wet_ghost(pv[i], wet_b(c, fx));
                    if (fy >= 0) pv[i] = wet_ghost(pv[i], wet_b(c, fy));
                }
            }
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                const int q = min(tid + i * NT, S::RXY - 1);
                const int ly = q / RX, lx = q - ly * RX;
                const int sx = map_coord(x0 + lx - 2, nx, c.bc[0], 0, fxs[i]);
                const int sy = map_coord(y0 + ly - 2, ny, c.bc[2], 2, fys[i]);
                const size_t s = (size_t)sy * nx + sx;
                rv[i] = in.r[s];
                uv[i] = in.u[s];
                vv[i] = in.v[s];
            }
        }
#pragma unroll
        for (int i = 0; i < NP; ++i)
            if (tid + i * NT < S::PXY) sp[tid + i * NT] = pv[i];
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const int q = tid + i * NT;
            if (q < S::RXY) {
                T u = uv[i], v = vv[i];
                const int fx = fxs[i], fy = fys[i];
                if (fx >= 0) {
                    u = fmaT(c.fs[fx][0], u, c.fo[fx][0]);
                    v = fmaT(c.fs[fx][1], v, c.fo[fx][1]);
                }
                if (fy >= 0) {
                    u = fmaT(c.fs[fy][0], u, c.fo[fy][0]);
                    v = fmaT(c.fs[fy][1], v, c.fo[fy][1]);
                }
                sr[q] = rv[i];
                su[q] = u;
                sv[q] = v;
            }
        }
    }
    __syncthreads();

    // ---- mu^n on tile+3
#pragma unroll
    for (int q = tid; q < S::MXY; q += NT) {
        const int ly = q / MX, lx = q - ly * MX;
        int ex = lx + 1, ey = ly + 1;  // phi-region coordinates
        if (mirror) {
            ex = ghost_src(lx, 3, x0, nx, c.bc[0], 0, MX - 1) + 1;
            ey = ghost_src(ly, 3, y0, ny, c.bc[2], 0, S::MY - 1) + 1;
        }
        smu[q] = chem_a<T, PX, AXI>(c, sp, ey * PX + ex, inv_radius<AXI, T>(y0 + ey - 4));
    }
    __syncthreads();

    // ---- phi* on tile+2
#pragma unroll
    for (int q = tid; q < S::RXY; q += NT) {
        const int ly = q / RX, lx = q - ly * RX;
        int ex = lx, ey = ly;  // flow-region coordinates of the evaluation node
        if (mirror) {
            ex = ghost_src(lx, 2, x0, nx, c.bc[0], 0, RX - 1);
            ey = ghost_src(ly, 2, y0, ny, c.bc[2], 0, S::RY - 1);
        }
        const int ep = (ey + 2) * PX + (ex + 2);  // phi region
        const int em = (ey + 1) * MX + (ex + 1);  // mu region
        const int ef = ey * RX + ex;
        const T gxp = gisox_num<T, PX>(sp, ep), gyp = gisoy_num<T, PX>(sp, ep);
        const T adv = fmaT(su[ef], gxp, sv[ef] * gyp) * c.gi;
        const T rhs = fmaT(c.mob * c.li, lap_a<T, MX, AXI>(smu, em, inv_radius<AXI, T>(y0 + ey - 2)), -adv);
        T val = fmaT(c.dt, rhs, sp[ep]);
        if (mirror && c.wet) {  // a ghost position takes the wetting rule of its wall faces
            const int gx = x0 + lx - 2, gy = y0 + ly - 2;
            if (gx < 0) val = wet_ghost(val, c.wb[0]);
            if (gx >= nx) val = wet_ghost(val, c.wb[1]);
            if (gy < 0) val = wet_ghost(val, c.wb[2]);
            if (gy >= ny) val = wet_ghost(val, c.wb[3]);
        }
        sps[q] = val;
    }
    // phi^n and the surface-tension force -dt phi G_iso mu at this thread's
    // output nodes, while phi^n and mu^n are still in LDS
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
        const int q = min(tid + k * NT, TX * TY - 1);
        const int ly = q / TX, lx = q - ly * TX;
        const int ep = (ly + 4) * PX + (lx + 4);  // phi region
        const int em = (ly + 3) * MX + (lx + 3);  // mu region
        const T pc = sp[ep];
        pcq[k] = pc;
        fsx[k] = -c.dt * pc * (gisox_num<T, MX>(smu, em) * c.gi);
        fsy[k] = -c.dt * pc * (gisoy_num<T, MX>(smu, em) * c.gi);
    }
    __syncthreads();

    // ---- mu* on tile+1 (over phi^n) and drho' on tile+1 (over mu^n)
#pragma unroll
    for (int q = tid; q < S::DXY; q += NT) {
        const int ly = q / DX, lx = q - ly * DX;
        int ex = lx + 1, ey = ly + 1;  // phi*-region coordinates
        if (mirror) {
            ex = ghost_src(lx, 1, x0, nx, c.bc[0], 0, DX - 1) + 1;
            ey = ghost_src(ly, 1, y0, ny, c.bc[2], 0, S::DY - 1) + 1;
        }
        sms[q] = chem_a<T, RX, AXI>(c, sps, ey * RX + ex, inv_radius<AXI, T>(y0 + ey - 2));
    }
#pragma unroll
    for (int q = tid; q < S::DXY; q += NT) {
        const int ly = q / DX, lx = q - ly * DX;
        int ex = lx + 1, ey = ly + 1;  // flow-region coordinates
        if (mirror) {
            ex = ghost_src(lx, 1, x0, nx, c.bc[0], 0, DX - 1) + 1;
            ey = ghost_src(ly, 1, y0, ny, c.bc[2], 0, S::DY - 1) + 1;
        }
        const int e = ey * RX + ex;
        const T rc = sr[e];
        const T rE = sr[e + 1], rW = sr[e - 1], rN = sr[e + RX], rS = sr[e - RX];
        T div, lap;
        if constexpr (AXI) {  // cylindrical flux forms (kern_axisym.h)
            axi_continuity(c.rho0, T(y0 + ey - 2), inv_radius<AXI, T>(y0 + ey - 2), rc, rE, rW, rN, rS, su[e + 1],
                           su[e - 1], sv[e], sv[e + RX], sv[e - RX], div, lap);
        } else {
            div = mdiff(rE, su[e + 1], rW, su[e - 1], c.rho0) + mdiff(rN, sv[e + RX], rS, sv[e - RX], c.rho0);
            lap = ((rE + rW) + (rN + rS)) - T(4) * rc;
        }
        srn[q] = fmaT(-c.cg, div, fmaT(c.kr, lap, rc));
    }
    __syncthreads();

    // ---- outputs on the tile
    const T rho0 = c.rho0, cs2 = c.cs2;
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
        const int q = tid + k * NT;
        if (q >= TX * TY) break;
        const int ly = q / TX, lx = q - ly * TX;
        const int gx = x0 + lx, gy = y0 + ly;
        if (gx >= nx || gy >= ny) continue;
        const int e = (ly + 2) * RX + (lx + 2);   // flow / phi* region
        const int d = (ly + 1) * DX + (lx + 1);   // drho' / mu* region
        // flow
        const T rc = sr[e], uc = su[e], vc = sv[e];
        const T rE = sr[e + 1], rW = sr[e - 1], rN = sr[e + RX], rS = sr[e - RX];
        const T uE = su[e + 1], uW = su[e - 1], uN = su[e + RX], uS = su[e - RX];
        const T vE = sv[e + 1], vW = sv[e - 1], vN = sv[e + RX], vS = sv[e - RX];
        const T mxC = momc2(rc, uc, rho0), myC = momc2(rc, vc, rho0);
        const T mxE = momc2(rE, uE, rho0), mxW = momc2(rW, uW, rho0);
        const T mxN = momc2(rN, uN, rho0), mxS = momc2(rS, uS, rho0);
        const T myE = momc2(rE, vE, rho0), myW = momc2(rW, vW, rho0);
        const T myN = momc2(rN, vN, rho0), myS = momc2(rS, vS, rho0);
        const T rnC = srn[d];
        const T irc = inv_radius<AXI, T>(gy);
        T fxx, fyy, lpx, lpy;
        if constexpr (AXI) {  // cylindrical flux forms, hoop term, -m_r / r^2 (kern_axisym.h)
            axi_momentum(cs2, T(gy), irc, rc, rE, rW, rN, rS, uE, uW, vc, vN, vS, mxC, mxE, mxW, mxN, mxS, myC, myE,
                         myW, myN, myS, fxx, fyy, lpx, lpy);
        } else {
            fxx = (fmaT(mxE, uE, cs2 * rE) - fmaT(mxW, uW, cs2 * rW)) + (mxN * vN - mxS * vS);
            fyy = (myE * uE - myW * uW) + (fmaT(myN, vN, cs2 * rN) - fmaT(myS, vS, cs2 * rS));
            lpx = ((mxE + mxW) + (mxN + mxS)) - T(4) * mxC;
            lpy = ((myE + myW) + (myN + myS)) - T(4) * myC;
        }
        const T sx = (srn[d + 1] - srn[d - 1]) - (rE - rW);
        const T sy = (srn[d + DX] - srn[d - DX]) - (rN - rS);
        const T rho_n = rho0 + rnC;
        const T pc = pcq[k], fstx = fsx[k], fsty = fsy[k];
        T gx_ = c.gdt[0];
        if (c.fx) gx_ = fmaT(c.dt, c.fx[gy], gx_);
        const T dmx = fmaT(rho_n, gx_, fmaT(-c.ks, sx, fmaT(c.kv, lpx, fmaT(-c.cg, fxx, fstx))));
        const T dmy = fmaT(rho_n, c.gdt[1], fmaT(-c.ks, sy, fmaT(c.kv, lpy, fmaT(-c.cg, fyy, fsty))));
        const T drn = rnC - rc;
        const T inv = recipT(rho_n);
        // Cahn-Hilliard second stage
        const T gxs = gisox_num<T, RX>(sps, e), gys = gisoy_num<T, RX>(sps, e);
        const T adv = fmaT(uc, gxs, vc * gys) * c.gi;
        const T rhs = fmaT(c.mob * c.li, lap_a<T, DX, AXI>(sms, d, irc), -adv);
        const T phin = T(0.5) * fmaT(c.dt, rhs, pc + sps[e]);
        const size_t o = (size_t)gy * nx + gx;
        out.r[o] = rnC;
        out.u[o] = fmaT(fmaT(-uc, drn, dmx), inv, uc);
        out.v[o] = fmaT(fmaT(-vc, drn, dmy), inv, vc);
        out.phi[o] = phin;
    }
}

// ---------------------------------------------------------------------------
// The same step as a register march along y (march2d.h): a wave owns a window
// of 64 VX columns (four columns of halo on each side) and marches it down a
// chunk of rows; every stage of the step follows the one before it by a row.
// When phi of row n arrives,
//   mu is formed on row n - 1, phi* and the force on row n - 2 (whose flow
//   arrives then), mu* on row n - 3, phi^{n+1} and the flow on row n - 4.
// No LDS and no barrier: the tile kernel spends five barriers and 1.6 to 3.1
// times the nodes of a 32 x 16 tile on its halos (44 x 28 staged for phi); here
// only a chunk's ends repeat rows, and a row's sums E + W are formed once for
// the three rows that use them.  Each value is formed by the expressions of the
// tile kernel in the same order.
// Bound by vector instructions (about 180 per row and wave of 64).  us per
// step, tile kernel -> march: 256 x 256 7.7 -> 6.0, 1024 x 1024 18.3 -> 14.5
// (doubles 26.7 -> 20.7), axisymmetric 2048 x 1024 31.5 -> 23.0 (doubles 49.6
// -> 35.4), 4096 x 2048 88 -> 51.  Two columns per lane (FP32) halve the halo
// columns' share: axisymmetric 2048 x 1024 24.7 -> 23.0; small grids lose
// waves by it (512 x 512 8.3 -> 8.5).
// ---------------------------------------------------------------------------
namespace march2p {

// one field of the phase-field pipeline by row modulo 6, and its x sums E + W
template <typename T, int VX>
struct Ring {
    T f[6][VX], s[6][VX];
};

// rows y0 .. y1 - 1 of the window starting at column xs; lanes l0 .. l1 - 1 store
template <typename T, int VX, bool WX, bool AXI>
__device__ __forceinline__ void run(const Coef<T>& c, const State<T>& in, const State<T>& out, int xs, int l0, int l1,
                                    int y0, int y1)
{
    const int nx = c.nx, ny = c.ny, lane = threadIdx.x & 63;
    const bool wallx = WX && c.bc[0] != BC_PERIODIC, wally = AXI || c.bc[2] != BC_PERIODIC;
    const unsigned pitch = (unsigned)nx * (unsigned)sizeof(T), fbytes = pitch * (unsigned)ny;
    int x = xs + VX * lane;
    if (wallx) {
        x = min(x, nx - VX);
    } else {
        x = x < 0 ? x + nx : (x >= nx ? x - nx : x);
        if (x < 0 || x >= nx) x = ((x % nx) + nx) % nx;
    }
    const unsigned loff = (unsigned)x * (unsigned)sizeof(T);
    const unsigned soff = (lane >= l0 && lane < l1) ? loff : fbytes;  // past the end: dropped
    march::Edge<T> eg;
    eg.l = wallx && xs == 0 && lane == 0;
    eg.r = wallx && xs + VX * (lane + 1) == nx;
    eg.any = wallx && (xs == 0 || xs + 64 * VX >= nx);
    if (WX) {
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            eg.s[a] = eg.l ? c.fs[0][a] : c.fs[1][a];
            eg.o[a] = eg.l ? c.fo[0][a] : c.fo[1][a];
        }
    }
    const __amdgpu_buffer_rsrc_t ip = march::field_rsrc(in.phi, fbytes), ir = march::field_rsrc(in.r, fbytes),
                                 iu = march::field_rsrc(in.u, fbytes), iv = march::field_rsrc(in.v, fbytes),
                                 qp = march::field_rsrc(out.phi, fbytes), qr = march::field_rsrc(out.r, fbytes),
                                 qu = march::field_rsrc(out.u, fbytes), qv = march::field_rsrc(out.v, fbytes);
    // neighbours in x; beyond an x face the node itself (its mirror)
    typedef T V[VX];
    auto east_west = [&](const V& f, V& ea, V& we) {
        march::east_west(f, ea, we);
        if (WX) {
            ea[VX - 1] = eg.r ? f[VX - 1] : ea[VX - 1];
            we[0] = eg.l ? f[0] : we[0];
        }
    };

    march::Level<T, VX> L;
    Ring<T, VX> P, M, PS, MS;  // phi, mu, phi*, mu*
    T fst[3][2][VX];       // two-phase force by row modulo 3
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int j = 0; j < VX; ++j) {
            L.r[q][j] = L.u[q][j] = L.v[q][j] = T(0);
            P.f[q][j] = P.s[q][j] = M.f[q][j] = M.s[q][j] = T(0);
            PS.f[q][j] = PS.s[q][j] = MS.f[q][j] = MS.s[q][j] = T(0);
            if (q < 3) {
                L.mx[q][j] = L.my[q][j] = L.pxy[q][j] = L.pyy[q][j] = T(0);
                L.rn[q][j] = L.gr[q][j] = fst[q][0][j] = fst[q][1][j] = T(0);
            }
        }
    // a walled bottom face starts at its ghost row; flow rows lag two behind
    const int nb = wally ? max(y0 - 4, -1) : y0 - 4, ne = y1 + 3;
    auto wrap = [&](int y) { return wally ? y : ((y % ny) + ny) % ny; };
    int yp = wrap(nb), yf = wrap(nb - 2);  // next rows to fetch
    auto row_of = [&](int& y) {
        const int r = wally ? min(max(y, 0), ny - 1) : y;
        y = !wally && y + 1 == ny ? 0 : y + 1;
        return (unsigned)r * pitch;
    };
    auto fetch = [&](auto slot) {
        constexpr int sl = decltype(slot)::value;
        march::row_load<T, VX>(P.f[sl], ip, loff, row_of(yp));
        const unsigned o = row_of(yf);
        march::row_load<T, VX>(L.r[sl], ir, loff, o);
        march::row_load<T, VX>(L.u[sl], iu, loff, o);
        march::row_load<T, VX>(L.v[sl], iv, loff, o);
    };
    constexpr int PD = VX == 1 ? 2 : 1;
    fetch(std::integral_constant<int, 0>{});
    if constexpr (PD == 2) fetch(std::integral_constant<int, 1>{});

    // dt times the x force and 1 / (row + 1/2) of 64 rows at a time, lane l holding row ib + l
    int ib = nb;
    T irv = T(0), fxv = c.gdt[0];
    auto fill = [&](int from) {
        ib = from;
        if (AXI) irv = T(1) / (T(from + lane) + T(0.5));
        if (c.fx) fxv = fmaT(c.dt, c.fx[min(max(from + lane, 0), ny - 1)], c.gdt[0]);
    };
    fill(nb);
    auto inv_r = [&](int row) { return march::lane_value(irv, (row - ib) & 63); };
    auto force = [&](int row) { return march::lane_value(fxv, (row - ib) & 63); };

    // sums of the D2Q9 stencils around row b (N above, S below), in the order of liso_num, gisox_num, gisoy_num
    typedef Ring<T, VX> Rows;
    auto gy = [&](const Rows& A, int nn, int ss, int j) {
        return fmaT(T(4), A.f[nn][j] - A.f[ss][j], A.s[nn][j] - A.s[ss][j]);
    };
    auto gx = [&](const Rows& A, int nn, int b, int ss, V& g) {
        V t, fe, fw, te, tw;
#pragma unroll
        for (int j = 0; j < VX; ++j) t[j] = A.f[nn][j] + A.f[ss][j];
        east_west(A.f[b], fe, fw);
        east_west(t, te, tw);
#pragma unroll
        for (int j = 0; j < VX; ++j) g[j] = fmaT(T(4), fe[j] - fw[j], te[j] - tw[j]);
    };
    auto lap0 = [&](const Rows& A, int nn, int b, int ss, int j) {
        return fmaT(T(4), A.s[b][j] + (A.f[nn][j] + A.f[ss][j]), A.s[nn][j] + A.s[ss][j]) - T(20) * A.f[b][j];
    };
    auto lap = [&](const Rows& A, int nn, int b, int ss, T hirc, int j) {
        const T l = lap0(A, nn, b, ss, j);
        if constexpr (AXI) return fmaT(hirc, gy(A, nn, ss, j), l);
        else return l;
    };
    auto chem = [&](const Rows& A, int nn, int b, int ss, T irc, V& m) {
#pragma unroll
        for (int j = 0; j < VX; ++j) {
            const T p = A.f[b][j];
            m[j] = fmaT(c.a4 * p, fmaT(p, p, T(-1)), -c.kap6 * lap0(A, nn, b, ss, j));
            if constexpr (AXI) m[j] = fmaT(T(-0.5) * c.kap6 * irc, gy(A, nn, ss, j), m[j]);
        }
    };
    auto sums = [&](Rows& A, int b) {
        V ea, we;
        east_west(A.f[b], ea, we);
#pragma unroll
        for (int j = 0; j < VX; ++j) A.s[b][j] = ea[j] + we[j];
    };
    // ghost row of an intermediate: row 0 is the mirror of row -1, row ny - 1 of row ny
    auto ghost = [&](Rows& A, int row, int b, int ss) {
#pragma unroll
        for (int j = 0; j < VX; ++j) {
            if (wally && row == 0) A.f[ss][j] = A.f[b][j], A.s[ss][j] = A.s[b][j];
            if (wally && row == ny) A.f[b][j] = A.f[ss][j], A.s[b][j] = A.s[ss][j];
        }
    };

    // phi of row n and the flow of row n - 2 have arrived (slot J): mu of row
    // n - 1, phi* and the force of row n - 2, mu* of row n - 3, the new state of row n - 4
    auto iterate = [&](int n, auto jc) {
        constexpr int J = decltype(jc)::value;
        constexpr int a = J, b = (J + 5) % 6, d = (J + 4) % 6, e = (J + 3) % 6, f = (J + 2) % 6, h = (J + 1) % 6;
        V pn, r, u, v, g, pc;  // pc: phi of row n - 4, whose slot the fetch takes
#pragma unroll
        for (int j = 0; j < VX; ++j) pc[j] = P.f[f][j];
        fetch(std::integral_constant<int, (J + PD) % 6>{});
        sums(P, a);
        if (n - 1 >= y0 - 3) {
            chem(P, a, b, d, AXI ? inv_r(n - 1) : T(0), M.f[b]);
            sums(M, b);
            ghost(M, n - 1, b, d);
        }
        bool have = false;
        if (n - 2 >= y0 - 2) {
            const T hirc = AXI ? T(0.5) * inv_r(n - 2) : T(0);
            gx(P, b, d, e, g);
#pragma unroll
            for (int j = 0; j < VX; ++j) {
                const T adv = fmaT(L.u[J][j], g[j], L.v[J][j] * gy(P, b, e, j)) * c.gi;
                const T rhs = fmaT(c.mob * c.li, lap(M, b, d, e, hirc, j), -adv);
                PS.f[d][j] = fmaT(c.dt, rhs, P.f[d][j]);
            }
            sums(PS, d);
            ghost(PS, n - 2, d, e);
            gx(M, b, d, e, g);
#pragma unroll
            for (int j = 0; j < VX; ++j) {
                fst[J % 3][0][j] = -c.dt * P.f[d][j] * (g[j] * c.gi);
                fst[J % 3][1][j] = -c.dt * P.f[d][j] * (gy(M, b, e, j) * c.gi);
            }
            if (n - 3 >= y0 - 1) {
                chem(PS, d, e, f, AXI ? inv_r(n - 3) : T(0), MS.f[e]);
                sums(MS, e);
                ghost(MS, n - 3, e, f);
            }
            if (n - 4 >= y0) {
                const T hirc2 = AXI ? T(0.5) * inv_r(n - 4) : T(0);
                constexpr int o = (J + 4) % 6;
                gx(PS, e, f, h, g);
#pragma unroll
                for (int j = 0; j < VX; ++j) {
                    const T adv = fmaT(L.u[o][j], g[j], L.v[o][j] * gy(PS, e, h, j)) * c.gi;
                    const T rhs = fmaT(c.mob * c.li, lap(MS, e, f, h, hirc2, j), -adv);
                    pn[j] = T(0.5) * fmaT(c.dt, rhs, pc[j] + PS.f[f][j]);
                }
            }
            have = march::push<J, T, VX, WX, true, AXI>(c, L, n - 2, y0, wally, eg, inv_r, force, r, u, v,
                                                        fst[(J + 1) % 3]);
        }
        const unsigned so = have ? soff : fbytes, o = have ? (unsigned)(n - 4) * pitch : 0u;
        march::row_store<T, VX>(r, qr, so, o);
        march::row_store<T, VX>(u, qu, so, o);
        march::row_store<T, VX>(v, qv, so, o);
        march::row_store<T, VX>(pn, qp, so, o);
    };
    int n = nb;
    for (;;) {
        if (n - ib >= 48 && (AXI || c.fx)) fill(n - 5);  // the next six iterations use rows n - 4 .. n + 4
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

template <typename T, int VX, bool WX, bool AXI>
__global__ __launch_bounds__(256) void twophase_march_kernel(Coef<T> c, State<T> in, State<T> out, int nw, int rows)
{
    const int item = 4 * xcd_remap(blockIdx.x, gridDim.x) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int chunk = item / nw, w = item - chunk * nw;
    const int y0 = chunk * rows, y1 = min(y0 + rows, c.ny);
    if (y0 >= c.ny) return;
    int xs, l0, l1;
    march::Windows<VX, 2>::window(c.nx, WX && c.bc[0] != BC_PERIODIC, w, nw, xs, l0, l1);
    run<T, VX, WX, AXI>(c, in, out, xs, l0, l1, y0, y1);
}

int compute_units()
{
    static const int ncu = [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            return 256;
        return n;
    }();
    return ncu;
}

// Modelled time of one launch in us, fitted to 380 measured shapes (96 x 96 to
// 2048 x 1024, 2.6 % rms).  us[w - 1]: time of one row of one wave, per wave,
// when w waves share a SIMD; more waves than a SIMD holds run one round after
// the other.  3.1 rows stand for the eight halo rows, which are formed in part.
// extra: factor on the rows' time.
constexpr double LAUNCH_US = 2.9;
double launch_us(int vx, int nw, int ny, int rows, bool f64, bool axi, double bytes, double extra = 1.0)
{
    static const double f32_1[4] = {0.593, 0.398, 0.369, 0.329}, f32_2[2] = {0.838, 0.618}, f64_1[2] = {0.775, 0.575};
    const double* us = f64 ? f64_1 : vx == 2 ? f32_2 : f32_1;
    const int ncu = compute_units();
    const int nb = (nw * ((ny + rows - 1) / rows) + 3) / 4, held = us == f32_1 ? 4 : 2;
    const int whole = (nb + ncu - 1) / ncu, full = whole / held, rest = whole % held;
    double alu = full * held * us[held - 1] + (rest ? rest * us[rest - 1] : 0.0);
    if (whole > 2) alu *= (0.19 * nb / ncu + 0.81 * whole) / whole;
    alu *= (rows + 3.1) * (axi ? 1.05 : 1.0) * extra;
    const double mem = bytes * (1.0 + 2.0 / rows) / (bytes < 230e6 ? 8.1e6 : 5.5e6);
    return LAUNCH_US + std::max(alu, mem) + 0.3 * std::min(alu, mem);
}

// Launch shape: columns per lane and rows per chunk; vx = 0: not marched.
struct Plan {
    int vx, rows;
};

// Modelled time in us of the tile kernel's launch (32 x 16 tiles), fitted to
// 1800 measured grids (8 to 4000 columns, 8 to 20000 rows, 4 % rms).  n: tiles
// per compute unit.
double tiles_us(double n, bool f64, bool axi, bool walls)
{
    const double c = std::ceil(n);
    if (axi) return f64 ? 7.5 + 0.28 * n + 2.33 * c : 7.8 + 0.21 * n + 1.19 * c;
    return (f64 ? 5.8 + 0.45 * n + 1.81 * c : 5.9 + 0.16 * n + 1.05 * c) + (walls ? 0.75 : 0.0);
}

// The shape with the least modelled time.  Not marched: wetting walls (their
// ghosts take a rule of their own), rho0 != 1, and grids on which the tile
// kernel is ahead: those whose rows fill few of the lanes, and some of few
// rows or few tiles.  us per step, tiles and march: 16 x 15602 axisymmetric
// doubles 17.1 and 22.0, 1632 x 78 doubles 9.1 and 10.3, 1983 x 174 8.8 and 9.8,
// 512 x 512 doubles 10.5 and 11.0; but 512 x 400 doubles 10.9 and 10.2, 1024 x
// 1024 18.3 and 14.5.
template <typename T>
Plan plan(const Coef<T>& c, bool axi)
{
    Plan best{0, 0};
    const bool f64 = sizeof(T) == 8, wall = c.bc[0] != BC_PERIODIC;
    const double nodes = (double)c.nx * c.ny;
    if (c.wet || c.rho0 != T(1) || nodes * sizeof(T) >= 2147483648.0) return best;
    double least = 0.0;
    for (int vx = 1; vx <= (f64 ? 1 : 2); ++vx) {
        if (vx == 2 && !march::Windows<2, 2>::fits(c.nx, wall)) continue;
        const int nw = vx == 2 ? march::Windows<2, 2>::count(c.nx, wall) : march::Windows<1, 2>::count(c.nx, wall);
        for (int r = 1; r <= 64 && r <= c.ny; ++r) {
            const double t = launch_us(vx, nw, c.ny, r, f64, axi, 8.0 * nodes * sizeof(T));
            if (best.vx == 0 || t < least) best = Plan{vx, r}, least = t;
        }
    }
    const double n = (double)((c.nx + 31) / 32) * ((c.ny + 15) / 16) / compute_units();
    // not in the model: the x faces' selects, and what wide grids of few rows take
    // more (7 to 14 % beyond 1300 columns)
    double extra = wall ? 1.16 : 1.02;
    if (c.ny < 170 && c.nx > 800) extra *= 1.0 + 0.12 * std::log2(std::min(c.nx, 1600) / 800.0);
    const int nw = best.vx == 2 ? march::Windows<2, 2>::count(c.nx, wall) : march::Windows<1, 2>::count(c.nx, wall);
    const double us = launch_us(best.vx, nw, c.ny, best.rows, f64, axi, 8.0 * nodes * sizeof(T), extra);
    if (us > 0.97 * tiles_us(n, f64, axi, c.nonperiodic != 0)) best.vx = 0;
    return best;
}

template <typename T, int VX, bool AXI>
hipError_t launch_vx(const Coef<T>& c, const State<T>& in, const State<T>& out, int rows, hipStream_t s)
{
    const bool wall = c.bc[0] != BC_PERIODIC;
    const int nw = march::Windows<VX, 2>::count(c.nx, wall);
    const int nb = (nw * ((c.ny + rows - 1) / rows) + 3) / 4;
    if (wall)
        hipLaunchKernelGGL((twophase_march_kernel<T, VX, true, AXI>), dim3(nb), dim3(256), 0, s, c, in, out, nw, rows);
    else
        hipLaunchKernelGGL((twophase_march_kernel<T, VX, false, AXI>), dim3(nb), dim3(256), 0, s, c, in, out, nw, rows);
    return hipGetLastError();
}

}  // namespace march2p

template <typename T, int TX, int TY, int NT, bool AXI>
static hipError_t launch2p_variant(const Coef<T>& c, const State<T>& in, const State<T>& out, hipStream_t s)
{
    const int nbx = (c.nx + TX - 1) / TX, nby = (c.ny + TY - 1) / TY;
    hipLaunchKernelGGL((twophase2d_kernel<T, TX, TY, NT, AXI>), dim3(nbx * nby), dim3(NT), 0, s, c, in, out, nbx);
    return hipGetLastError();
}

template <typename T, bool AXI>
static hipError_t launch2p(const Coef<T>& c, const State<T>& in, const State<T>& out, int tile, hipStream_t s)
{
    if (tile == 0) {
        const march2p::Plan p = march2p::plan(c, AXI);
        if constexpr (sizeof(T) == 4)
            if (p.vx == 2) return march2p::launch_vx<T, 2, AXI>(c, in, out, p.rows, s);
        if (p.vx == 1) return march2p::launch_vx<T, 1, AXI>(c, in, out, p.rows, s);
    }
    switch (tile) {
        case 1: return launch2p_variant<T, 32, 8, 256, AXI>(c, in, out, s);
        case 2: return launch2p_variant<T, 64, 8, 256, AXI>(c, in, out, s);
        case 3: return launch2p_variant<T, 16, 16, 256, AXI>(c, in, out, s);
        default: return launch2p_variant<T, 32, 16, 256, AXI>(c, in, out, s);
    }
}

template <typename T>
hipError_t launch_twophase2d(const Coef<T>& c, const State<T>& in, const State<T>& out, int tile, hipStream_t s)
{
    return launch2p<T, false>(c, in, out, tile, s);
}

template <typename T>
hipError_t launch_twophase_axisym2d(const Coef<T>& c, const State<T>& in, const State<T>& out, int tile,
                                    hipStream_t s)
{
    return launch2p<T, true>(c, in, out, tile, s);
}

template hipError_t launch_twophase2d<float>(const Coef<float>&, const State<float>&, const State<float>&, int, hipStream_t);
template hipError_t launch_twophase2d<double>(const Coef<double>&, const State<double>&, const State<double>&, int, hipStream_t);
template hipError_t launch_twophase_axisym2d<float>(const Coef<float>&, const State<float>&, const State<float>&, int,
                                                    hipStream_t);
template hipError_t launch_twophase_axisym2d<double>(const Coef<double>&, const State<double>&, const State<double>&,
                                                     int, hipStream_t);

}  // namespace acm
