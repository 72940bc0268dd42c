// 2D single-phase SMAME step as a register march along y: LV steps in one
// pass over the state, no LDS and no barrier.  Shared by the single-case
// launches (kern_march2d.hip) and the batched launch (kern_batch.hip).
//
// What bounds the step and why this layout.  A step reads and writes 24
// bytes per node and evaluates about 75 FP32 instructions; a tile kernel adds
// as many again for LDS traffic, region coordinates and the halo of every
// tile, and pays three latencies (load, two barriers) and a launch per step.
// Here a wave owns a window of 64 VX columns (lane l holds VX consecutive
// ones) and marches it down a chunk of rows:
//  * x neighbours are the lane's own registers or come from the adjacent lane
//    through a wave-wide DPP rotation;
//  * y neighbours are the rows already in registers: each row's momenta and
//    fluxes are formed once and used as north, centre and south;
//  * rows are fetched PD ahead, so the loads of later rows are in flight while
//    earlier ones compute;
//  * a finished row of step n+1 is the input row of step n+2 right away (the
//    next level), so LV steps cost one read and one write of the state.
// A level needs one row of drho' on both sides and one more of the fields, so
// level l runs 2 (LV - l) rows and columns past the owned ones on each side;
// the window's outer columns hold partial results there, which are never
// stored.  Every value is formed by the expressions of tile2d.h (axisymmetric
// runs: kern_axisym.h) in the same order, so the state does not depend on the
// kernel, the window or LV.
//
// Walls and symmetry planes: at each level the ghost row beyond a y face is
// its mirror row with the face's velocity rule, and drho' of a ghost is that
// of its mirror; beyond an x face the neighbour of the outermost node is
// formed from that node.  No corner ghost is ever read in 2D.
#pragma once

#include <type_traits>

#include "acm_internal.h"
#include "kern_axisym.h"
#include "tile2d.h"

namespace acm {
namespace march {

// rows fetched ahead: a row of 128 columns and two levels takes over a
// microsecond, so one is enough there, and with it the kernel fits three waves
// per SIMD (two where x faces are walls)
constexpr int rows_ahead(int vx, int lv) { return vx * lv >= 4 ? 1 : 2; }

// Windows of one row of nx nodes: 64 VX columns each, HL lanes of halo
// between neighbouring windows (2 LV columns).  wall: the x faces are walls or
// symmetry planes (the outermost windows then begin at node 0 and end at node
// nx - 1 and need no halo there), else periodic (a row of exactly 64 VX nodes
// is closed by the rotation itself; otherwise columns wrap modulo nx).
template <int VX, int LV>
struct Windows {
    static constexpr int HL = (2 * LV + VX - 1) / VX;  // halo lanes
    static constexpr int NV = 64 - 2 * HL;             // lanes between the halos
    static constexpr int WID = 64 * VX;

    // A walled row must end on a lane's last node: one window when VX divides
    // nx, else several, the last one aligned to the end.  A periodic row must
    // wrap between two lanes, and no lane holds both ends.
    __host__ __device__ static bool fits(int nx, bool wall) { return (nx % VX == 0 && nx >= 2 * VX) || (wall && nx >= WID); }
    __host__ __device__ static int count(int nx, bool wall)
    {
        if (wall) return nx <= WID ? 1 : (nx - 2 * HL * VX + NV * VX - 1) / (NV * VX);
        return nx == WID ? 1 : ((nx + VX - 1) / VX + NV - 1) / NV;
    }
    // first column of window i (may be negative: periodic halo) and the lanes that store
    __host__ __device__ static void window(int nx, bool wall, int i, int n, int& xs, int& l0, int& l1)
    {
        if (wall) {
            const int last = nx <= WID ? 0 : nx - WID;
            xs = i == n - 1 ? last : i * NV * VX;
            l0 = i == 0 ? 0 : HL;
            l1 = i == n - 1 ? (nx <= WID ? nx / VX : 64) : 64 - HL;
        } else if (nx == WID) {
            xs = 0;
            l0 = 0;
            l1 = 64;
        } else {
            const int lanes = (nx + VX - 1) / VX - i * NV;  // lanes still to store
            xs = (i * NV - HL) * VX;
            l0 = HL;
            l1 = HL + (lanes < NV ? lanes : NV);
        }
    }
};

// wave-wide rotations by one lane (DPP): the value of the lane below (lane 0
// gets lane 63's) or above
template <int CTRL>
__device__ __forceinline__ float rot1(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ double rot1(double x)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
    const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)b, CTRL, 0xF, 0xF, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ float lane_value(float x, int l)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), l));
}
__device__ __forceinline__ double lane_value(double x, int l)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), l);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
template <typename T>
__device__ __forceinline__ T lane_below(T x) { return rot1<0x13C>(x); }
template <typename T>
__device__ __forceinline__ T lane_above(T x) { return rot1<0x134>(x); }

// VX consecutive values of one row by one buffer access: descriptor of the
// whole field (below 2 GiB), per-lane byte offset, row's byte offset in the
// scalar operand.  An access past the descriptor's end is dropped.  (The
// builtins return integer vectors; they are cast whole before an element is
// read.)
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
template <typename T, int VX>
__device__ __forceinline__ void row_load(T (&d)[VX], __amdgpu_buffer_rsrc_t p, unsigned off, unsigned soff)
{
    constexpr int B = VX * (int)sizeof(T);
    static_assert(B == 4 || B == 8 || B == 16, "one buffer access per lane");
    if constexpr (VX == 1 && B == 4) {
        d[0] = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(p, off, soff, 0));
    } else if constexpr (VX == 1) {
        d[0] = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(p, off, soff, 0));
    } else {
        typedef T V __attribute__((ext_vector_type(VX)));
        V q;
        if constexpr (B == 8) q = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(p, off, soff, 0));
        else q = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(p, off, soff, 0));
#pragma unroll
        for (int j = 0; j < VX; ++j) d[j] = q[j];
    }
}
template <typename T, int VX>
__device__ __forceinline__ void row_store(const T (&d)[VX], __amdgpu_buffer_rsrc_t p, unsigned off, unsigned soff)
{
    constexpr int B = VX * (int)sizeof(T);
    if constexpr (VX == 1 && B == 4) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, d[0]), p, off, soff, 0);
    } else if constexpr (VX == 1) {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, d[0]), p, off, soff, 0);
    } else {
        typedef T V __attribute__((ext_vector_type(VX)));
        V q;
#pragma unroll
        for (int j = 0; j < VX; ++j) q[j] = d[j];
        if constexpr (B == 8) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, q), p, off, soff, 0);
        else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, q), p, off, soff, 0);
    }
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t field_rsrc(const void* base, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}

// east and west neighbours of a lane's nodes
template <typename T, int VX>
__device__ __forceinline__ void east_west(const T (&f)[VX], T (&e)[VX], T (&w)[VX])
{
#pragma unroll
    for (int j = 0; j + 1 < VX; ++j) {
        e[j] = f[j + 1];
        w[j + 1] = f[j];
    }
    e[VX - 1] = lane_above(f[0]);
    w[0] = lane_below(f[VX - 1]);
}

// m = u + drho u (rho0 = 1)
template <typename T>
__device__ __forceinline__ T mom1(T r, T u) { return fmaT(r, u, u); }

// registers of one level, by row modulo 6 (fields) and modulo 3 (values
// derived from a row); only the rows still needed are live
template <typename T, int VX>
struct Level {
    T r[6][VX], u[6][VX], v[6][VX];
    T mx[3][VX], my[3][VX], pxy[3][VX], pyy[3][VX];  // momenta, fluxes m_x v and m_y v + cs^2 drho
    T rn[3][VX], gr[3][VX];                          // drho', drho_E - drho_W
};

// The walled ends of a row, as a lane sees them.
template <typename T>
struct Edge {
    bool l, r;     // this lane's first / last node is the first / last node of a walled row
    bool any;      // some lane's is (wave-uniform)
    T s[2], o[2];  // the face's velocity rule u_g = s u + o (u, v), per lane
};

struct NoForce {};

// Row n (slot J of the level's ring) has arrived: drho' of row n - 1, then
// the new state of row n - 2 into (ro, uo, vo) when that row is wanted
// (>= mlo; returns whether it was formed).  fst: the two-phase force on row
// n - 2, -dt phi G_iso mu (fst[axis][node]), or NoForce.
template <int J, typename T, int VX, bool WX, bool WY, bool AXI, typename IR, typename FR, typename FS = NoForce>
__device__ __forceinline__ bool push(const Coef<T>& c, Level<T, VX>& L, int row, int mlo, bool wally, const Edge<T>& eg,
                                     const IR& inv_r, const FR& force, T (&ro)[VX], T (&uo)[VX], T (&vo)[VX],
                                     const FS& fst = FS())
{
    constexpr int n = J % 6, k = (J + 5) % 6, m = (J + 4) % 6, s = (J + 3) % 6;
    constexpr int dk = (J + 2) % 3, dm = (J + 1) % 3, ds = J % 3;
    const T rho0 = T(1), cs2 = c.cs2;
    if (WY && wally) {
        if (row == 0) {  // the ghost row below the grid
#pragma unroll
            for (int j = 0; j < VX; ++j) {
                L.r[k][j] = L.r[n][j];
                L.u[k][j] = fmaT(c.fs[2][0], L.u[n][j], c.fo[2][0]);
                L.v[k][j] = fmaT(c.fs[2][1], L.v[n][j], c.fo[2][1]);
            }
        }
        if (row == c.ny) {  // the ghost row above it
#pragma unroll
            for (int j = 0; j < VX; ++j) {
                L.r[n][j] = L.r[k][j];
                L.u[n][j] = fmaT(c.fs[3][0], L.u[k][j], c.fo[3][0]);
                L.v[n][j] = fmaT(c.fs[3][1], L.v[k][j], c.fo[3][1]);
            }
        }
    }
    // momenta and y fluxes of row n - 1
#pragma unroll
    for (int j = 0; j < VX; ++j) {
        const T r = L.r[k][j], v = L.v[k][j];
        L.mx[dk][j] = mom1(r, L.u[k][j]);
        L.my[dk][j] = mom1(r, v);
        L.pxy[dk][j] = L.mx[dk][j] * v;
        L.pyy[dk][j] = fmaT(L.my[dk][j], v, cs2 * r);
    }
    if (row - 1 < mlo - 1) return false;
    // drho' of row n - 1
    {
        T rE[VX], rW[VX], uE[VX], uW[VX];
        east_west(L.r[k], rE, rW);
        east_west(L.u[k], uE, uW);
        if (WX && eg.any) {
            // the ghost beside the lane's outer node (a lane has at most one)
            const T r = eg.l ? L.r[k][0] : L.r[k][VX - 1];
            const T u = fmaT(eg.s[0], eg.l ? L.u[k][0] : L.u[k][VX - 1], eg.o[0]);
            rW[0] = eg.l ? r : rW[0];
            uW[0] = eg.l ? u : uW[0];
            rE[VX - 1] = eg.r ? r : rE[VX - 1];
            uE[VX - 1] = eg.r ? u : uE[VX - 1];
        }
        const T irk = AXI ? inv_r(row - 1) : T(0);
#pragma unroll
        for (int j = 0; j < VX; ++j) {
            const T rc = L.r[k][j], rN = L.r[n][j], rS = L.r[m][j];
            const T vN = L.v[n][j], vS = L.v[m][j];
            T div, lap;
            if constexpr (AXI) {
                axi_continuity(rho0, T(row - 1), irk, rc, rE[j], rW[j], rN, rS, uE[j], uW[j], L.v[k][j], vN, vS,
                               div, lap);
            } else {
                div = mdiff(rE[j], uE[j], rW[j], uW[j], rho0) + mdiff(rN, vN, rS, vS, rho0);
                lap = fmaT(T(-4), rc, (rE[j] + rW[j]) + (rN + rS));  // 4 rc is exact
            }
            L.rn[dk][j] = fmaT(-c.cg, div, fmaT(c.kr, lap, rc));
            L.gr[dk][j] = rE[j] - rW[j];
        }
        if (WY && wally) {  // a ghost row's drho' is its mirror row's
            if (row == 1) {
#pragma unroll
                for (int j = 0; j < VX; ++j) L.rn[dm][j] = L.rn[dk][j];
            }
            if (row - 1 == c.ny) {
#pragma unroll
                for (int j = 0; j < VX; ++j) L.rn[dk][j] = L.rn[dm][j];
            }
        }
    }
    if (row - 2 < mlo) return false;
    // momentum update of row n - 2 (as momentum_node2d_at)
    T xx[VX], yx[VX], a[VX], b[VX], q[VX], xxE[VX], xxW[VX], yxE[VX], yxW[VX], aE[VX], aW[VX], bE[VX], bW[VX];
    T qE[VX], qW[VX];
#pragma unroll
    for (int j = 0; j < VX; ++j) {
        a[j] = L.mx[dm][j];
        b[j] = L.my[dm][j];
        q[j] = L.rn[dm][j];
        xx[j] = fmaT(a[j], L.u[m][j], cs2 * L.r[m][j]);
        yx[j] = b[j] * L.u[m][j];
    }
    east_west(xx, xxE, xxW);
    east_west(yx, yxE, yxW);
    east_west(a, aE, aW);
    east_west(b, bE, bW);
    east_west(q, qE, qW);
    if (WX && eg.any) {
        const T r = eg.l ? L.r[m][0] : L.r[m][VX - 1];
        const T u = fmaT(eg.s[0], eg.l ? L.u[m][0] : L.u[m][VX - 1], eg.o[0]);
        const T v = fmaT(eg.s[1], eg.l ? L.v[m][0] : L.v[m][VX - 1], eg.o[1]);
        const T ga = mom1(r, u), gb = mom1(r, v);
        const T gxx = fmaT(ga, u, cs2 * r), gyx = gb * u;
        xxW[0] = eg.l ? gxx : xxW[0];
        yxW[0] = eg.l ? gyx : yxW[0];
        aW[0] = eg.l ? ga : aW[0];
        bW[0] = eg.l ? gb : bW[0];
        qW[0] = eg.l ? q[0] : qW[0];
        xxE[VX - 1] = eg.r ? gxx : xxE[VX - 1];
        yxE[VX - 1] = eg.r ? gyx : yxE[VX - 1];
        aE[VX - 1] = eg.r ? ga : aE[VX - 1];
        bE[VX - 1] = eg.r ? gb : bE[VX - 1];
        qE[VX - 1] = eg.r ? q[VX - 1] : qE[VX - 1];
    }
    const T irm = AXI ? inv_r(row - 2) : T(0);
    const T gx = force(row - 2);
#pragma unroll
    for (int j = 0; j < VX; ++j) {
        const T rc = L.r[m][j], uc = L.u[m][j], vc = L.v[m][j];
        const T rN = L.r[k][j], rS = L.r[s][j];
        const T mxN = L.mx[dk][j], mxS = L.mx[ds][j], myN = L.my[dk][j], myS = L.my[ds][j];
        T fxx, fyy, lx, ly;
        if constexpr (AXI) {
            // axi_momentum (kern_axisym.h) on the shared per-row values
            const T g = T(row - 2), irc = irm;
            const T pxyN = L.pxy[dk][j], pyyN = L.pyy[dk][j];
            fxx = (xxE[j] - xxW[j]) + axi_div_r(g, irc, pxyN - L.pxy[ds][j], L.pxy[dm][j] + pxyN);
            fyy = (yxE[j] - yxW[j]) + axi_div_r(g, irc, pyyN - L.pyy[ds][j], L.pyy[dm][j] + pyyN) -
                  T(2) * cs2 * rc * irc;
            lx = fmaT(T(-2), a[j], aE[j] + aW[j]) + axi_lap_r(g, irc, a[j], mxN, mxS);
            ly = fmaT(T(-2), b[j], bE[j] + bW[j]) + axi_lap_r(g, irc, b[j], myN, myS) - b[j] * irc * irc;
        } else {
            fxx = (xxE[j] - xxW[j]) + (L.pxy[dk][j] - L.pxy[ds][j]);
            fyy = (yxE[j] - yxW[j]) + (L.pyy[dk][j] - L.pyy[ds][j]);
            lx = fmaT(T(-4), a[j], (aE[j] + aW[j]) + (mxN + mxS));
            ly = fmaT(T(-4), b[j], (bE[j] + bW[j]) + (myN + myS));
        }
        const T rnC = q[j];
        const T sx = (qE[j] - qW[j]) - L.gr[dm][j];
        const T sy = (L.rn[dk][j] - L.rn[ds][j]) - (rN - rS);
        const T rho_n = rho0 + rnC;
        T px = -c.cg * fxx, py = -c.cg * fyy;
        if constexpr (!std::is_same<FS, NoForce>::value) {
            px = fmaT(-c.cg, fxx, fst[0][j]);
            py = fmaT(-c.cg, fyy, fst[1][j]);
        }
        const T dmx = fmaT(rho_n, gx, fmaT(-c.ks, sx, fmaT(c.kv, lx, px)));
        const T dmy = fmaT(rho_n, c.gdt[1], fmaT(-c.ks, sy, fmaT(c.kv, ly, py)));
        const T drn = rnC - rc;
        const T inv = recipT(rho_n);
        ro[j] = rnC;
        uo[j] = fmaT(fmaT(-uc, drn, dmx), inv, uc);
        vo[j] = fmaT(fmaT(-vc, drn, dmy), inv, vc);
    }
    return true;
}

// LV steps of rows y0 .. y1 - 1 on the window starting at column xs; lanes
// l0 .. l1 - 1 store.  WX, WY: the x, the y faces may be walls or symmetry planes.
template <typename T, int VX, int LV, bool WX, bool WY, bool AXI>
__device__ __forceinline__ void run(const Coef<T>& c, const State<T>& in, const State<T>& out, int xs, int l0, int l1,
                                    int y0, int y1)
{
    const int nx = c.nx, ny = c.ny, lane = threadIdx.x & 63;
    const bool wallx = WX && c.bc[0] != BC_PERIODIC, wally = WY && c.bc[2] != BC_PERIODIC;
    const unsigned pitch = (unsigned)nx * (unsigned)sizeof(T), fbytes = pitch * (unsigned)ny;
    // the lane's columns x .. x + VX - 1
    int x = xs + VX * lane;
    if (wallx) {
        x = min(x, nx - VX);  // lanes past a short row repeat its last nodes
    } else {
        x = x < 0 ? x + nx : (x >= nx ? x - nx : x);
        if (x < 0 || x >= nx) x = ((x % nx) + nx) % nx;  // rows shorter than the halo
    }
    const unsigned loff = (unsigned)x * (unsigned)sizeof(T);
    const unsigned soff = (lane >= l0 && lane < l1) ? loff : fbytes;  // past the end: dropped
    Edge<T> eg;
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

    const __amdgpu_buffer_rsrc_t ir = field_rsrc(in.r, fbytes), iu = field_rsrc(in.u, fbytes),
                                 iv = field_rsrc(in.v, fbytes), qr = field_rsrc(out.r, fbytes),
                                 qu = field_rsrc(out.u, fbytes), qv = field_rsrc(out.v, fbytes);
    Level<T, VX> L[LV];
    int yf = 0;  // next row to fetch, inside the grid
    auto fetch = [&](auto slot) {
        constexpr int sl = decltype(slot)::value;
        const unsigned o = (unsigned)yf * pitch;
        row_load<T, VX>(L[0].r[sl], ir, loff, o);
        row_load<T, VX>(L[0].u[sl], iu, loff, o);
        row_load<T, VX>(L[0].v[sl], iv, loff, o);
        // past a walled face the last row again (replaced by its ghost or never used)
        yf = yf + 1 == ny ? (wally ? yf : 0) : yf + 1;
    };

    // first row read, last row pushed; a walled bottom face has no rows below 0
    const int nb = wally ? max(y0 - 2 * LV, 0) : y0 - 2 * LV;
    const int ne = y1 + 2 * LV - 1;
    // first row wanted of level l (0-based)
    auto first = [&](int l) {
        const int f = y0 - 2 * (LV - 1 - l);
        return wally ? max(f, 0) : f;
    };
    // rows before the first: zero, so that nothing undefined enters the rings
#pragma unroll
    for (int l = 0; l < LV; ++l)
#pragma unroll
        for (int q = 0; q < 6; ++q)
#pragma unroll
            for (int j = 0; j < VX; ++j) {
                L[l].r[q][j] = L[l].u[q][j] = L[l].v[q][j] = T(0);
                if (q < 3) {
                    L[l].mx[q][j] = L[l].my[q][j] = L[l].pxy[q][j] = L[l].pyy[q][j] = T(0);
                    L[l].rn[q][j] = L[l].gr[q][j] = T(0);
                }
            }
    yf = nb < 0 ? nb + ny : nb;
    if (yf < 0) yf = ((nb % ny) + ny) % ny;
    constexpr int PD = rows_ahead(VX, LV);
    fetch(std::integral_constant<int, 0>{});
    if constexpr (PD == 2) fetch(std::integral_constant<int, 1>{});

    // Row values of 64 rows at a time, lane l holding row ib + l: dt times the
    // x force, and 1 / (row + 1/2) (axisymmetric).
    int ib = nb;
    T irv = T(0), fxv = c.gdt[0];
    auto fill = [&](int from) {
        ib = from;
        if (AXI) irv = T(1) / (T(from + lane) + T(0.5));
        if (c.fx) {
            int y = from + lane;  // rows outside the grid: the wrapped row's (periodic; else not used)
            y = y < 0 ? y + ny : (y >= ny ? y - ny : y);
            if (y < 0 || y >= ny) y = ((y % ny) + ny) % ny;
            fxv = fmaT(c.dt, c.fx[y], c.gdt[0]);
        }
    };
    fill(nb);
    auto inv_r = [&](int row) { return lane_value(irv, (row - ib) & 63); };
    auto force = [&](int row) { return lane_value(fxv, (row - ib) & 63); };

    // row n = nb + i, J = i mod 6
    auto iterate = [&](int n, auto jc) {
        constexpr int J = decltype(jc)::value;
        fetch(std::integral_constant<int, (J + PD) % 6>{});
        T r[VX], u[VX], v[VX];
        bool have = push<J, T, VX, WX, WY, AXI>(c, L[0], n, first(0), wally, eg, inv_r, force, r, u, v);
        if constexpr (LV >= 2) {
            constexpr int J1 = (J + 4) % 6;
            if (have) {
#pragma unroll
                for (int j = 0; j < VX; ++j) L[1].r[J1][j] = r[j], L[1].u[J1][j] = u[j], L[1].v[J1][j] = v[j];
                have = push<J1, T, VX, WX, WY, AXI>(c, L[1], n - 2, first(1), wally, eg, inv_r, force, r, u, v);
            }
        }
        if constexpr (LV >= 3) {
            constexpr int J2 = (J + 2) % 6;
            if (have) {
#pragma unroll
                for (int j = 0; j < VX; ++j) L[LV - 1].r[J2][j] = r[j], L[LV - 1].u[J2][j] = u[j], L[LV - 1].v[J2][j] = v[j];
                have = push<J2, T, VX, WX, WY, AXI>(c, L[LV - 1], n - 4, first(2), wally, eg, inv_r, force, r, u, v);
            }
        }
        // No memory access stands in a branch: the waits for a row's loads then
        // leave the later rows' loads and the stores in flight.  A row not
        // formed is stored past the end, which drops it.
        const unsigned so = have ? soff : fbytes, o = have ? (unsigned)(n - 2 * LV) * pitch : 0u;
        row_store<T, VX>(r, qr, so, o);
        row_store<T, VX>(u, qu, so, o);
        row_store<T, VX>(v, qv, so, o);
    };
    static_assert(LV >= 1 && LV <= 3, "one to three levels");
    int n = nb;
    for (;;) {
        if (n - ib >= 48 && (AXI || c.fx)) fill(n - 2 * LV);  // the next six pushes use rows n - 2 LV .. n + 4
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
