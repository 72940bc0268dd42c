// Two-phase SMAME step in 3D for gfx950: the flow update with the
// surface-tension force and the Cahn-Hilliard equation (Eq. 2.14) by Heun's
// method, as three launches per step (Sec. 2, two-phase paragraphs):
//   1. mu      = 4 a phi (phi^2 - 1) - kappa L_iso phi on the tile and its ring,
//      then F_a = phi G_iso,a mu;  phi* = phi + dt (M L_iso mu - u_a G_iso,a phi)
//   2. flow    = single-phase 3D step (Eqs. 2.10-2.11) with -dt F_a added to the momentum
//   3. mu*     = mu(phi*) on the tile and its ring,
//      then phi^{n+1} = (phi + phi* + dt (M L_iso mu* - u_a G_iso,a phi*)) / 2
// u is u^n in both Heun stages.  Isotropic stencils with D3Q19 weights:
//   G_iso,a f = [2 (f_{+a} - f_{-a}) + sum_{b != a} (f_{+a+b} + f_{+a-b} - f_{-a+b} - f_{-a-b})] / (12 dx)
//   L_iso f   = [2 (sum of the 6 face neighbours) + (sum of the 12 edge neighbours) - 24 f] / (6 dx^2)
// Ghosts: mu is mirrored across walls and symmetry planes (no flux); phi
// and phi* are mirrored, then take the wetting rule of each crossed wall
// face (x, y, z order).  One thread per node; phi is staged per workgroup in
// LDS with a two-node halo, mu is formed in LDS on the tile plus a one-node
// ring (a wall or symmetry ghost takes the value of its mirror node, a
// periodic ghost is formed from wrapped data and equals its image), so mu
// never goes through global memory.
#include <algorithm>

#include "acm_internal.h"
#include "march3d.h"

namespace acm {

namespace {

// value of a scalar field at node (i, j, k), which may lie one layer outside
// the grid; WET applies the wetting rule across wall faces, with the face's
// coefficient from the table wbt (LDS: a per-lane lookup there costs no
// scratch memory, unlike one into the kernel arguments)
template <bool WET, typename T>
__device__ __forceinline__ T at(const Coef<T>& c, const T* __restrict__ f, int i, int j, int k, const T* wbt)
{
    int fx, fy, fz;
    const int si = map_coord(i, c.nx, c.bc[0], 0, fx);
    const int sj = map_coord(j, c.ny, c.bc[2], 2, fy);
    const int sk = map_coord(k, c.nz, c.bc[4], 4, fz);
    T v = f[((size_t)sk * c.ny + sj) * c.nx + si];
    if constexpr (WET) {
        if (c.wet) {
            if (fx >= 0) v = wet_ghost(v, wbt[fx]);
            if (fy >= 0) v = wet_ghost(v, wbt[fy]);
            if (fz >= 0) v = wet_ghost(v, wbt[fz]);
        }
    }
    return v;
}

// numerators (the 1/(12 dx) and 1/(6 dx^2) factors are applied by the caller)
template <typename T>
__device__ __forceinline__ T lap_num(const T n[3][3][3])
{
    const T ax = ((n[2][1][1] + n[0][1][1]) + (n[1][2][1] + n[1][0][1])) + (n[1][1][2] + n[1][1][0]);
    const T xy = (n[2][2][1] + n[2][0][1]) + (n[0][2][1] + n[0][0][1]);
    const T xz = (n[2][1][2] + n[2][1][0]) + (n[0][1][2] + n[0][1][0]);
    const T yz = (n[1][2][2] + n[1][2][0]) + (n[1][0][2] + n[1][0][0]);
    return fmaT(T(2), ax, (xy + xz) + yz) - T(24) * n[1][1][1];
}
template <typename T>
__device__ __forceinline__ T gx_num(const T n[3][3][3])
{
    const T e = ((n[2][2][1] + n[2][0][1]) - (n[0][2][1] + n[0][0][1])) +
                ((n[2][1][2] + n[2][1][0]) - (n[0][1][2] + n[0][1][0]));
    return fmaT(T(2), n[2][1][1] - n[0][1][1], e);
}
template <typename T>
__device__ __forceinline__ T gy_num(const T n[3][3][3])
{
    const T e = ((n[2][2][1] + n[0][2][1]) - (n[2][0][1] + n[0][0][1])) +
                ((n[1][2][2] + n[1][2][0]) - (n[1][0][2] + n[1][0][0]));
    return fmaT(T(2), n[1][2][1] - n[1][0][1], e);
}
template <typename T>
__device__ __forceinline__ T gz_num(const T n[3][3][3])
{
    const T e = ((n[2][1][2] + n[0][1][2]) - (n[2][1][0] + n[0][1][0])) +
                ((n[1][2][2] + n[1][0][2]) - (n[1][2][0] + n[1][0][0]));
    return fmaT(T(2), n[1][1][2] - n[1][1][0], e);
}

// Workgroup tile BX x BY x BZ nodes; R region = the tile plus a one-node
// ring (mu), P region = the tile plus two nodes (phi, ghost rules applied
// while staging), so a node's neighbours come from LDS instead of 19
// separate global loads.
// Threads BX x BY x TZ; each owns ZR nodes of its column, TZ planes apart,
// so the staged halo is shared by twice the nodes (the tile is BZ = TZ ZR deep).
constexpr int BX = 32, BY = 4, TZ = 4, ZR = 2, BZ = TZ * ZR, NTH = BX * BY * TZ;
constexpr int RX = BX + 2, RY = BY + 2, RZ = BZ + 2, RXYZ = RX * RY * RZ;

// halo-2 region of a staged phi field and the D3Q19 neighbourhood of LDS
// index e in a region of row length SX and plane height SY
constexpr int PX = BX + 4, PY = BY + 4, PZ = BZ + 4, PXYZ = PX * PY * PZ;

template <int SX, int SY, typename T>
__device__ __forceinline__ void nb19at(const T* s, int e, T n[3][3][3])
{
#pragma unroll
    for (int dz = -1; dz <= 1; ++dz)
#pragma unroll
        for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
            for (int dx = -1; dx <= 1; ++dx) {
                if ((dx != 0) + (dy != 0) + (dz != 0) == 3) continue;
                n[1 + dx][1 + dy][1 + dz] = s[e + dx + SX * (dy + SY * dz)];
            }
}

template <bool WET, typename T>
__device__ __forceinline__ void stage_halo2(const Coef<T>& c, const T* __restrict__ f, int i0, int j0, int k0, T* s,
                                            const T* wbt)
{
    const int tid = threadIdx.x + BX * (threadIdx.y + BY * threadIdx.z);
    constexpr int NIT = (PXYZ + NTH - 1) / NTH;
    T v[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int q = min(tid + it * NTH, PXYZ - 1);
        const int lz = q / (PX * PY), r = q - lz * (PX * PY), ly = r / PX, lx = r - ly * PX;
        v[it] = at<WET>(c, f, i0 + lx - 2, j0 + ly - 2, k0 + lz - 2, wbt);
    }
#pragma unroll
    for (int it = 0; it < NIT; ++it)
        if (tid + it * NTH < PXYZ) s[tid + it * NTH] = v[it];
}

// mu on the tile plus a one-node ring (R region) from phi staged with halo 2
template <typename T>
__device__ __forceinline__ void mu_ring(const Coef<T>& c, int i0, int j0, int k0, const T* sp, T* sm)
{
    const int tid = threadIdx.x + BX * (threadIdx.y + BY * threadIdx.z);
    for (int q = tid; q < RXYZ; q += NTH) {
        const int lz = q / (RX * RY), r = q - lz * (RX * RY), ly = r / RX, lx = r - ly * RX;
        // source node: the mirror node for a wall / symmetry ghost, else the position itself
        int sx = i0 + lx - 1, sy = j0 + ly - 1, sz = k0 + lz - 1;
        if (c.nonperiodic) {
            sx = mirror_coord(sx, c.nx, c.bc[0]);
            sy = mirror_coord(sy, c.ny, c.bc[2]);
            sz = mirror_coord(sz, c.nz, c.bc[4]);
        }
        // P-region coordinates, clamped (only ragged positions no output reads can leave the range)
        const int px = min(max(sx - i0 + 2, 1), PX - 2), py = min(max(sy - j0 + 2, 1), PY - 2);
        const int pz = min(max(sz - k0 + 2, 1), PZ - 2);
        T n[3][3][3];
        nb19at<PX, PY>(sp, px + PX * (py + PY * pz), n);
        const T p = n[1][1][1];
        sm[q] = fmaT(c.a4 * p, fmaT(p, p, T(-1)), -c.kap6 * lap_num(n));
    }
}

// the wetting coefficients of the six faces into LDS (constant indices only)
template <typename T>
__device__ __forceinline__ void wet_table(const Coef<T>& c, T* wbt)
{
    if (threadIdx.x + threadIdx.y + threadIdx.z == 0) {
        wbt[0] = c.wb[0];
        wbt[1] = c.wb[1];
        wbt[2] = c.wb[2];
        wbt[3] = c.wb[3];
        wbt[4] = c.wb[4];
        wbt[5] = c.wb[5];
    }
    __syncthreads();
}

struct Node {
    int i, j, k;
    bool in;
};
// the thread's r-th node (r < ZR) and its local z in the tile
template <typename T>
__device__ __forceinline__ Node my_node(const Coef<T>& c, int r)
{
    Node n;
    n.i = blockIdx.x * BX + threadIdx.x;
    n.j = blockIdx.y * BY + threadIdx.y;
    n.k = blockIdx.z * BZ + threadIdx.z + TZ * r;
    n.in = n.i < c.nx && n.j < c.ny && n.k < c.nz;
    return n;
}

// mu of phi on the tile and its ring, then F_a = phi G_iso,a mu and
// phi* = phi + dt (M L_iso mu - u_a G_iso,a phi)
template <typename T>
__global__ __launch_bounds__(NTH) void stage1_kernel(Coef<T> c, State<T> in, T* __restrict__ fx,
                                                     T* __restrict__ fy, T* __restrict__ fz, T* __restrict__ phis)
{
    __shared__ T sp[PXYZ], sm[RXYZ], wbt[6];
    const int i0 = blockIdx.x * BX, j0 = blockIdx.y * BY, k0 = blockIdx.z * BZ;
    wet_table(c, wbt);
    stage_halo2<true>(c, in.phi, i0, j0, k0, sp, wbt);
    __syncthreads();
    mu_ring(c, i0, j0, k0, sp, sm);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ZR; ++r) {
        const Node d = my_node(c, r);
        if (!d.in) continue;
        const int lz = threadIdx.z + TZ * r;
        const size_t o = ((size_t)d.k * c.ny + d.j) * c.nx + d.i;
        T m[3][3][3], p[3][3][3];
        nb19at<RX, RY>(sm, (threadIdx.x + 1) + RX * ((threadIdx.y + 1) + RY * (lz + 1)), m);
        nb19at<PX, PY>(sp, (threadIdx.x + 2) + PX * ((threadIdx.y + 2) + PY * (lz + 2)), p);
        const T pc = p[1][1][1];
        fx[o] = pc * (gx_num(m) * c.gi);
        fy[o] = pc * (gy_num(m) * c.gi);
        fz[o] = pc * (gz_num(m) * c.gi);
        const T adv = fmaT(in.u[o], gx_num(p), fmaT(in.v[o], gy_num(p), in.w[o] * gz_num(p))) * c.gi;
        const T rhs = fmaT(c.mob * c.li, lap_num(m), -adv);
        phis[o] = fmaT(c.dt, rhs, pc);
    }
}

// mu* of phi* on the tile and its ring, then
// phi^{n+1} = (phi + phi* + dt (M L_iso mu* - u_a G_iso,a phi*)) / 2
template <typename T>
__global__ __launch_bounds__(NTH) void stage2_kernel(Coef<T> c, State<T> in, const T* __restrict__ phis,
                                                     T* __restrict__ phi_out)
{
    __shared__ T sp[PXYZ], sm[RXYZ], wbt[6];
    const int i0 = blockIdx.x * BX, j0 = blockIdx.y * BY, k0 = blockIdx.z * BZ;
    wet_table(c, wbt);
    stage_halo2<true>(c, phis, i0, j0, k0, sp, wbt);
    __syncthreads();
    mu_ring(c, i0, j0, k0, sp, sm);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ZR; ++r) {
        const Node d = my_node(c, r);
        if (!d.in) continue;
        const int lz = threadIdx.z + TZ * r;
        const size_t o = ((size_t)d.k * c.ny + d.j) * c.nx + d.i;
        T m[3][3][3], p[3][3][3];
        nb19at<RX, RY>(sm, (threadIdx.x + 1) + RX * ((threadIdx.y + 1) + RY * (lz + 1)), m);
        nb19at<PX, PY>(sp, (threadIdx.x + 2) + PX * ((threadIdx.y + 2) + PY * (lz + 2)), p);
        const T adv = fmaT(in.u[o], gx_num(p), fmaT(in.v[o], gy_num(p), in.w[o] * gz_num(p))) * c.gi;
        const T rhs = fmaT(c.mob * c.li, lap_num(m), -adv);
        phi_out[o] = T(0.5) * fmaT(c.dt, rhs, in.phi[o] + p[1][1][1]);
    }
}

// ---------------------------------------------------------------------------
// The two phase-field passes as a register march along z (FP32, no wetting on
// the x faces): a wave owns RY rows of a window of 64 columns, as in
// march3d.h; no LDS, no barrier.  The LDS kernels above stage 3.4 values per
// node and read 37 per node back from LDS.  Here x neighbours come from the
// adjacent lane, and the sums that the D3Q19 stencils share are formed once:
// with s = f_E + f_W, t = f_N + f_S and q = f_U + f_D of a row,
//   xy edges = t_E + t_W, xz edges = q_E + q_W, yz edges = q_N + q_S,
//   G_x = 2 (f_E - f_W) + (t_E - t_W) + (q_E - q_W),
//   G_y = 2 (f_N - f_S) + (s_N - s_S) + (q_N - q_S),
//   G_z = 2 (f_U - f_D) + (s_U - s_D) + (t_U - t_D),
// the sums of lap_num, gx_num, gy_num and gz_num in the same order.
// Bound by instruction issue (vector and scalar together fill the slots; the
// unrolled loops of 36 to 66 KB miss the instruction cache on 2 % of fetches).
// Whole two-phase step, LDS kernels -> march, in us, drop between walls in z:
// 32^3 31.0 -> 16.5, 64^3 33.7 -> 21.9, 96^3 51.5 -> 40.8, 128^3 94 -> 75.
// RY = 4 needs 228 to 256 registers: 55 on 96^3.  Two planes loaded ahead
// instead of one: the same time.  The wetting rule costs 3 us on 96^3: it is
// placed on the few rows and planes that can be ghosts, in one branch each; as
// a loop over the rows with one copy of the rule the step took 49.
// ---------------------------------------------------------------------------
namespace phase {
constexpr int RY = 2;

// one field: values of rows y0 - H .. y0 + RY - 1 + H and their x sums, by plane modulo 6
// (four planes are live, one arrives)
template <int H, int NP>
struct Rows {
    float f[NP][RY + 2 * H], s[NP][RY + 2 * H];
};

// Shape of a march: windows of a row, bands of RY rows, planes per chunk.
struct Shape {
    int nw, nby, zc;
};

// STAGE 1: o0 = phi*, o1..o3 = phi G_iso mu; STAGE 2 (src = phi*): o0 = phi^{n+1}
template <int STAGE>
__device__ __forceinline__ void phase_run(const Coef<float>& c, const State<float>& in, const float* src, float* o0,
                                          float* o1, float* o2, float* o3, const Shape& sh, int item)
{
    const int tt = item / sh.nby, y0 = (item - tt * sh.nby) * RY;
    const int chunk = tt / sh.nw, win = tt - chunk * sh.nw;
    const int z0 = chunk * sh.zc, z1 = min(z0 + sh.zc, c.nz);
    if (z0 >= c.nz) return;
    const int nx = c.nx, ny = c.ny, nz = c.nz, lane = threadIdx.x & 63;
    const bool wallx = c.bc[0] != BC_PERIODIC, wally = c.bc[2] != BC_PERIODIC, wallz = c.bc[4] != BC_PERIODIC;
    int xs, l0, l1;
    march::Windows<1, 1>::window(nx, wallx, win, sh.nw, xs, l0, l1);
    int x = xs + lane;
    if (wallx) {
        x = min(x, nx - 1);
    } else {
        x = x < 0 ? x + nx : (x >= nx ? x - nx : x);
        if (x < 0 || x >= nx) x = ((x % nx) + nx) % nx;
    }
    const bool left = wallx && xs == 0 && lane == 0, right = wallx && xs + lane + 1 == nx;
    const bool edge = wallx && (xs == 0 || xs + 64 >= nx);  // wave-uniform
    const bool st = lane >= l0 && lane < l1;
    const bool endy = wally && (y0 == 0 || y0 + RY >= ny);
    const bool wety = wally && c.wet && (y0 == 0 || y0 + RY + 1 >= ny);
    const unsigned pitch = (unsigned)nx * 4u, pbytes = pitch * (unsigned)ny, fbytes = pbytes * (unsigned)nz;
    const unsigned loff = (unsigned)x * 4u;
    unsigned yoff[RY + 4];
#pragma unroll
    for (int i = 0; i < RY + 4; ++i) {
        int y = y0 - 2 + i;
        if (wally) {
            y = y < 0 ? -1 - y : (y >= ny ? 2 * ny - 1 - y : y);
            y = min(max(y, 0), ny - 1);
        } else {
            y = y < 0 ? y + ny : (y >= ny ? y - ny : y);
            if (y < 0 || y >= ny) y = ((y % ny) + ny) % ny;
        }
        yoff[i] = (unsigned)y * pitch;
    }
    const __amdgpu_buffer_rsrc_t rs = march::field_rsrc(src, fbytes), ru = march::field_rsrc(in.u, fbytes),
                                 rv = march::field_rsrc(in.v, fbytes), rw = march::field_rsrc(in.w, fbytes),
                                 rp = march::field_rsrc(in.phi, fbytes);
    const __amdgpu_buffer_rsrc_t q0 = march::field_rsrc(o0, fbytes), q1 = march::field_rsrc(o1, fbytes),
                                 q2 = march::field_rsrc(o2, fbytes), q3 = march::field_rsrc(o3, fbytes);
    auto plane_in = [&](int p) {
        if (wallz) return min(max(p, 0), nz - 1);
        p = p < 0 ? p + nz : (p >= nz ? p - nz : p);
        return (p < 0 || p >= nz) ? ((p % nz) + nz) % nz : p;
    };
    auto get = [&](__amdgpu_buffer_rsrc_t r, unsigned o) {
        float d[1];
        march::row_load<float, 1>(d, r, loff, o);
        return d[0];
    };
    auto put = [&](float v, __amdgpu_buffer_rsrc_t r, unsigned so, unsigned o) {
        const float d[1] = {v};
        march::row_store<float, 1>(d, r, so, o);
    };
    // neighbours in x; beyond an x face the node itself (mirror; a sum of mirrored values likewise)
    auto east = [&](float v) {
        const float e = march::lane_above(v);
        return edge && right ? v : e;
    };
    auto west = [&](float v) {
        const float w = march::lane_below(v);
        return edge && left ? v : w;
    };

    // phi (or phi*): rows y0 - 2 .. y0 + RY + 1; mu: rows y0 - 1 .. y0 + RY
    Rows<2, 6> P;
    Rows<1, 6> M;
    float vu[2][RY], vv[2][RY], vw[2][RY], vp[2][RY];  // u, v, w (and phi in stage 2) of the output plane
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int i = 0; i < RY + 4; ++i) {
            P.f[q][i] = P.s[q][i] = 0.f;
            if (i < RY + 2) M.f[q][i] = M.s[q][i] = 0.f;
        }
    const int nb = wallz ? max(z0 - 2, -1) : z0 - 2, ne = z1 + 1;
    auto fetch = [&](int p, auto slot) {
        constexpr int sl = decltype(slot)::value;
        const unsigned pz = (unsigned)plane_in(p) * pbytes;
#pragma unroll
        for (int i = 0; i < RY + 4; ++i) P.f[sl][i] = get(rs, pz + yoff[i]);
    };
    auto fetch_velocity = [&](int p, auto slot) {
        constexpr int sl = decltype(slot)::value;
        const unsigned pz = (unsigned)plane_in(p) * pbytes;
#pragma unroll
        for (int i = 0; i < RY; ++i) {
            vu[sl][i] = get(ru, pz + yoff[i + 2]);
            vv[sl][i] = get(rv, pz + yoff[i + 2]);
            vw[sl][i] = get(rw, pz + yoff[i + 2]);
            if (STAGE == 2) vp[sl][i] = get(rp, pz + yoff[i + 2]);
        }
    };
    fetch(nb, std::integral_constant<int, 0>{});
    fetch_velocity(nb - 2, std::integral_constant<int, 0>{});

    // plane n has arrived (slot J): mu of plane n - 1, outputs of plane n - 2
    auto iterate = [&](int n, auto jc) {
        constexpr int J = decltype(jc)::value;
        constexpr int a = J, k = (J + 5) % 6, m = (J + 4) % 6, d = (J + 3) % 6;  // planes n, n - 1, n - 2, n - 3
        fetch(n + 1, std::integral_constant<int, (J + 1) % 6>{});
        fetch_velocity(n - 1, std::integral_constant<int, (J + 1) % 2>{});
        if (wety) {  // wetting rule of the y faces on the ghost rows; y0 is even, so they stand at few places
            if (y0 == 0) P.f[a][1] = wet_ghost(P.f[a][1], c.wb[2]);
            if (y0 + RY + 1 >= ny) {
                const int e = ny - y0;  // 1, 2 or 3: the ghost row is e + 2
                const float g = wet_ghost(e == 1 ? P.f[a][3] : e == 2 ? P.f[a][4] : P.f[a][5], c.wb[3]);
                P.f[a][3] = e == 1 ? g : P.f[a][3];
                P.f[a][4] = e == 2 ? g : P.f[a][4];
                P.f[a][5] = e == 3 ? g : P.f[a][5];
            }
        }
        if (wallz && c.wet && (n == -1 || n == nz)) {  // then of the z faces on a ghost plane
            const float b = n == -1 ? c.wb[4] : c.wb[5];
#pragma unroll
            for (int i = 0; i < RY + 4; ++i) P.f[a][i] = wet_ghost(P.f[a][i], b);
        }
#pragma unroll
        for (int i = 1; i < RY + 3; ++i) P.s[a][i] = east(P.f[a][i]) + west(P.f[a][i]);
        if (n - 1 >= z0 - 1) {
            // mu of plane n - 1 on rows y0 - 1 .. y0 + RY
            float q[RY + 4];
#pragma unroll
            for (int i = 0; i < RY + 4; ++i) q[i] = P.f[a][i] + P.f[m][i];
#pragma unroll
            for (int i = 0; i < RY + 2; ++i) {
                const float p = P.f[k][i + 1], t = P.f[k][i + 2] + P.f[k][i], qc = q[i + 1];
                const float ax = (P.s[k][i + 1] + t) + qc;
                const float xy = east(t) + west(t), xz = east(qc) + west(qc), yz = q[i + 2] + q[i];
                const float lap = fmaT(2.f, ax, (xy + xz) + yz) - 24.f * p;
                M.f[k][i] = fmaT(c.a4 * p, fmaT(p, p, -1.f), -c.kap6 * lap);
            }
            if (endy) {  // mu is mirrored across every face
                if (y0 == 0) M.f[k][0] = M.f[k][1];
#pragma unroll
                for (int i = 2; i < RY + 2; ++i)
                    if (y0 - 1 + i == ny) M.f[k][i] = M.f[k][i - 1];
            }
#pragma unroll
            for (int i = 0; i < RY + 2; ++i) M.s[k][i] = east(M.f[k][i]) + west(M.f[k][i]);
            if (wallz && (n == 1 || n - 1 == nz)) {
#pragma unroll
                for (int i = 0; i < RY + 2; ++i) {
                    if (n == 1) M.f[m][i] = M.f[k][i], M.s[m][i] = M.s[k][i];
                    if (n - 1 == nz) M.f[k][i] = M.f[m][i], M.s[k][i] = M.s[m][i];
                }
            }
        }
        const bool out = n - 2 >= z0;
        float r0[RY], r1[RY], r2[RY], r3[RY];
        if (out) {
            float qp[RY + 2], qm[RY + 2];  // f_U + f_D on rows y0 - 1 .. y0 + RY
#pragma unroll
            for (int i = 0; i < RY + 2; ++i) {
                qp[i] = P.f[k][i + 1] + P.f[d][i + 1];
                qm[i] = M.f[k][i] + M.f[d][i];
            }
#pragma unroll
            for (int i = 0; i < RY; ++i) {
                // phi gradients at row y0 + i (P row i + 2, qp row i + 1)
                const float p = P.f[m][i + 2], tp = P.f[m][i + 3] + P.f[m][i + 1], qc = qp[i + 1];
                const float tU = P.f[k][i + 3] + P.f[k][i + 1], tD = P.f[d][i + 3] + P.f[d][i + 1];
                const float gx = fmaT(2.f, east(p) - west(p), (east(tp) - west(tp)) + (east(qc) - west(qc)));
                const float gy = fmaT(2.f, P.f[m][i + 3] - P.f[m][i + 1],
                                      (P.s[m][i + 3] - P.s[m][i + 1]) + (qp[i + 2] - qp[i]));
                const float gz = fmaT(2.f, P.f[k][i + 2] - P.f[d][i + 2],
                                      (P.s[k][i + 2] - P.s[d][i + 2]) + (tU - tD));
                // mu at the same row (M row i + 1)
                const float mc = M.f[m][i + 1], tm = M.f[m][i + 2] + M.f[m][i], qmc = qm[i + 1];
                const float tE = east(tm), tW = west(tm), qE = east(qmc), qW = west(qmc);
                const float lap = fmaT(2.f, (M.s[m][i + 1] + tm) + qmc, ((tE + tW) + (qE + qW)) + (qm[i + 2] + qm[i])) -
                                  24.f * mc;
                const float adv = fmaT(vu[J % 2][i], gx, fmaT(vv[J % 2][i], gy, vw[J % 2][i] * gz)) * c.gi;
                const float rhs = fmaT(c.mob * c.li, lap, -adv);
                if (STAGE == 1) {
                    const float mU = M.f[k][i + 2] + M.f[k][i], mD = M.f[d][i + 2] + M.f[d][i];
                    const float hx = fmaT(2.f, east(mc) - west(mc), (tE - tW) + (qE - qW));
                    const float hy = fmaT(2.f, M.f[m][i + 2] - M.f[m][i],
                                          (M.s[m][i + 2] - M.s[m][i]) + (qm[i + 2] - qm[i]));
                    const float hz = fmaT(2.f, M.f[k][i + 1] - M.f[d][i + 1],
                                          (M.s[k][i + 1] - M.s[d][i + 1]) + (mU - mD));
                    r1[i] = p * (hx * c.gi);
                    r2[i] = p * (hy * c.gi);
                    r3[i] = p * (hz * c.gi);
                    r0[i] = fmaT(c.dt, rhs, p);
                } else {
                    r0[i] = 0.5f * fmaT(c.dt, rhs, vp[J % 2][i] + p);
                }
            }
        }
        // stores stand outside the branch (march2d.h); rows not formed or past the grid are dropped
        const unsigned pz = out ? (unsigned)(n - 2) * pbytes : 0u;
#pragma unroll
        for (int i = 0; i < RY; ++i) {
            const unsigned so = (out && st && y0 + i < ny) ? loff : fbytes, o = pz + yoff[i + 2];
            put(r0[i], q0, so, o);
            if (STAGE == 1) {
                put(r1[i], q1, so, o);
                put(r2[i], q2, so, o);
                put(r3[i], q3, so, o);
            }
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

__device__ __forceinline__ int item_of_wave(int block, int blocks)
{
    return 4 * xcd_remap(block, blocks) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}

__global__ __launch_bounds__(256) void stage1_march_kernel(Coef<float> c, State<float> in, float* phis, float* fx,
                                                           float* fy, float* fz, Shape sh)
{
    phase_run<1>(c, in, in.phi, phis, fx, fy, fz, sh, item_of_wave(blockIdx.x, gridDim.x));
}

// The flow step with the force and the second phase-field stage need nothing
// of each other: one launch, the first half of the workgroups on the flow.
__global__ __launch_bounds__(256) void flow_stage2_march_kernel(Coef<float> c, State<float> in, State<float> out,
                                                                const float* phis, Shape sh)
{
    const int nbf = gridDim.x / 2;
    if ((int)blockIdx.x >= nbf) {
        phase_run<2>(c, in, phis, out.phi, out.phi, out.phi, out.phi, sh,
                     item_of_wave(blockIdx.x - nbf, nbf));
        return;
    }
    const int item = item_of_wave(blockIdx.x, nbf);
    const int t = item / sh.nby, by = item - t * sh.nby;
    const int chunk = t / sh.nw, w = t - chunk * sh.nw;
    const int z0 = chunk * sh.zc, z1 = min(z0 + sh.zc, c.nz);
    if (z0 >= c.nz) return;
    int xs, l0, l1;
    march::Windows<1, 1>::window(c.nx, c.bc[0] != BC_PERIODIC, w, sh.nw, xs, l0, l1);
    march::run3<float, 1, RY, true, true, true>(c, in, out, xs, l0, l1, by * RY, z0, z1);
}

// The march applies: FP32, no wetting on the x faces (their ghosts are mirrors
// only), rho0 = 1, and the 14 fields of a step (56 bytes per node) within twice
// the 256 MB cache.  Whole steps: 200^3 (448 MB) 324 us with the LDS kernels,
// 270 with the march; 256^3 (940 MB) 581 and 582; 320^3 1007 and 1099.
// Not marched either, being slower than the LDS kernels: rows of up to half a
// window on launches of many waves (13 x 161 x 281 slab 58 us with the LDS
// kernels, 70 marched, 16 x 253 x 33 periodic 30 and 35; with few waves the march
// is ahead: 13 x 10 x 51 24 and 15, and on larger grids again: 18 x 258 x 242 106
// and 90), and rows of whole 64-column tiles that fill at most three quarters
// of the windows, once the fields no longer fit the cache (128 x 254 x 182, 331
// MB, 190 and 219; 192 x 205 x 135, 297 MB, 174 and 189; but 192 x 152 x 151, 246
// MB, 155 and 136).
bool march_ok(const Coef<float>& c)
{
    const double bytes = 56.0 * c.nx * c.ny * c.nz;
    const int nw = march::Windows<1, 1>::count(c.nx, c.bc[0] != BC_PERIODIC);
    const double rows = (double)((c.ny + RY - 1) / RY) * c.nz;  // bands times planes
    const bool narrow = c.nx <= 32 && rows >= 2500.0 && rows < 28000.0;
    const bool gaps = c.nx % 64 == 0 && c.nx <= 48 * nw && bytes > 260e6;
    return c.wb[0] == 0.f && c.wb[1] == 0.f && c.rho0 == 1.f && c.ny >= 2 && c.nz >= 2 && bytes <= 512e6 && !narrow &&
           !gaps;
}

// Planes per chunk so that the waves of one launch are resident together, three
// per SIMD (the registers allow three): longer chunks repeat fewer planes, but
// a wave more than fits starts a second turn.  96^3, stage 1 3 planes: flow and
// stage 2 with 6 and 6 planes (3072 waves of 3072) 40.8 us per step, 6 and 4
// (3840) 43.7, 12 and 4 43.6, 8 and 6 43.6.  Beyond 8 (of one) and 16 planes
// (of two together) the cache loses the neighbouring bands: 160^3 128 us with
// 13 and 25 planes, 116 with 6 and 12.
int chunk_planes(int rows_of_waves, int parts, int most)
{
    static const int ncu = [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            return 256;
        return n;
    }();
    const long long waves = 12ll * ncu;
    return (int)std::min<long long>(most, std::max<long long>(1, ((long long)parts * rows_of_waves + waves - 1) / waves));
}

hipError_t launch_march(const Coef<float>& c, const State<float>& in, const State<float>& out, float* phis,
                        float* const* f, hipStream_t s)
{
    const int nw = march::Windows<1, 1>::count(c.nx, c.bc[0] != BC_PERIODIC), nby = (c.ny + RY - 1) / RY;
    auto blocks = [&](const Shape& sh) { return (nw * nby * ((c.nz + sh.zc - 1) / sh.zc) + 3) / 4; };
    const Shape s1{nw, nby, chunk_planes(nw * nby * c.nz, 1, 8)}, s2{nw, nby, chunk_planes(nw * nby * c.nz, 2, 16)};
    hipLaunchKernelGGL(stage1_march_kernel, dim3(blocks(s1)), dim3(256), 0, s, c, in, phis, f[0], f[1], f[2], s1);
    Coef<float> cf = c;
    for (int a = 0; a < 3; ++a) cf.fst[a] = f[a];
    hipLaunchKernelGGL(flow_stage2_march_kernel, dim3(2 * blocks(s2)), dim3(256), 0, s, cf, in, out, phis, s2);
    return hipGetLastError();
}
}  // namespace phase

}  // namespace

template <typename T>
hipError_t launch_twophase3d(const Coef<T>& c, const State<T>& in, const State<T>& out, T* scratch, int tile,
                             hipStream_t s)
{
    const size_t n = (size_t)c.nx * c.ny * c.nz;
    T* phis = scratch;
    T* f[3] = {scratch + n, scratch + 2 * n, scratch + 3 * n};
    const dim3 block(BX, BY, TZ), grid((c.nx + BX - 1) / BX, (c.ny + BY - 1) / BY, (c.nz + BZ - 1) / BZ);
    if constexpr (sizeof(T) == 4)
        if (tile == 0 && phase::march_ok(c)) return phase::launch_march(c, in, out, phis, f, s);
    hipLaunchKernelGGL(stage1_kernel<T>, grid, block, 0, s, c, in, f[0], f[1], f[2], phis);
    Coef<T> cf = c;
    for (int a = 0; a < 3; ++a) cf.fst[a] = f[a];
    hipError_t e = launch_step3d<T>(cf, in, out, tile, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(stage2_kernel<T>, grid, block, 0, s, c, in, phis, out.phi);
    return hipGetLastError();
}

template hipError_t launch_twophase3d<float>(const Coef<float>&, const State<float>&, const State<float>&, float*,
                                             int, hipStream_t);
template hipError_t launch_twophase3d<double>(const Coef<double>&, const State<double>&, const State<double>&,
                                              double*, int, hipStream_t);

}  // namespace acm
