// 2D single-phase launches of the register march (march2d.h): planar and
// axisymmetric, one to three steps per launch.
//
// Measured per step against the LDS tile kernels (FP32, runs of 100 steps, two
// steps per launch): 1024^2 periodic 8.8 -> 5.9 us, 4096 x 2048 axisymmetric
// pipe 50.5 -> 31 us (a copy of the state takes 23.6), 401 x 257 cavity 4.2 ->
// 3.6 us; 64^2 FP64 3.8 -> 2.4 us.  The march is bound by instruction issue
// (about 65 VALU instructions per node and step, 100 axisymmetric) and, on
// small grids, by the 1.7 us of a launch inside a graph and the serial rows of
// a chunk.
#include <algorithm>

#include "acm_internal.h"
#include "kern_axisym.h"
#include "march2d.h"

namespace acm {

namespace {

template <typename T, int VX, int LV, bool WX, bool WY, bool AXI>
__global__ __launch_bounds__(256) void march2d_kernel(Coef<T> c, State<T> in, State<T> out, int nw, int rows)
{
    using W = march::Windows<VX, LV>;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int item = 4 * xcd_remap(blockIdx.x, gridDim.x) + wave;
    const int chunk = item / nw, w = item - chunk * nw;
    const int y0 = chunk * rows, y1 = min(y0 + rows, c.ny);
    if (y0 >= c.ny) return;
    int xs, l0, l1;
    W::window(c.nx, WX && c.bc[0] != BC_PERIODIC, w, nw, xs, l0, l1);
    march::run<T, VX, LV, WX, WY, AXI>(c, in, out, xs, l0, l1, y0, y1);
}

template <typename T, int VX, int LV, bool WX, bool WY, bool AXI>
hipError_t launch(const Coef<T>& c, const State<T>& in, const State<T>& out, int rows, hipStream_t s)
{
    const int nw = march::Windows<VX, LV>::count(c.nx, c.bc[0] != BC_PERIODIC);
    const int nb = (nw * ((c.ny + rows - 1) / rows) + 3) / 4;
    hipLaunchKernelGGL((march2d_kernel<T, VX, LV, WX, WY, AXI>), dim3(nb), dim3(256), 0, s, c, in, out, nw, rows);
    return hipGetLastError();
}

template <typename T, int VX, int LV>
hipError_t launch_faces(const Coef<T>& c, const State<T>& in, const State<T>& out, bool axi, int rows, hipStream_t s)
{
    const bool wx = c.bc[0] != BC_PERIODIC;
    if (axi && wx) return launch<T, VX, LV, true, true, true>(c, in, out, rows, s);
    if (axi) return launch<T, VX, LV, false, true, true>(c, in, out, rows, s);
    if (wx) return launch<T, VX, LV, true, true, false>(c, in, out, rows, s);
    // Two nodes per lane and two steps: without the y faces' code the compiler
    // takes 171 registers (two waves per SIMD), with it 166 (three).
    if constexpr (VX * LV == 4) return launch<T, VX, LV, false, true, false>(c, in, out, rows, s);
    else if (c.nonperiodic) return launch<T, VX, LV, false, true, false>(c, in, out, rows, s);
    else return launch<T, VX, LV, false, false, false>(c, in, out, rows, s);
}

int compute_units()
{
    static const int n = [] {
        int dev = 0, ncu = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu <= 0)
            return 256;
        return ncu;
    }();
    return n;
}

// Windows of a row, or 0 where this width and level cannot march it.
template <int VX, int LV>
int windows(int nx, bool wall)
{
    using W = march::Windows<VX, LV>;
    return W::fits(nx, wall) ? W::count(nx, wall) : 0;
}
int windows_of(int vx, int lv, int nx, bool wall)
{
    switch (10 * vx + lv) {
        case 11: return windows<1, 1>(nx, wall);
        case 12: return windows<1, 2>(nx, wall);
        case 13: return windows<1, 3>(nx, wall);
        case 21: return windows<2, 1>(nx, wall);
        case 22: return windows<2, 2>(nx, wall);
        default: return 0;
    }
}

// Modelled time of one launch in us, fitted to 117 measured shapes (401 x 257
// to 4096 x 2048, 7 % rms).  rho', momentum: instructions of a row of drho' and
// of a row of new momenta per wave, from the compiled loops.  An instruction
// takes ns[w - 1] of a SIMD's time when w waves share it (four and more alike;
// with fewer, scalar work and waits are not hidden); more waves than a SIMD
// holds run one round after the other.  3.1 us is a launch inside a graph
// (1.7), the first loads and the last stores.  Memory: 8.1 TB/s while both
// state sets stay in the 256 MB cache, else 5.5.
double launch_us(int vx, int lv, int nw, int ny, int rows, bool f64, bool axi, bool wall, double bytes)
{
    static const double ns[4] = {3.04, 1.87, 1.70, 1.55};
    const double unit = (f64 ? 1.35 : 1.0) * (axi ? 1.31 : 1.0);
    const double rho = unit * (6 + 19 * vx) + (wall ? 5 : 0), mom = unit * (9 + 39 * vx) + (wall ? 12 : 0);
    double work = 11.0 * (rows + 4 * lv);
    for (int l = 1; l <= lv; ++l)
        work += (rows + 4 * (lv - l) + 2) * rho + (rows + 4 * (lv - l)) * mom;
    const int nb = (nw * ((ny + rows - 1) / rows) + 3) / 4, ncu = compute_units();
    const int whole = (nb + ncu - 1) / ncu;  // waves of the busiest SIMD
    // waves that a SIMD holds (registers of the compiled kernels)
    const int held1 = lv == 1 ? 7 : lv == 3 ? 3 : axi && wall ? 4 : 5, held2 = lv == 1 ? 4 : wall ? 2 : 3;
    const int held = f64 ? 4 - lv : vx == 1 ? held1 : held2;
    const int full = whole / held, rest = whole % held;
    double alu = full * held * ns[std::min(held, 4) - 1] + (rest ? rest * ns[std::min(rest, 4) - 1] : 0.0);
    if (whole > 2) alu *= (0.24 * nb / ncu + 0.76 * whole) / whole;  // the others take up some of its work
    alu *= work * 1e-3;
    const double traffic = bytes * (1.0 + 2.0 * lv / rows);  // halo rows are read twice
    const double mem = traffic / (bytes < 230e6 ? 8.1e6 : 5.5e6);
    return 3.07 + std::max(alu, mem) + 0.3 * std::min(alu, mem);
}

}  // namespace

// The launch shape of lv steps: window width and rows per chunk with the
// least modelled time.
template <typename T>
March2d march2d_plan(const Coef<T>& c, bool axi, int lv)
{
    March2d best{0, lv, 0, 0.0};
    const bool f64 = sizeof(T) == 8, wall = c.bc[0] != BC_PERIODIC;
    const double nodes = (double)c.nx * c.ny;
    if (c.rho0 != T(1) || nodes * sizeof(T) >= 2147483648.0) return best;
    // Tall grids of rows of up to half a window stay on the axisymmetric tiles:
    // us per step, tiles and march (two steps per launch), doubles 20 x 12320
    // 8.6 and 10.0, 13 x 7319 5.8 and 6.5, FP32 10 x 10316 5.8 and 6.3; 12 x 4217
    // doubles 5.7 and 5.8.  Planar ones march at 0.67 of the tiles' time.
    if (axi && c.nx <= 32 && c.ny >= (f64 ? 4000 : 8000)) return best;
    for (int vx = 1; vx <= (f64 ? 1 : 2); vx *= 2) {
        const int nw = windows_of(vx, lv, c.nx, wall);
        if (nw == 0 || (f64 && lv == 3)) continue;
        for (int r = 1; r <= 64; ++r) {
            const double t = launch_us(vx, lv, nw, c.ny, r, f64, axi, wall, 6.0 * nodes * sizeof(T)) / lv;
            if (best.vx == 0 || t < best.us) best = March2d{vx, lv, r, t};
            if (r >= c.ny) break;
        }
    }
    return best;
}

template <typename T>
March2d march2d_multi_plan(const Coef<T>& c, bool axi)
{
    March2d best = march2d_plan(c, axi, 1);
    for (int lv = 2; lv <= 3; ++lv) {
        const March2d p = march2d_plan(c, axi, lv);
        if (p.vx && p.us < best.us) best = p;
    }
    return best;
}

template <typename T>
hipError_t launch_march2d(const Coef<T>& c, const State<T>& in, const State<T>& out, bool axi, const March2d& p,
                          hipStream_t s)
{
    switch (10 * p.vx + p.lv) {
        case 11: return launch_faces<T, 1, 1>(c, in, out, axi, p.rows, s);
        case 12: return launch_faces<T, 1, 2>(c, in, out, axi, p.rows, s);
        default: break;
    }
    if constexpr (sizeof(T) == 4) {
        switch (10 * p.vx + p.lv) {
            case 13: return launch_faces<T, 1, 3>(c, in, out, axi, p.rows, s);
            case 21: return launch_faces<T, 2, 1>(c, in, out, axi, p.rows, s);
            case 22: return launch_faces<T, 2, 2>(c, in, out, axi, p.rows, s);
            default: break;
        }
    }
    return hipErrorInvalidValue;
}

#define MARCH2D(T)                                                                                           \
    template March2d march2d_plan<T>(const Coef<T>&, bool, int);                                             \
    template March2d march2d_multi_plan<T>(const Coef<T>&, bool);                                            \
    template hipError_t launch_march2d<T>(const Coef<T>&, const State<T>&, const State<T>&, bool, const March2d&, \
                                          hipStream_t);
MARCH2D(float)
MARCH2D(double)
#undef MARCH2D

}  // namespace acm
