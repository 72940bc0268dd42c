// 3D single-phase launches of the register march (march3d.h).
#include <algorithm>

#include "acm_internal.h"
#include "march3d.h"

namespace acm {

namespace {

template <typename T, int VX, int RY, bool WX, bool WYZ>
__global__ __launch_bounds__(256) void march3d_kernel(Coef<T> c, State<T> in, State<T> out, int nw, int nby, int zc)
{
    using W = march::Windows<VX, 1>;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int item = 4 * xcd_remap(blockIdx.x, gridDim.x) + wave;
    const int t = item / nby, by = item - t * nby;
    const int chunk = t / nw, w = t - chunk * nw;
    const int z0 = chunk * zc, z1 = min(z0 + zc, c.nz);
    if (z0 >= c.nz) return;
    int xs, l0, l1;
    W::window(c.nx, WX && c.bc[0] != BC_PERIODIC, w, nw, xs, l0, l1);
    march::run3<T, VX, RY, WX, WYZ, false>(c, in, out, xs, l0, l1, by * RY, z0, z1);
}

template <typename T, int VX, int RY, bool WX, bool WYZ>
hipError_t launch(const Coef<T>& c, const State<T>& in, const State<T>& out, int zc, hipStream_t s)
{
    const int nw = march::Windows<VX, 1>::count(c.nx, c.bc[0] != BC_PERIODIC);
    const int nby = (c.ny + RY - 1) / RY;
    const int nb = (nw * nby * ((c.nz + zc - 1) / zc) + 3) / 4;
    hipLaunchKernelGGL((march3d_kernel<T, VX, RY, WX, WYZ>), dim3(nb), dim3(256), 0, s, c, in, out, nw, nby, zc);
    return hipGetLastError();
}

template <typename T, int VX, int RY>
hipError_t launch_faces(const Coef<T>& c, const State<T>& in, const State<T>& out, int zc, hipStream_t s)
{
    const bool wx = c.bc[0] != BC_PERIODIC;
    if (wx) return launch<T, VX, RY, true, true>(c, in, out, zc, s);
    if (c.nonperiodic) return launch<T, VX, RY, false, true>(c, in, out, zc, s);
    return launch<T, VX, RY, false, false>(c, in, out, zc, s);
}

}  // namespace

static int compute_units()
{
    static const int cus = [] {
        int dev = 0, ncu = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu <= 0)
            return 256;
        return ncu;
    }();
    return cus;
}
static int workgroups(int nw, int ny, int nz, int ry, int zc)
{
    return (nw * ((ny + ry - 1) / ry) * ((nz + zc - 1) / zc) + 3) / 4;
}

// Modelled time of one launch in us, fitted to 78 measured shapes (40^3 to
// 200 x 200 x 160, 7 % rms); the form is that of the 2D march's model.
constexpr double LAUNCH3_US = 4.96;
static double launch3_us(int nw, int ny, int nz, int ry, int zc, bool wall, double bytes)
{
    static const double ns[3] = {2.56, 2.03, 1.70};
    const double rho = (ry + 2) * (63.6 + (wall ? 8.7 : 0)), mom = ry * (18.7 + (wall ? 37 : 0));
    const double work = (zc + 4) * 12.5 * (ry + 4) + (zc + 2) * rho + zc * mom;
    const int nb = workgroups(nw, ny, nz, ry, zc), cus = compute_units();
    const int whole = (nb + cus - 1) / cus, held = ry == 2 ? 3 : 2;
    const int full = whole / held, rest = whole % held;
    double alu = full * held * ns[held - 1] + (rest ? rest * ns[rest - 1] : 0.0);
    if (whole > 2) alu *= (0.23 * nb / cus + 0.77 * whole) / whole;
    alu *= work * 1e-3;
    const double mem = bytes * (1.0 + 2.0 / zc) / (bytes < 230e6 ? 8.1e6 : 5.5e6);
    return LAUNCH3_US + std::max(alu, mem) + 0.3 * std::min(alu, mem);
}

// The march applies: rho0 = 1, no per-node force, and both state sets (32
// bytes per node) within the 256 MB cache: the rows that a wave loads beside
// its own come from there.  200 x 200 x 160 (205 MB): 54 us against 75 for the
// columns; 256^3 with walls (537 MB): 206 against 152.
bool march3d_ok(const Coef<float>& c)
{
    return c.rho0 == 1.f && !c.fst[0] && c.nz >= 2 && 32.0 * c.nx * c.ny * c.nz <= 256e6;
}

// Rows per wave (two, or four where that leaves enough waves) and planes per
// chunk with the least modelled time.  The time given back corrects the model
// by the faces, for chunks of few planes and for a chip that is partly used,
// fitted to 640 random grids (8 to 320 nodes a side, 6 % rms).
March3d march3d_plan(const Coef<float>& c)
{
    const bool wall = c.bc[0] != BC_PERIODIC;
    const int nw = march::Windows<1, 1>::count(c.nx, wall);
    const double bytes = 32.0 * c.nx * c.ny * c.nz;
    March3d best{2, 4, -1.0};
    for (int r = 2; r <= 4; r += 2)
        for (int z = 2; z <= 64; z += z < 16 ? 1 : 8) {
            const double t = launch3_us(nw, c.ny, c.nz, r, z, wall, bytes);
            if (best.us < 0.0 || t < best.us) best = March3d{r, z, t};
            if (z >= c.nz) break;
        }
    const double used = std::min(1.0, (double)workgroups(nw, c.ny, c.nz, best.ry, best.zc) / compute_units());
    const double start = wall ? 3.0 : c.nonperiodic ? 2.9 : 1.8, rate = wall ? 0.945 : c.nonperiodic ? 1.03 : 1.01;
    best.us = start + 1.25 * used + (best.us - LAUNCH3_US) * (rate + 1.8 / std::max(c.nz, 8));
    return best;
}

hipError_t launch_march3d(const Coef<float>& c, const State<float>& in, const State<float>& out, const March3d& p,
                          hipStream_t s)
{
    if (p.ry == 4) return launch_faces<float, 1, 4>(c, in, out, p.zc, s);
    return launch_faces<float, 1, 2>(c, in, out, p.zc, s);
}

}  // namespace acm
