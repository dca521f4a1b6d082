// ww_update.hip -- launchers of the flux-difference / CT / RK update kernels
// (device code in ww_update_dev.h).
#include "ww_index.h"
#include "ww_update_dev.h"

namespace ww {
namespace {

using up::UpdArgs;

// One thread per cell.
template <int ACT, typename T>
__global__ __launch_bounds__(256) void update_kernel(UpdArgs<T> a, FastDiv n0, FastDiv n1, uint32_t ncell)
{
    const uint32_t t = blockIdx.x * (uint32_t)blockDim.x + threadIdx.x;
    if (t >= ncell) return;
    const uint32_t r = n0.div(t), k = n1.div(r);
    const int pos[3] = { (int)(t - r * n0.d), (int)(r - k * n1.d), (int)k };
    up::update_cell<ACT>(a, pos);
}

template <int ACT, typename T>
hipError_t launch_cells(const UpdArgs<T> &a, hipStream_t st)
{
    const long ncell = (long)a.G.n[0] * a.G.n[1] * a.G.n[2];
    // fewer than 2^24 blocks of 256 threads per launch: cell numbers fit 32 bits
    if ((ncell + 255) / 256 >= (1L << 24)) return hipErrorInvalidConfiguration;
    // (blocks of one wave on small boxes: more CUs, each with its own L1)
    const int nt = ncell <= 64L * 1024 ? 64 : 256;
    hipLaunchKernelGGL((update_kernel<ACT, T>), dim3((unsigned)((ncell + nt - 1) / nt)), dim3(nt), 0, st, a,
                       FastDiv((uint32_t)a.G.n[0]), FastDiv((uint32_t)a.G.n[1]), (uint32_t)ncell);
    return hipGetLastError();
}

constexpr int MX_TX = 64, MX_TY = 4, MX_KZ = 16;   // march tile: x lanes, y rows, z cells
constexpr int NXCD = 8;                              // MI355X: 8 XCDs, blocks dealt round-robin
constexpr int MX_BLOCKS = 1024;                      // blocks that fill the chip (four per CU)

// Three active axes: one thread per (i, j) column segment of kz cells,
// marching in k (up::march_column).  Hardware block b runs on XCD b % 8;
// blocks are renumbered so that each XCD owns a contiguous range of tiles
// (neighbouring rows share its L2).
template <typename T, bool STAG>
__global__ __launch_bounds__(256) void update_march_kernel(UpdArgs<T> a, int ntx, int nty, int ntz, int kz,
                                                           int per_xcd)
{
    const Geom &G = a.G;
    const int hb = blockIdx.x;
    const int lb = (hb % NXCD) * per_xcd + hb / NXCD;
    if (lb >= ntx * nty * ntz) return;
    const int bx = lb % ntx, by = (lb / ntx) % nty, bz = lb / (ntx * nty);
    const int i = bx * MX_TX + threadIdx.x, j = by * MX_TY + threadIdx.y;
    if (i >= G.n[0] || j >= G.n[1]) return;
    const int k0 = bz * kz, k1 = min(k0 + kz, G.n[2]);
    up::march_column<T, STAG>(a, i, j, k0, k1);
}

}  // namespace

template <typename T>
hipError_t launch_update(const T *u0, const T *acc_in, T *acc_out, T *out, const T *fx,
                         const T *fy, const T *fz, const FaceBox *F, const Geom &G,
                         const StageCoef &c, hipStream_t st, long odelta, long osv)
{
    UpdArgs<T> a;
    a.odelta = odelta;
    a.osv = osv > 0 ? osv : G.sv;
    a.u0 = u0; a.acc_in = acc_in; a.acc_out = acc_out; a.out = out;
    a.ff[0] = fx; a.ff[1] = fy; a.ff[2] = fz;
    for (int d = 0; d < 3; ++d) a.fb[d] = F[d];
    a.G = G;
    a.c = c;
    // B only: by columns (by cells 2-3 % slower in whole steps of 128^3 to 256^3,
    // no faster at 96^3)
    if (c.bonly) {
        if (!(G.act[0] && G.act[1] && G.act[2])) return hipErrorInvalidValue;
        const int ntx = (G.n[0] + MX_TX - 1) / MX_TX, nty = (G.n[1] + MX_TY - 1) / MX_TY;
        // A march is a serial chain of one memory latency (about 6 us with
        // the arithmetic) per cell.  Segments of MX_KZ cells reuse the carried
        // fluxes best and serve boxes that fill the chip with them; smaller
        // boxes are cut into shorter segments, down to one cell, until they
        // do: at 32^3 (16 blocks of 16 cells) the FP64 update took 112 us.
        int kz = MX_KZ;
        while (kz > 1 && (long)ntx * nty * ((G.n[2] + kz - 1) / kz) < MX_BLOCKS) kz /= 2;
        const int ntz = (G.n[2] + kz - 1) / kz;
        int nb = ntx * nty * ntz, per = (nb + NXCD - 1) / NXCD;
        const dim3 grd(per * NXCD), blk(MX_TX, MX_TY);
        if (c.stag)
            hipLaunchKernelGGL((update_march_kernel<T, true>), grd, blk, 0, st, a, ntx, nty, ntz, kz, per);
        else
            hipLaunchKernelGGL((update_march_kernel<T, false>), grd, blk, 0, st, a, ntx, nty, ntz, kz, per);
        return hipGetLastError();
    }
    switch (G.act[0] + 2 * G.act[1] + 4 * G.act[2]) {
    case 1: return launch_cells<1, T>(a, st);
    case 2: return launch_cells<2, T>(a, st);
    case 3: return launch_cells<3, T>(a, st);
    case 4: return launch_cells<4, T>(a, st);
    case 5: return launch_cells<5, T>(a, st);
    case 6: return launch_cells<6, T>(a, st);
    case 7: return launch_cells<7, T>(a, st);
    default: return hipErrorInvalidValue;
    }
}

template hipError_t launch_update<double>(const double *, const double *, double *, double *,
                                          const double *, const double *, const double *,
                                          const FaceBox *, const Geom &, const StageCoef &,
                                          hipStream_t, long, long);
template hipError_t launch_update<float>(const float *, const float *, float *, float *,
                                         const float *, const float *, const float *,
                                         const FaceBox *, const Geom &, const StageCoef &,
                                         hipStream_t, long, long);

}  // namespace ww
