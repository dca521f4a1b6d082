// ww_sweep.hip -- launchers of the characteristic WENO5 sweep kernels (one
// tile per block; the device code is in ww_sweep_dev.h).
#include "ww_sweep_dev.h"

namespace ww {
namespace {

// At least two waves per SIMD.  The FP64 kernels sit at 248-253 VGPRs; without
// this the WENO-Z instantiations took a few AGPRs more and dropped to one
// wave per SIMD (the x sweep ran 40 % slower).  With it every sweep kernel
// fits in 256 VGPRs without spilling.  The WENO-JS and FP32 code is unchanged
// by it.
#define WW_TWO_WAVES __attribute__((amdgpu_waves_per_eu(2)))

// 256-thread blocks of a launch: HIP takes fewer than 2^32 threads per axis.
// Tile and face numbers therefore fit 32 bits.
constexpr long MAX_BLOCKS = 1L << 24;

// x sweeps stage the cells' fluxes with the cells (sw::NQ_PRE) in FP32 only:
// the FP32 fused x sweep ran 1.8 % faster at 512^3.  The FP64 sweeps ran 2 %
// slower with them (the larger live set spilled at 256 VGPRs), and the FP32
// y/z tiles lost a block per CU to the larger LDS footprint and ran 5 % slower.
template <typename T> constexpr bool pre_x() { return sizeof(T) == 4; }

// x sweep of short rows: 2-D grid (ta, tb) of 4 rows x 64 faces.
template <typename T, bool WZ, bool GLF>
__global__ __launch_bounds__(256) WW_TWO_WAVES void sweep_xrows_kernel(const T *__restrict__ u,
                                                           T *__restrict__ flux, Geom G, FaceBox F, Phys P)
{
    __shared__ T sq[sw::NQ * sw::XROWS_CELLS];
    sw::sweep_tile_xrows<T, WZ, GLF>(u, flux, G, F, P, blockIdx.x, blockIdx.y, sq);
}

template <typename T, bool WZ, bool GLF>
__global__ __launch_bounds__(256) WW_TWO_WAVES void sweep_xseg_kernel(const T *__restrict__ u, T *__restrict__ flux,
                                                         Geom G, FaceBox F, Phys P, sw::XSegArgs A)
{
    __shared__ T sq[sw::nq<pre_x<T>()>() * sw::XSEG_CELLS];
    sw::sweep_tile_xseg<T, WZ, GLF, pre_x<T>()>(u, flux, G, F, P, A, blockIdx.x, sq);
}

// The fused x sweep renumbers blocks so that each XCD walks a contiguous
// range of tiles: neighbouring rows, whose cells read the same y faces, then
// meet in one L2.

template <typename T, bool WZ, bool GLF>
__global__ __launch_bounds__(256) WW_TWO_WAVES void sweep_xfused_kernel(const T *__restrict__ u,
                                                           T *__restrict__ flux, Geom G, FaceBox F, Phys P,
                                                           XFuse<T> xf, sw::XSegArgs A, uint32_t ntile,
                                                           uint32_t per_xcd)
{
    __shared__ T sq[sw::nq<pre_x<T>()>() * sw::XSEG_CELLS];
    __shared__ T hx[5 * sw::TILE * sw::ROWS];
    const uint32_t tile = (blockIdx.x % sw::NXCD) * per_xcd + blockIdx.x / sw::NXCD;
    if (tile >= ntile) return;
    sw::sweep_tile_xseg_fused<T, WZ, GLF, pre_x<T>()>(u, flux, G, F, P, A, tile, sq, hx, xf);
}

template <typename T, bool WZ, bool GLF>
hipError_t launch_xfused(const T *u, T *flux, const Geom &G, const FaceBox &F, const Phys &P, const XFuse<T> &xf,
                         hipStream_t st)
{
    const long total = (long)F.cnt[0] * F.cnt[1] * F.cnt[2];
    const long nt = (total - 1 + sw::XFUSE_STRIDE - 1) / sw::XFUSE_STRIDE;
    const long per = (nt + sw::NXCD - 1) / sw::NXCD;
    if (per * sw::NXCD >= MAX_BLOCKS) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((sweep_xfused_kernel<T, WZ, GLF>), dim3((unsigned)(per * sw::NXCD)), dim3(sw::TILE, sw::ROWS), 0,
                       st, u, flux, G, F, P, xf, sw::xseg_args(F), (uint32_t)nt, (uint32_t)per);
    return hipGetLastError();
}

// y/z tiles.  FP64: 32 positions x 8 faces (1.6 staged cells per face instead
// of 2.25 with 64 x 4, in 43 KB of LDS), measured 3 % faster at 512^3.  FP32:
// 64 positions x 8 faces, two faces per thread; the FP64 shape is 12 % slower
// there.
template <typename T> constexpr int yz_pw() { return sizeof(T) == 8 ? 32 : 64; }
constexpr int YZ_FT = 8;

template <int DIR, typename T, bool WZ, bool GLF>
__global__ __launch_bounds__(256) WW_TWO_WAVES void sweep_yz_kernel(const T *__restrict__ u, T *__restrict__ flux,
                                                       Geom G, FaceBox F, Phys P, sw::YZArgs Y)
{
    constexpr int PW = yz_pw<T>();
    __shared__ T sq[sw::NQ * sw::yz_cells<PW, YZ_FT>()];
    uint32_t ta, tb;
    uint32_t lb;
    if (!sw::column_tile(Y, ta, tb, lb)) return;
    sw::sweep_tile_yz<DIR, PW, YZ_FT, T, WZ, GLF>(u, flux, G, F, P, Y, ta, tb, sq);
}

template <int DIR, typename T, bool WZ, bool GLF>
hipError_t launch_yz(const T *u, T *flux, const Geom &G, const FaceBox &F, const Phys &P, hipStream_t st)
{
    constexpr int PW = yz_pw<T>(), B = DIR == 1 ? 2 : 1;
    const long nt = ((long)F.cnt[0] * F.cnt[B] + PW - 1) / PW * ((F.cnt[DIR] + YZ_FT - 1) / YZ_FT);
    if (nt + sw::NXCD >= MAX_BLOCKS) return hipErrorInvalidConfiguration;
    const sw::YZArgs Y = sw::yz_args<DIR, PW, YZ_FT>(F, sw::NXCD);
    hipLaunchKernelGGL((sweep_yz_kernel<DIR, T, WZ, GLF>), dim3(Y.per_xcd * sw::NXCD), dim3(sw::TILE, sw::ROWS), 0, st,
                       u, flux, G, F, P, Y);
    return hipGetLastError();
}

template <typename T, bool WZ, bool GLF>
hipError_t launch_x(const T *u, T *flux, const Geom &G, const FaceBox &F, const Phys &P, hipStream_t st)
{
    if (F.cnt[0] >= sw::XSEG_MIN) {
        // long rows: flattened face segments, no ragged tile per row
        const long total = (long)F.cnt[0] * F.cnt[1] * F.cnt[2];
        const long nt = (total + sw::TILE * sw::ROWS - 1) / (sw::TILE * sw::ROWS);
        if (nt >= MAX_BLOCKS) return hipErrorInvalidConfiguration;
        hipLaunchKernelGGL((sweep_xseg_kernel<T, WZ, GLF>), dim3((unsigned)nt), dim3(sw::TILE, sw::ROWS), 0, st,
                           u, flux, G, F, P, sw::xseg_args(F));
        return hipGetLastError();
    }
    long na, nb;
    sw::xrows_tiles(F, na, nb);
    hipLaunchKernelGGL((sweep_xrows_kernel<T, WZ, GLF>), dim3((unsigned)na, (unsigned)nb),
                       dim3(sw::TILE, sw::ROWS), 0, st, u, flux, G, F, P);
    return hipGetLastError();
}

template <typename T, bool WZ, bool GLF>
hipError_t launch_dirs(int dir, const T *u, T *flux, const Geom &G, const FaceBox &F, const Phys &P,
                       hipStream_t st)
{
    switch (dir) {
    case 0: return launch_x<T, WZ, GLF>(u, flux, G, F, P, st);
    case 1: return launch_yz<1, T, WZ, GLF>(u, flux, G, F, P, st);
    default: return launch_yz<2, T, WZ, GLF>(u, flux, G, F, P, st);
    }
}

}  // namespace

template <typename T>
hipError_t launch_sweep(int dir, const T *u, T *flux, const Geom &G, const FaceBox &F,
                        const Phys &P, int weights, hipStream_t st)
{
    const bool z = weights == WEIGHTS_Z, glf = P.ag != nullptr;
    if (z && glf) return launch_dirs<T, true, true>(dir, u, flux, G, F, P, st);
    if (z) return launch_dirs<T, true, false>(dir, u, flux, G, F, P, st);
    if (glf) return launch_dirs<T, false, true>(dir, u, flux, G, F, P, st);
    return launch_dirs<T, false, false>(dir, u, flux, G, F, P, st);
}

int sweep_x_fused_min_faces() { return sw::XSEG_MIN; }

template <typename T>
hipError_t launch_sweep_x_fused(const T *u, T *flux, const Geom &G, const FaceBox &F, const Phys &P,
                                int weights, const XFuse<T> &xf, hipStream_t st)
{
    if (F.cnt[0] < sw::XSEG_MIN || !(G.act[0] && G.act[1] && G.act[2])) return hipErrorInvalidValue;
    const bool z = weights == WEIGHTS_Z, glf = P.ag != nullptr;
    if (z && glf) return launch_xfused<T, true, true>(u, flux, G, F, P, xf, st);
    if (z) return launch_xfused<T, true, false>(u, flux, G, F, P, xf, st);
    if (glf) return launch_xfused<T, false, true>(u, flux, G, F, P, xf, st);
    return launch_xfused<T, false, false>(u, flux, G, F, P, xf, st);
}

template hipError_t launch_sweep_x_fused<double>(const double *, double *, const Geom &, const FaceBox &,
                                                 const Phys &, int, const XFuse<double> &, hipStream_t);
template hipError_t launch_sweep_x_fused<float>(const float *, float *, const Geom &, const FaceBox &,
                                                const Phys &, int, const XFuse<float> &, hipStream_t);

template hipError_t launch_sweep<double>(int, const double *, double *, const Geom &,
                                         const FaceBox &, const Phys &, int, hipStream_t);
template hipError_t launch_sweep<float>(int, const float *, float *, const Geom &,
                                        const FaceBox &, const Phys &, int, hipStream_t);

}  // namespace ww
