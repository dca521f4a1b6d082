// ww_batch.hip -- many independent periodic patches advanced by one
// persistent launch per RK stage.
//
// The patches (arXiv:1808.10633, Sec. 2.2: the domain is cut into patches of
// 18^3-32^3 zones with ghost zones, each computed independently once its
// boundary zones are present) live in one arena.  Resident blocks take work
// items from a shared counter (one atomic per item), so a block that finishes
// early takes the next one and the stage ends when the work runs out, not when
// the unluckiest block does.  An item is a whole patch, or a share of a patch
// that would keep one block busy beyond the others' end (ww_batch_plan.h; 1024
// FP32 patches of 16-64 cells per axis were bound by one block's 64^3 patch:
// 71.5 ms a step as whole patches, 45.2 ms split).  A patch is taken through
// the full stage: (stage 0 only) the patch's CFL
// time step (0, and the patch left unadvanced, if any cell is non-physical),
// x/y/z characteristic WENO sweeps into the patch's face-flux scratch
// (y and z first; the flattened x tiles also apply the rho, m, E update),
// then CT and the B part of the RK update -- the same device functions as
// the single-box kernels.  The patches are periodic, and the sweep tiles
// stage each ghost cell from its periodic image: the ghost zones of the
// arena are neither filled nor read.
#include "ww_batch.h"
#include "ww_sweep_dev.h"
#include "ww_update_dev.h"

namespace ww {
namespace {

constexpr int RB = BATCH_THREADS;

// The patch number comes from a shared counter through LDS, so the compiler
// takes everything read by it for per-lane data: geometry, strides and loop
// bounds then sit in vector registers and every address is vector 64-bit
// arithmetic.  The descriptor is read through the constant address space at a
// scalar index instead (it never changes during the kernel).
__device__ __forceinline__ PatchDesc load_desc(const PatchDesc *pd, int p)
{
    typedef const unsigned long long __attribute__((address_space(4))) *cptr;
    constexpr int NW = sizeof(PatchDesc) / 8;
    unsigned long long w[NW];
    cptr q = (cptr)(pd + p);
#pragma unroll
    for (int i = 0; i < NW; ++i) w[i] = q[i];
    PatchDesc D;
    __builtin_memcpy(&D, w, sizeof D);
    return D;
}
// One 32-bit word of a table that does not change during the kernel.
__device__ __forceinline__ int load_word(const int *p)
{
    return *(const int __attribute__((address_space(4))) *)p;
}
__device__ __forceinline__ BatchItem load_item(const BatchItem *items, int i)
{
    const int *q = (const int *)(items + i);
    return BatchItem{ load_word(q), load_word(q + 1), load_word(q + 2), load_word(q + 3),
                      load_word(q + 4), load_word(q + 5), load_word(q + 6), load_word(q + 7) };
}
__device__ __forceinline__ SplitDesc load_split(const SplitDesc *split, int i)
{
    const int *q = (const int *)(split + i);
    return SplitDesc{ { load_word(q), load_word(q + 1), load_word(q + 2) }, 0 };
}

// Largest signal speed sum and count of non-physical cells of cells c_lo ..
// c_hi - 1 of a patch, in FP64 (valid in thread 0; neither depends on the
// order).
template <typename T>
__device__ __forceinline__ void patch_speed(const T *__restrict__ u, const PatchDesc &D, const Geom &G, double gamma,
                                            int c_lo, int c_hi, double &mx_out, int &bad_out)
{
    __shared__ double smx[sw::ROWS];
    __shared__ int sfl[sw::ROWS];
    const int tid = threadIdx.x + sw::TILE * threadIdx.y;
    const int ncell = c_hi;     // < 2^31 for edges of at most 1024
    const T *const ub = u + G.base;
    double mx = 0.0;
    int bad = 0;
    // DT_IT cells per thread and pass: all their loads first, then the
    // arithmetic (at two waves per SIMD one cell at a time waits a full
    // memory latency per cell); the maximum and the count do not depend on
    // the order
    constexpr int DT_IT = 4;
    for (int c0 = c_lo + tid; c0 < ncell; c0 += DT_IT * RB) {
        T w[DT_IT][8];
#pragma unroll
        for (int it = 0; it < DT_IT; ++it) {
            const int c = c0 + it * RB;
            if (c < ncell) {
                const uint32_t jk = D.nx.div(c), k = D.ny.div(jk);
                const uint32_t e = (c - jk * D.nx.d) + (jk - k * D.ny.d) * (uint32_t)G.s[1] + k * (uint32_t)G.s[2];
#pragma unroll
                for (int v = 0; v < 8; ++v) w[it][v] = sw::uniform(ub + v * G.sv)[e];
            }
        }
#pragma unroll
        for (int it = 0; it < DT_IT; ++it) {
            if (c0 + it * RB >= ncell) continue;
            double q[8];
            bool fin = true;
            for (int v = 0; v < 8; ++v) { q[v] = (double)w[it][v]; fin = fin && isfinite(q[v]); }
            double r = q[0], ir = 1.0 / r;
            double vx = q[1] * ir, vy = q[2] * ir, vz = q[3] * ir;
            double b2 = q[4] * q[4] + q[5] * q[5] + q[6] * q[6];
            double pr = (gamma - 1.0) * (q[7] - 0.5 * (q[1] * vx + q[2] * vy + q[3] * vz) - 0.5 * b2);
            if (!fin || !(r > 0.0) || !(pr > 0.0)) { ++bad; continue; }
            double a2 = gamma * pr * ir;
            double v[3] = { vx, vy, vz };
            double s = 0.0;
            for (int d = 0; d < 3; ++d) {
                double bn2 = q[4 + d] * q[4 + d] * ir;
                double bt2 = b2 * ir - bn2;
                bt2 = bt2 < 0.0 ? 0.0 : bt2;
                double dd = a2 - bn2;
                double cf2 = 0.5 * (a2 + bn2 + bt2 + sqrt(dd * dd + bt2 * (2.0 * a2 + 2.0 * bn2 + bt2)));
                s += (fabs(v[d]) + sqrt(cf2)) * G.idl[d];
            }
            mx = fmax(mx, s);
        }
    }
    // butterfly over the wave's 64 lanes, then the four waves in order
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) {
        mx = fmax(mx, __shfl_xor(mx, m));
        bad += __shfl_xor(bad, m);
    }
    if (threadIdx.x == 0) { smx[threadIdx.y] = mx; sfl[threadIdx.y] = bad; }
    __syncthreads();
    if (tid == 0)
        for (int w = 1; w < sw::ROWS; ++w) { mx = fmax(mx, smx[w]); bad += sfl[w]; }
    mx_out = mx;
    bad_out = bad;
    __syncthreads();
}
__device__ __forceinline__ void store_dt(double mx, int bad, double cfl, double *dt_out, int32_t *flag_out)
{
    const bool ok = mx > 0.0 && bad == 0;
    *dt_out = ok ? cfl / mx : 0.0;
    *flag_out = bad > 0 ? bad : (ok ? 0 : 1);
}

// Waits and counts between the blocks of a split patch.  Every wave of the
// counting block waits until its stores are in the L2, then one wave writes
// the L2 back and counts; in the waiting block one wave drops the CU's and the
// L2's stale lines before the others go on (a fence per wave costs four of
// each).  The waits are written out: with none of a wave's own stores
// outstanding the compiler leaves out the one between a release fence's
// write-back and the atomic that it guards.
__device__ __forceinline__ void wait_memory() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void release_all()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    wait_memory();
}
__device__ __forceinline__ void acquire_all()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    wait_memory();
}
__device__ __forceinline__ void wait_count(const int32_t *count, int target)
{
    if (threadIdx.x == 0 && threadIdx.y == 0) {
        while (__hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target)
            __builtin_amdgcn_s_sleep(16);
        acquire_all();
    }
    __syncthreads();
}
// Returns the count after this item (in thread 0).
__device__ __forceinline__ int count_done(int32_t *count)
{
    wait_memory();
    __syncthreads();
    int n = 0;
    if (threadIdx.x == 0 && threadIdx.y == 0) {
        release_all();
        n = __hip_atomic_fetch_add(count, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
    }
    return n;
}

// y or z sweep of a patch: tiles of 64 positions of the transverse plane (x
// fastest) x FT faces, wave w taking rows and faces w, w + 4, ..: row and face
// numbers are uniform, positions per lane.  Ghost cells are staged from their
// periodic images.  Each 64-position column is walked along the sweep axis,
// so that a tile's five halo rows are still in the L2.
template <int DIR, int FT, typename T>
__device__ __forceinline__ void sweep_yz_patch(const T *__restrict__ u, T *__restrict__ flux, const PatchDesc &D,
                                               const Geom &G, const FaceBox &F, const Phys &P, int t_lo, int t_hi,
                                               T *sq)
{
    constexpr int N = DIR, T1 = (DIR + 1) % 3, T2 = (DIR + 2) % 3, B = DIR == 1 ? 2 : 1;
    constexpr int NC = sw::TILE * (FT + 5), IT = (FT + 5 + sw::ROWS - 1) / sw::ROWS;
    const int cm[8] = { 0, 1 + N, 1 + T1, 1 + T2, 4 + N, 4 + T1, 4 + T2, 7 };
    const int gc[7] = { 0, 1 + N, 1 + T1, 1 + T2, 4, 5, 6 };
    const int lane = threadIdx.x, w = __builtin_amdgcn_readfirstlane(threadIdx.y);
    const int npos = F.cnt[0] * F.cnt[B];
    for (int t = t_lo; t < t_hi; ++t) {
        const int p0 = t * sw::TILE;
        const bool ok = p0 + lane < npos;
        // position - 1; lanes and rows beyond the end repeat the last one, so
        // that the loads need no branches (values loaded under one were kept,
        // and spilled, through the whole tile loop)
        const uint32_t pp = ok ? p0 + lane : npos - 1, b = D.na.div(pp), a = pp - b * D.na.d;
        const uint32_t es = sw::pwrap((int)a - 1, G.n[0]) + sw::pwrap((int)b - 1, G.n[B]) * (uint32_t)G.s[B];
        const uint32_t ef = a + b * (uint32_t)F.s[B];
        for (int f0 = 0; f0 < F.cnt[N]; f0 += FT) {
            sw::stage_begin();
            const int rows = min(FT + 5, G.n[N] + 6 - f0);       // cells f0 - 3 .. n + 2
            T q[IT][8];
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                const int r = min(w + it * sw::ROWS, rows - 1);
                const T *const ub = u + G.base + sw::pwrap(f0 - 3 + r, G.n[N]) * G.s[N];
#pragma unroll
                for (int v = 0; v < 8; ++v) q[it][v] = sw::uniform(ub + cm[v] * G.sv)[es];
            }
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                const int r = w + it * sw::ROWS;
                if (r < rows) sw::stage_values<T>(q[it], P.gamma, sq + r * sw::TILE + lane, NC);
            }
            __syncthreads();
            sw::stage_end();
            if (ok) {
                for (int r = w; r < FT && f0 + r < F.cnt[N]; r += sw::ROWS) {
                    T out[7];
                    sw::face_flux<T>(sq, NC, r * sw::TILE + lane, sw::TILE, P.gamma, P.igm1, (T)P.eps, out);
                    T *const fb = flux + (f0 + r) * F.s[N];
#pragma unroll
                    for (int c = 0; c < 7; ++c) sw::uniform(fb + gc[c] * F.sc)[ef] = out[c];
                }
            }
            __syncthreads();
        }
    }
}

// The x sweep for short rows with the rho, m, E part of the update fused in
// (the batched counterpart of sweep_tile_xseg_fused): tiles of XF_FACES faces
// of the flattened (row, face) space overlapping by one (tile t starts at face
// (XF_FACES - 1) t), one per thread (two faces per thread spill registers, and
// the batched FP32 step measured 4% slower).  A tile stages every cell of the
// rows it touches, at most xflat_cells(n, rows), ghost cells from their
// periodic images; the fluxes' rho, m, E go to LDS (hx, 5 x XF_FACES) and
// thread tid takes the cell right of its face when the next face is in the
// same row and the row is interior.  Only the transverse-B fluxes of the x
// faces are stored.  sq: NQ * XF_MAXC elements.  A flattened row holds at most
// 266 cells and a patch edge 1024, so a variable is under 2^32 bytes and
// every offset fits 32 bits.  Tiles t_lo .. t_hi - 1.
constexpr int XF_FACES = sw::TILE * sw::ROWS;
constexpr int XF_MAXC = 544;     // 4-cell rows: at most 53 rows of 10 cells
inline int xflat_cells(int nx, long nrows)
{
    long span = (XF_FACES + nx) / (nx + 1) + 1;
    if (span > nrows) span = nrows;
    return (int)(span * (nx + 6));
}

template <typename T>
__device__ __forceinline__ void sweep_xflat_patch(const T *__restrict__ u, T *__restrict__ flux, const PatchDesc &D,
                                                  const Geom &G, const FaceBox &F, const Phys &P, int t_lo, int t_hi,
                                                  T *sq, T *hx, const XFuse<T> &xf)
{
    constexpr int STRIDE = XF_FACES - 1, IT = (XF_MAXC + RB - 1) / RB;
    const int tid = threadIdx.x + sw::TILE * threadIdx.y;
    const int total = (int)F.sc, nrows = F.cnt[1] * F.cnt[2];
    // the patch's faces and RK arrays from its cell (0, 0, 0) on
    sw::FusedTile<T> B;
    B.nx2 = G.n[0] + 2;
    B.fy = xf.fy + 1 + xf.by.s[2];
    B.fz = xf.fz + 1 + B.nx2;
    B.u0 = xf.u0 + G.base;
    B.acc_in = xf.acc_in + G.base;
    B.acc_out = xf.acc_out + G.base;
    B.out = xf.out + G.base;
    for (int t = t_lo; t < t_hi; ++t) {
        const int g0 = t * STRIDE;
        sw::stage_begin();
        const int r_lo = (int)D.nf.div(g0);
        int r_hi = (int)D.nf.div(g0 + XF_FACES - 1);
        if (r_hi > nrows - 1) r_hi = nrows - 1;
        const int ncell = (r_hi - r_lo + 1) * (int)D.nxp.d;
        T q[IT][8];
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int c = min(tid + it * RB, ncell - 1);
            const uint32_t rr = D.nxp.div(c), row = r_lo + rr, kk = D.n1f.div(row);
            const int x = sw::pwrap((int)(c - rr * D.nxp.d) - 3, G.n[0]);
            const int j = sw::pwrap((int)(row - kk * D.n1f.d) - 1, G.n[1]), k = sw::pwrap((int)kk - 1, G.n[2]);
            const uint32_t e = x + j * (uint32_t)G.s[1] + k * (uint32_t)G.s[2];
#pragma unroll
            for (int v = 0; v < 8; ++v) q[it][v] = sw::ld32(u + G.base + v * G.sv, e);
        }
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int c = tid + it * RB;
            if (c < ncell) sw::stage_values<T>(q[it], P.gamma, sq + c, XF_MAXC);
        }
        __syncthreads();
        sw::stage_end();
        const int g = g0 + tid;
        const bool valid = g < total;
        const uint32_t row = D.nf.div(g), kk = D.n1f.div(row);
        const int i = (int)(g - row * D.nf.d), j = (int)(row - kk * D.n1f.d) - 1, k = (int)kk - 1;
        if (valid) {
            T out[7];
            sw::face_flux<T>(sq, XF_MAXC, (int)((row - r_lo) * D.nxp.d) + i, 1, P.gamma, P.igm1, (T)P.eps, out);
            hx[0 * XF_FACES + tid] = out[0];
            hx[1 * XF_FACES + tid] = out[1];
            hx[2 * XF_FACES + tid] = out[2];
            hx[3 * XF_FACES + tid] = out[3];
            hx[4 * XF_FACES + tid] = out[6];
            if (tid < STRIDE || g == total - 1) {
                sw::st32<T>(flux + 4 * F.sc + g0, tid, out[4]);
                sw::st32<T>(flux + 5 * F.sc + g0, tid, out[5]);
            }
        }
        // the cell's global loads in flight before the barrier
        const bool cell = valid && tid < STRIDE && g + 1 < total && i < G.n[0] && j >= 0 && j < G.n[1] && k >= 0 &&
                          k < G.n[2];
        // (lanes without a cell load cell (0, 0, 0)'s values: no branch)
        const uint32_t ci = cell ? i : 0, cj = cell ? j : 0, ck = cell ? k : 0;
        const uint32_t rel = ci + cj * (uint32_t)G.s[1] + ck * (uint32_t)G.s[2], rj = ci + cj * (uint32_t)B.nx2;
        sw::FusedCell<T> fc;
        sw::fused_tile_load(xf, B, G.sv, rj + ck * (uint32_t)xf.by.s[2], rj + ck * (uint32_t)xf.bz.s[2], rel, fc);
        __syncthreads();
        if (cell) sw::fused_tile_store(xf, B, G, hx, XF_FACES, tid, rel, fc);
        __syncthreads();
    }
}

// Constrained transport and the B part of the RK stage of a patch whose x
// sweep did the rho, m, E part: one thread per (i, j) column segment of up to
// KSEG cells marching in k, the z-level EMFs carried (every EMF formed once
// per column instead of once per adjacent cell, as in update_cell), the loads
// of level k+1 issued before the arithmetic of level k (two waves per SIMD
// hide little latency).  Operands, expressions and order of march_column.
// Shares t_lo .. t_hi - 1 of RB segments.
template <typename T>
struct BLevel {
    T x5h0, x5h1, y4h0, y4h1;          // FX5(i|i+1, j, k+1), FY4(i, j|j+1, k+1)
    T z4m, z4c, z4p;                   // FZ4(i-1|i|i+1, j, k+1)
    T z5m, z5c, z5p;                   // FZ5(i, j-1|j|j+1, k+1)
    T x4[6];                           // FX4 at (i, j-1), (i, j), (i+1, j-1), (i+1, j), (i, j+1), (i+1, j+1), level k
    T y5[6];                           // FY5 at (i-1, j), (i, j), (i+1, j), (i-1, j+1), (i, j+1), (i+1, j+1), level k
    T w0[3], w1[3];                    // u0 and acc_in of B at the cell
};

// Bases of the face components and RK arrays at cell (0, 0, 0) and the plane
// strides of the three face boxes and the state.
template <typename T>
struct BPatch {
    const T *x4, *x5, *y4, *y5, *z4, *z5, *u0, *acc_in;
    T *acc_out, *out;
    int X0, X01, Y0, Y01, Z01, s2;     // rows and planes (rows of z faces as of y faces)
    long sv;
    bool ru0, rac;                     // the stage reads u0, acc_in
};

template <typename T>
__device__ __forceinline__ void blevel_upper(const BPatch<T> &B, uint32_t ox, uint32_t oy, uint32_t oz, BLevel<T> &L)
{
    L.x5h0 = sw::ld32(B.x5 + B.X01, ox);
    L.x5h1 = sw::ld32(B.x5 + B.X01 + 1, ox);
    L.y4h0 = sw::ld32(B.y4 + B.Y01, oy);
    L.y4h1 = sw::ld32(B.y4 + B.Y01 + B.Y0, oy);
    L.z4m = sw::ld32(B.z4 + B.Z01 - 1, oz);
    L.z4c = sw::ld32(B.z4 + B.Z01, oz);
    L.z4p = sw::ld32(B.z4 + B.Z01 + 1, oz);
    L.z5m = sw::ld32(B.z5 + B.Z01 - B.Y0, oz);
    L.z5c = sw::ld32(B.z5 + B.Z01, oz);
    L.z5p = sw::ld32(B.z5 + B.Z01 + B.Y0, oz);
}
template <typename T>
__device__ __forceinline__ void blevel_load(const BPatch<T> &B, uint32_t ox, uint32_t oy, uint32_t oz, uint32_t os,
                                            BLevel<T> &L)
{
    blevel_upper(B, ox, oy, oz, L);
    L.x4[0] = sw::ld32(B.x4 - B.X0, ox);
    L.x4[1] = sw::ld32(B.x4, ox);
    L.x4[2] = sw::ld32(B.x4 - B.X0 + 1, ox);
    L.x4[3] = sw::ld32(B.x4 + 1, ox);
    L.x4[4] = sw::ld32(B.x4 + B.X0, ox);
    L.x4[5] = sw::ld32(B.x4 + B.X0 + 1, ox);
    L.y5[0] = sw::ld32(B.y5 - 1, oy);
    L.y5[1] = sw::ld32(B.y5, oy);
    L.y5[2] = sw::ld32(B.y5 + 1, oy);
    L.y5[3] = sw::ld32(B.y5 + B.Y0 - 1, oy);
    L.y5[4] = sw::ld32(B.y5 + B.Y0, oy);
    L.y5[5] = sw::ld32(B.y5 + B.Y0 + 1, oy);
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        L.w0[m] = B.ru0 ? sw::ld32(B.u0 + (4 + m) * B.sv, os) : T(0);
        L.w1[m] = B.rac ? sw::ld32(B.acc_in + (4 + m) * B.sv, os) : T(0);
    }
}

template <typename T>
__device__ __forceinline__ void update_b_patch(const T *fx, const T *fy, const T *fz, const PatchDesc &D,
                                               const Geom &G, const FaceBox (&F)[3], const XFuse<T> &xf, int t_lo,
                                               int t_hi)
{
    constexpr int KSEG = 16;
    BPatch<T> B;
    B.X0 = G.n[0] + 1; B.X01 = (int)F[0].s[2];
    B.Y0 = G.n[0] + 2; B.Y01 = (int)F[1].s[2]; B.Z01 = (int)F[2].s[2];
    B.s2 = (int)G.s[2];
    B.x4 = fx + 4 * F[0].sc + B.X0 + B.X01; B.x5 = fx + 5 * F[0].sc + B.X0 + B.X01;
    B.y4 = fy + 4 * F[1].sc + 1 + B.Y01;    B.y5 = fy + 5 * F[1].sc + 1 + B.Y01;
    B.z4 = fz + 4 * F[2].sc + 1 + B.Y0;     B.z5 = fz + 5 * F[2].sc + 1 + B.Y0;
    B.u0 = xf.u0 + G.base; B.acc_in = xf.acc_in + G.base;
    B.acc_out = xf.acc_out + G.base; B.out = xf.out + G.base;
    B.sv = G.sv;
    const StageCoef &c = xf.c;
    B.ru0 = c.s < 3; B.rac = c.s > 0;
    const T idx = T(G.idl[0]), idy = T(G.idl[1]), idz = T(G.idl[2]);
    const T q = T(0.25), bdt = T(c.bdt), cdt = T(c.cdt);
    const int tid = threadIdx.x + sw::TILE * threadIdx.y;
    const int items = min(G.n[0] * G.n[1] * ((G.n[2] + KSEG - 1) / KSEG), t_hi * RB);
    for (int it = t_lo * RB + tid; it < items; it += RB) {
        const uint32_t col = D.nx.div(it), ks = D.ny.div(col);
        const uint32_t i = it - col * D.nx.d, j = col - ks * D.ny.d, k0 = ks * KSEG;
        const int k1 = min((int)k0 + KSEG, G.n[2]);
        uint32_t ox = i + j * B.X0 + k0 * B.X01, oy = i + j * B.Y0 + k0 * B.Y01, oz = i + j * B.Y0 + k0 * B.Z01;
        uint32_t os = i + j * (uint32_t)G.s[1] + k0 * (uint32_t)B.s2;
        BLevel<T> cur, nxt;
        // carried values at the lower z-level k0 (as march_column): the upper
        // part of level k0 - 1
        T x5c0, x5c1, y4c0, y4c1, Ey0, Ey1, Ex0, Ex1;
        {
            // level k0 - 1 through bases one plane lower (k0 may be 0)
            BPatch<T> C = B;
            C.x5 -= B.X01; C.y4 -= B.Y01; C.z4 -= B.Z01; C.z5 -= B.Z01;
            BLevel<T> low;
            blevel_upper(C, ox, oy, oz, low);
            const T x5lo0 = sw::ld32(C.x5, ox), x5lo1 = sw::ld32(C.x5 + 1, ox);
            const T y4lo0 = sw::ld32(C.y4, oy), y4lo1 = sw::ld32(C.y4 + B.Y0, oy);
            blevel_load(B, ox, oy, oz, os, cur);
            x5c0 = low.x5h0; x5c1 = low.x5h1; y4c0 = low.y4h0; y4c1 = low.y4h1;
            T t;
            t = -low.z4m; t -= low.z4c; t += x5lo0; t += x5c0; Ey0 = q * t;
            t = -low.z4c; t -= low.z4p; t += x5lo1; t += x5c1; Ey1 = q * t;
            t = -y4lo0; t -= y4c0; t += low.z5m; t += low.z5c; Ex0 = q * t;
            t = -y4lo1; t -= y4c1; t += low.z5c; t += low.z5p; Ex1 = q * t;
        }
        for (int k = k0; k < k1; ++k) {
            if (k + 1 < k1) blevel_load(B, ox + B.X01, oy + B.Y01, oz + B.Z01, os + B.s2, nxt);
            T t;
            t = -cur.z4m; t -= cur.z4c; t += x5c0; t += cur.x5h0; const T Ey2 = q * t;
            t = -cur.z4c; t -= cur.z4p; t += x5c1; t += cur.x5h1; const T Ey3 = q * t;
            t = -y4c0; t -= cur.y4h0; t += cur.z5m; t += cur.z5c; const T Ex2 = q * t;
            t = -y4c1; t -= cur.y4h1; t += cur.z5c; t += cur.z5p; const T Ex3 = q * t;
            t = -cur.x4[0]; t -= cur.x4[1]; t += cur.y5[0]; t += cur.y5[1]; const T Ez00 = q * t;
            t = -cur.x4[2]; t -= cur.x4[3]; t += cur.y5[1]; t += cur.y5[2]; const T Ez10 = q * t;
            t = -cur.x4[1]; t -= cur.x4[4]; t += cur.y5[3]; t += cur.y5[4]; const T Ez01 = q * t;
            t = -cur.x4[3]; t -= cur.x4[5]; t += cur.y5[4]; t += cur.y5[5]; const T Ez11 = q * t;
            T r, bxl, bxr, byl, byr, bzl, bzr;
            r = T(0); r -= (Ez01 - Ez00) * idy; r += (Ey2 - Ey0) * idz; bxl = r;
            r = T(0); r -= (Ez11 - Ez10) * idy; r += (Ey3 - Ey1) * idz; bxr = r;
            r = T(0); r -= (Ex2 - Ex0) * idz; r += (Ez10 - Ez00) * idx; byl = r;
            r = T(0); r -= (Ex3 - Ex1) * idz; r += (Ez11 - Ez01) * idx; byr = r;
            r = T(0); r -= (Ey1 - Ey0) * idx; r += (Ex1 - Ex0) * idy; bzl = r;
            r = T(0); r -= (Ey3 - Ey2) * idx; r += (Ex3 - Ex2) * idy; bzr = r;
            const T Lb[3] = { T(0.5) * (bxl + bxr), T(0.5) * (byl + byr), T(0.5) * (bzl + bzr) };
            // rk_store_b's expressions on the preloaded u0 / acc_in values
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                T *const acc = B.acc_out + (4 + m) * B.sv, *const out = B.out + (4 + m) * B.sv;
                if (c.s == 0) {
                    sw::st32<T>(acc, os, cur.w0[m] + bdt * Lb[m]);
                    sw::st32<T>(out, os, cur.w0[m] + cdt * Lb[m]);
                } else if (c.s < 3) {
                    sw::st32<T>(acc, os, cur.w1[m] + bdt * Lb[m]);
                    sw::st32<T>(out, os, cur.w0[m] + cdt * Lb[m]);
                } else {
                    sw::st32<T>(out, os, cur.w1[m] + cdt * Lb[m]);
                }
            }
            Ey0 = Ey2; Ey1 = Ey3; Ex0 = Ex2; Ex1 = Ex3;
            x5c0 = cur.x5h0; x5c1 = cur.x5h1; y4c0 = cur.y4h0; y4c1 = cur.y4h1;
            ox += B.X01; oy += B.Y01; oz += B.Z01; os += B.s2;
            if (k + 1 < k1) cur = nxt;
        }
    }
}

// A patch's geometry and its face buffers, formed anew for each phase
// (the patch number is made opaque): kept through all phases, the scalars of
// one stood in the way of the next, with a thousand moves of spilled scalar
// registers.  232-344 are spilled (to lanes of VGPRs) all the same, 57-88 with
// whole patches only: the items' ranges and waits came on top.
template <typename T>
struct Patch {
    PatchDesc D;
    Geom G;
    FaceBox F[3];
    T *fx, *fy, *fz;
    __device__ __forceinline__ Patch(const BatchArgs<T> &a, int p, T *ff)
    {
        asm volatile("" : "+s"(p));
        D = load_desc(a.pd, p);
        patch_geom(D.n, a.dl, a.idl, G, F);
        fx = ff;
        fy = fx + NFC * F[0].sc;
        fz = fy + NFC * F[1].sc;
    }
    // the RK stage of this patch, with its own dt
    __device__ __forceinline__ StageCoef coef(const BatchArgs<T> &a, double dt) const
    {
        StageCoef c;
        c.mode = 1;
        c.s = a.s;
        c.bdt = a.bw * dt;
        c.cdt = a.cw * dt;
        return c;
    }
    __device__ __forceinline__ XFuse<T> xfuse(const BatchArgs<T> &a, double dt) const
    {
        return XFuse<T>{ a.u0 + D.soff, a.acc + D.soff, a.acc + D.soff, a.out + D.soff, fy, fz, F[1], F[2],
                         coef(a, dt) };
    }
};

template <int FT, typename T>
__device__ __forceinline__ void batch_stage(const BatchArgs<T> &a)
{
    constexpr int C0 = sw::XROWS_CELLS, C1 = sw::TILE * (FT + 5);
    constexpr int CMAX = (C0 > C1 ? C0 : C1) > XF_MAXC ? (C0 > C1 ? C0 : C1) : XF_MAXC;
    __shared__ T sq[sw::NQ * CMAX];
    __shared__ T hx[5 * XF_FACES];     // rho, m, E fluxes of the fused x tile
    __shared__ double sdt;
    __shared__ int next;
    const int tid = threadIdx.x + sw::TILE * threadIdx.y;
    for (;;) {
        if (tid == 0) next = atomicAdd(a.counter, 1);
        __syncthreads();
        const int qn = __builtin_amdgcn_readfirstlane(next);
        __syncthreads();
        if (qn >= a.nitem) break;
        const BatchItem I = load_item(a.items, qn);
        const int p = I.patch;
        const bool whole = I.split < 0;
        int32_t *const done = a.counter + 1 + 3 * I.split;      // items done per phase (split patches)
        T *ff;
        if (whole) {
            ff = a.scratch + (long)(a.nwhole <= a.nslot ? I.slot : (int)blockIdx.x) * a.slot_elems;
            if (a.s == 0) {
                const Patch<T> Q(a, p, ff);
                double mx;
                int bad;
                patch_speed<T>(a.u0 + Q.D.soff, Q.D, Q.G, a.P.gamma, 0, Q.G.n[0] * Q.G.n[1] * Q.G.n[2], mx, bad);
                if (tid == 0) store_dt(mx, bad, a.cfl, &a.dt[p], &a.flag[p]);
            }
        } else {
            ff = a.split_scratch + (long)I.slot * a.split_elems;
            // the slot's last patch done; the phases before this one done
            // (stage 0: and the time step stored, counted as one more)
            if (I.mask == ITEM_YZ && I.prev >= 0)
                wait_count(a.counter + 1 + 3 * I.prev + 2, load_split(a.split, I.prev).n[2]);
            if (I.mask == ITEM_X) wait_count(done, load_split(a.split, I.split).n[0] + (a.s == 0 ? 1 : 0));
            if (I.mask == ITEM_B) wait_count(done + 1, load_split(a.split, I.split).n[1]);
        }
        if (tid == 0) sdt = __hip_atomic_load(&a.dt[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        const double dtl = sdt;
        double dtp = __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(dtl)),
                                      __builtin_amdgcn_readfirstlane(__double2loint(dtl)));
        __syncthreads();
        // a non-physical patch has dt = 0 and is left unadvanced; the y and z
        // phase of a split patch in stage 0 runs before its dt is known
        const bool live = dtp != 0.0 || (!whole && I.mask == ITEM_YZ && a.s == 0);
        if (live && (I.mask & ITEM_YZ)) {
            // no ghost fill: the sweep tiles stage ghost cells from their
            // periodic images
            int lo = I.lo, hi = I.hi, ny;
            {
                const Patch<T> Q(a, p, ff);
                ny = (Q.F[1].cnt[0] * Q.F[1].cnt[2] + sw::TILE - 1) / sw::TILE;
                if (whole) { lo = 0; hi = ny; }
                sweep_yz_patch<1, FT, T>(a.us + Q.D.soff, Q.fy, Q.D, Q.G, Q.F[1], a.P, lo, min(hi, ny), sq);
            }
            {
                const Patch<T> Q(a, p, ff);
                const int nz = (Q.F[2].cnt[0] * Q.F[2].cnt[1] + sw::TILE - 1) / sw::TILE;
                sweep_yz_patch<2, FT, T>(a.us + Q.D.soff, Q.fz, Q.D, Q.G, Q.F[2], a.P, whole ? 0 : max(lo - ny, 0),
                                         whole ? nz : hi - ny, sq);
            }
        }
        // the x sweep: on the flattened x tiles it also differences every
        // direction's rho, m, E fluxes and applies their RK update, and the
        // update is left with constrained transport
        const bool flat = load_desc(a.pd, p).xflat != 0;
        if (live && flat && (I.mask & ITEM_X)) {
            const Patch<T> Q(a, p, ff);
            const int nt = ((int)Q.F[0].sc - 1 + XF_FACES - 2) / (XF_FACES - 1);
            sweep_xflat_patch<T>(a.us + Q.D.soff, Q.fx, Q.D, Q.G, Q.F[0], a.P, whole ? 0 : I.lo, whole ? nt : I.hi, sq,
                                 hx, Q.xfuse(a, dtp));
        }
        if (live && flat && (I.mask & ITEM_B)) {
            const Patch<T> Q(a, p, ff);
            update_b_patch<T>(Q.fx, Q.fy, Q.fz, Q.D, Q.G, Q.F, Q.xfuse(a, dtp), whole ? 0 : I.lo,
                              whole ? 0x7fffffff / RB : I.hi);
        }
        if (live && !flat) {         // whole patches only
            {
                const Patch<T> Q(a, p, ff);
                long na, nb;
                sw::xrows_tiles(Q.F[0], na, nb);
                for (long tb = 0; tb < nb; ++tb)
                    for (long ta = 0; ta < na; ++ta)
                        sw::sweep_tile_xrows<T, false, false, true>(a.us + Q.D.soff, Q.fx, Q.G, Q.F[0], a.P, ta, tb, sq);
            }
            // every variable: one thread per cell (marching with the hydro
            // fluxes carried too measured 1.5x slower here: more registers,
            // and whole passes of a small patch's columns half idle)
            const Patch<T> Q(a, p, ff);
            up::UpdArgs<T> ua;
            ua.u0 = a.u0 + Q.D.soff;
            ua.acc_in = a.acc + Q.D.soff;
            ua.acc_out = a.acc + Q.D.soff;
            ua.out = a.out + Q.D.soff;
            ua.ff[0] = Q.fx; ua.ff[1] = Q.fy; ua.ff[2] = Q.fz;
            ua.fb[0] = Q.F[0]; ua.fb[1] = Q.F[1]; ua.fb[2] = Q.F[2];
            ua.G = Q.G;
            ua.odelta = 0;
            ua.osv = Q.G.sv;
            ua.c = Q.coef(a, dtp);
            const int ncell = Q.G.n[0] * Q.G.n[1] * Q.G.n[2];
            for (int c = tid; c < ncell; c += RB) {
                int pos[3];
                pos[0] = c % Q.G.n[0];
                pos[1] = (c / Q.G.n[0]) % Q.G.n[1];
                pos[2] = c / (Q.G.n[0] * Q.G.n[1]);
                up::update_cell<7>(ua, pos);
            }
        }
        if (!whole) {
            const int phase = I.mask == ITEM_YZ ? 0 : I.mask == ITEM_X ? 1 : 2;
            if (phase == 0 && a.s == 0) {
                // this item's share of the patch's cells for the CFL maximum
                // (order-independent: a maximum and an integer sum)
                const Patch<T> Q(a, p, ff);
                const SplitDesc S = load_split(a.split, I.split);
                const int ncell = Q.G.n[0] * Q.G.n[1] * Q.G.n[2];
                const int c_lo = (int)((long)ncell * I.part / S.n[0]), c_hi = (int)((long)ncell * (I.part + 1) / S.n[0]);
                double mx;
                int bad;
                patch_speed<T>(a.u0 + Q.D.soff, Q.D, Q.G, a.P.gamma, c_lo, c_hi, mx, bad);
                SplitDt *const dt = a.sdt + I.split;
                if (tid == 0) {
                    __hip_atomic_fetch_max(&dt->mx, (unsigned long long)__double_as_longlong(mx), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_fetch_add(&dt->bad, bad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                if (count_done(done) == S.n[0]) {                 // thread 0 of the last item
                    acquire_all();
                    const unsigned long long m = __hip_atomic_load(&dt->mx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    const int nbad = __hip_atomic_load(&dt->bad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    store_dt(__longlong_as_double((long long)m), nbad, a.cfl, &a.dt[p], &a.flag[p]);
                    wait_memory();
                    release_all();
                    __hip_atomic_fetch_add(done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            } else {
                count_done(done + phase);
            }
        }
        __syncthreads();     // the scratch is reused by the next patch
    }
}

// Waves per SIMD: FP32 three up to 8 faces per tile, as the 48 KB of LDS
// allow, else two; FP64 two at 4 faces per tile (70 KB), else the LDS tile
// leaves room for one block per CU anyway.  The registers do not suffice for it:
// FP32 spills 18 VGPRs (76 B a lane) at 4 and 8 faces, FP64 51 (164 B) at 4; the
// other variants spill none (187-191 VGPRs; FP64 294-298 with AGPRs).  Held to one
// wave fewer these spill none either and are faster a block; more blocks win
// where the patches are many and small.  ms a step, spilled at the higher count
// / unspilled at the lower: 16384 patches of 5^3 FP32 5.17 / 6.10, FP64 8.59 / 10.52;
// 1024 of 16-64 FP32 46.1 / 43.9 (43.1 at 12 or 16 faces).
template <int FT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(FT <= 8 ? 3 : 2))) void batch_stage_f32(BatchArgs<float> a)
{
    batch_stage<FT, float>(a);
}

template <int FT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(FT <= 4 ? 2 : 1))) void batch_stage_f64(BatchArgs<double> a)
{
    batch_stage<FT, double>(a);
}

template <int FT, typename T> struct StageKernel;
template <int FT> struct StageKernel<FT, float> {
    static constexpr void (*fn)(BatchArgs<float>) = batch_stage_f32<FT>;
};
template <int FT> struct StageKernel<FT, double> {
    static constexpr void (*fn)(BatchArgs<double>) = batch_stage_f64<FT>;
};

template <int FT, typename T>
hipError_t launch_ft(const BatchArgs<T> &a, int nblocks, hipStream_t st)
{
    hipLaunchKernelGGL((StageKernel<FT, T>::fn), dim3(nblocks), dim3(sw::TILE, sw::ROWS), 0, st, a);
    return hipGetLastError();
}

}  // namespace

bool batch_xflat_ok(int nx, long nrows) { return nx >= 4 && xflat_cells(nx, nrows) <= XF_MAXC; }

template <typename T>
hipError_t launch_batch_stage(const BatchArgs<T> &a, int ft, int nblocks, hipStream_t st)
{
    switch (ft) {
    case 16: return launch_ft<16, T>(a, nblocks, st);
    case 12: return launch_ft<12, T>(a, nblocks, st);
    case 8: return launch_ft<8, T>(a, nblocks, st);
    default: return launch_ft<4, T>(a, nblocks, st);
    }
}

__global__ void batch_reset_kernel(int32_t *c, int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) c[i] = 0;
}

hipError_t launch_batch_reset(int32_t *counters, int n, hipStream_t st)
{
    hipLaunchKernelGGL(batch_reset_kernel, dim3((n + 255) / 256), dim3(256), 0, st, counters, n);
    return hipGetLastError();
}

template <typename T>
hipError_t batch_occupancy(int ft, int *blocks_per_cu)
{
    switch (ft) {
    case 16: return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, StageKernel<16, T>::fn, 256, 0);
    case 12: return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, StageKernel<12, T>::fn, 256, 0);
    case 8: return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, StageKernel<8, T>::fn, 256, 0);
    default: return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, StageKernel<4, T>::fn, 256, 0);
    }
}

template hipError_t launch_batch_stage<double>(const BatchArgs<double> &, int, int, hipStream_t);
template hipError_t launch_batch_stage<float>(const BatchArgs<float> &, int, int, hipStream_t);
template hipError_t batch_occupancy<double>(int, int *);
template hipError_t batch_occupancy<float>(int, int *);

}  // namespace ww
