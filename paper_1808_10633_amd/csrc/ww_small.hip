// ww_small.hip -- the sweeps of a small box in one launch.
//
// A small box (a tube, a 2-D problem, a 32^3 test box) has a few hundred tiles
// per direction or fewer: each sweep is one round of blocks, as long as one
// block's latency (8-23 us at 32^3 to 97 x 61 x 43), and a right-hand side was
// three ghost fills, three such sweeps in a row and the update.  Here every
// tile of the three directions is a block of one launch.  The tiles stage
// ghost cells from their interior images, so no sweep waits for the ghost
// fill, which runs as more blocks of the same launch where the caller's
// state is to have its ghosts (a step's own stage arrays need none).
//
// A block stages up to SMALL_CELLS cells of its tile, 256 faces, and computes
// one face per thread.  The three directions and the two x tilings differ in
// where a cell and a face lie; staging and flux are one piece of code with
// the sweep frame chosen at run time (three copies of the flux, 15 KB of code
// each, would be fetched cold by every launch).
#include "ww_ghost_dev.h"
#include "ww_sweep_dev.h"

namespace ww {
namespace {

constexpr int SMALL_CELLS = 592;   // x rows of 4 faces: 65 rows of 9 cells
constexpr int IT = 2;              // cells per thread loaded together (more only in short x rows)

// y/z tiles of pw positions x ft faces, at most 256 faces and SMALL_CELLS
// cells: of the shapes with 5 to 16 faces the one with the fewest tiles (with
// 8 faces the 33 faces of a 32-cell axis would take five tiles, the last with
// one face; 11 take three), the deeper tile of two (fewer staged cells).
struct YZShape {
    int pw, ft;
    long tiles;
};
YZShape yz_shape(const FaceBox &F, int d)
{
    YZShape best{ 32, 8, 0 };
    const long npos = (long)F.cnt[0] * F.cnt[3 - d];
    for (int ft = 5; ft <= 16; ++ft) {
        const int pw = 256 / ft;
        if (pw * (ft + 5) > SMALL_CELLS) continue;
        const long tiles = (npos + pw - 1) / pw * ((F.cnt[d] + ft - 1) / ft);
        if (best.tiles == 0 || tiles <= best.tiles) best = YZShape{ pw, ft, tiles };
    }
    return best;
}

template <typename T>
struct SmallArgs {
    T *u;
    T *flux[3];
    Geom G;
    FaceBox F[3];
    Phys P;
    uint32_t bx, by, bz;           // first block past the x, y, z tiles; ghost blocks follow
    FastDiv nf, n1, nxp;           // x faces per row, rows per plane, cells of a padded row
    struct YZ {
        FastDiv na, nb, pw;        // positions along x, tiles along the sweep axis, positions per tile
        uint32_t npos;
        int ft;
    } Y[2];                        // y and z tiles
    GhostArgs gh;
};

template <typename T>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void small_sweeps_kernel(SmallArgs<T> A)
{
    __shared__ T sq[sw::NQ * SMALL_CELLS];
    const Geom &G = A.G;
    const uint32_t blk = blockIdx.x;
    const int tid = threadIdx.x;
    if (blk >= A.bz) {
        const uint32_t t = (blk - A.bz) * 256u + tid;
        if (t < A.gh.total) ghost_fill(A.u, G, A.gh, t);
        return;
    }
    const int dir = blk < A.bx ? 0 : blk < A.by ? 1 : 2;
    const bool seg = A.nf.d >= (uint32_t)sw::XSEG_MIN;
    const FaceBox &F = A.F[dir];
    const int b = dir == 1 ? 2 : 1;                    // second axis of a y/z tile's positions
    // the tile
    XTile X;
    int ncell, r_lo = 0, f0 = 0;
    uint32_t p0 = 0, g0 = 0;
    const typename SmallArgs<T>::YZ &Y = A.Y[dir == 2 ? 1 : 0];
    const int pw = (int)Y.pw.d, ft = Y.ft;
    if (dir == 0) {
        g0 = blk * 256u;
        if (seg) {
            X = xtile(g0, (uint32_t)F.sc, A.nf, A.n1);
            ncell = X.ncell;
        } else {
            const uint32_t g1 = min(g0 + 255u, (uint32_t)F.sc - 1u);
            r_lo = (int)A.nf.div(g0);
            ncell = ((int)A.nf.div(g1) - r_lo + 1) * (int)A.nxp.d;
        }
    } else {
        const uint32_t t = blk - (dir == 1 ? A.bx : A.by), ta = Y.nb.div(t);
        p0 = ta * pw;
        f0 = (int)(t - ta * Y.nb.d) * ft;
        ncell = pw * min(ft + 5, G.n[dir] + 6 - f0);       // rows f0 - 3 .. n + 2 at most
    }
    const int t1 = dir == 2 ? 0 : dir + 1, t2 = dir == 0 ? 2 : dir - 1;
    // state offset of tile cell c, through its interior image
    auto cell = [&](int c) {
        int p[3];
        if (dir == 0) {
            if (seg) {
                const int s = X.row_of_cell(c);
                p[0] = c + X.fa0 - 3 - s * (X.nf + 5);
                p[1] = F.lo[1] + X.jj(s);
                p[2] = F.lo[2] + X.kk(s);
            } else {
                const uint32_t rr = A.nxp.div(c), row = r_lo + rr, kk = A.n1.div(row);
                p[0] = (int)(c - rr * A.nxp.d) - 3;
                p[1] = F.lo[1] + (int)(row - kk * A.n1.d);
                p[2] = F.lo[2] + (int)kk;
            }
        } else {
            const uint32_t r = Y.pw.div(c), q = min(p0 + (c - r * pw), Y.npos - 1), k = Y.na.div(q);
            p[0] = F.lo[0] + (int)(q - k * Y.na.d);
            const int pb = F.lo[b] + (int)k, y = f0 - 3 + (int)r;
            p[1] = b == 1 ? pb : y;
            p[2] = b == 2 ? pb : y;
        }
        uint32_t e = 0;
#pragma unroll
        for (int d = 0; d < 3; ++d)
            e += (uint32_t)ghost_image(p[d], G.n[d], A.gh.per[2 * d], A.gh.per[2 * d + 1]) * (uint32_t)G.s[d];
        return e;
    };
    const int cm[8] = { 0, 1 + dir, 1 + t1, 1 + t2, 4 + dir, 4 + t1, 4 + t2, 7 };
    // stage: a thread's loads first; cells past the end repeat the last one
    T w[IT][8];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const uint32_t e = cell(min(tid + it * 256, ncell - 1));
#pragma unroll
        for (int v = 0; v < 8; ++v) w[it][v] = sw::ld32(A.u + G.base + cm[v] * G.sv, e);
    }
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const int c = tid + it * 256;
        if (c < ncell) sw::stage_values<T>(w[it], A.P.gamma, sq + c, SMALL_CELLS);
    }
    for (int c = tid + IT * 256; c < ncell; c += 256) {
        const uint32_t e = cell(c);
        T x[8];
#pragma unroll
        for (int v = 0; v < 8; ++v) x[v] = sw::ld32(A.u + G.base + cm[v] * G.sv, e);
        sw::stage_values<T>(x, A.P.gamma, sq + c, SMALL_CELLS);
    }
    __syncthreads();
    // the thread's face: its first cell in the tile and its place in the flux box
    int off, cstr;
    uint32_t fi;
    bool act;
    if (dir == 0) {
        cstr = 1;
        fi = g0 + tid;
        act = fi < (uint32_t)F.sc;
        const uint32_t row = A.nf.div(fi);
        off = seg ? X.cell_of(tid, X.row_of(tid))
                  : ((int)row - r_lo) * (int)A.nxp.d + (int)(fi - row * A.nf.d);
    } else {
        cstr = pw;
        off = tid;
        const uint32_t r = Y.pw.div(tid), q = p0 + (tid - r * pw), k = Y.na.div(q);
        const int f = f0 + (int)r;
        act = (int)r < ft && q < Y.npos && f < F.cnt[dir];
        fi = (q - k * Y.na.d) + k * (uint32_t)F.s[b] + (uint32_t)f * (uint32_t)F.s[dir];
    }
    if (act) {
        T out[7];
        sw::face_flux<T>(sq, SMALL_CELLS, off, cstr, A.P.gamma, A.P.igm1, (T)A.P.eps, out);
        const int gc[7] = { 0, 1 + dir, 1 + t1, 1 + t2, 4, 5, 6 };   // sweep frame -> grid component
#pragma unroll
        for (int c = 0; c < 7; ++c) sw::st32<T>(A.flux[dir] + gc[c] * F.sc, fi, out[c]);
    }
}

}  // namespace

long small_sweep_tiles(const Geom &G, const FaceBox F[3])
{
    long n = 0;
    for (int d = 0; d < 3; ++d) {
        if (!G.act[d]) continue;
        n += d == 0 ? (F[0].sc + 255) / 256 : yz_shape(F[d], d).tiles;
    }
    return n;
}

template <typename T>
hipError_t launch_small_sweeps(T *u, T *const flux[3], const Geom &G, const FaceBox F[3], const Phys &P,
                               const int bc[6], bool ghosts, hipStream_t st)
{
    // offsets are 32-bit in bytes; a row of three faces does not occur (an
    // active axis has three cells)
    if (G.sv > (1L << 28) || small_sweep_tiles(G, F) > 2 * SMALL_TILES) return hipErrorInvalidValue;
    SmallArgs<T> A;
    A.u = u;
    for (int d = 0; d < 3; ++d) { A.flux[d] = flux[d]; A.F[d] = F[d]; }
    A.G = G;
    A.P = P;
    A.nf = FastDiv((uint32_t)F[0].cnt[0]);
    A.n1 = FastDiv((uint32_t)F[0].cnt[1]);
    A.nxp = FastDiv((uint32_t)(G.n[0] + 6));
    uint32_t tiles[2];
    for (int d = 1; d <= 2; ++d) {
        const YZShape S = yz_shape(F[d], d);
        typename SmallArgs<T>::YZ &Y = A.Y[d - 1];
        Y.npos = (uint32_t)F[d].cnt[0] * (uint32_t)F[d].cnt[3 - d];
        Y.na = FastDiv((uint32_t)F[d].cnt[0]);
        Y.nb = FastDiv((uint32_t)((F[d].cnt[d] + S.ft - 1) / S.ft));
        Y.pw = FastDiv((uint32_t)S.pw);
        Y.ft = S.ft;
        tiles[d - 1] = G.act[d] ? (uint32_t)S.tiles : 0u;
    }
    A.bx = G.act[0] ? (uint32_t)((F[0].sc + 255) / 256) : 0u;
    A.by = A.bx + tiles[0];
    A.bz = A.by + tiles[1];
    A.gh = ghost_args(G, bc);
    const uint32_t nb = A.bz + (ghosts ? (A.gh.total + 255) / 256 : 0u);
    hipLaunchKernelGGL((small_sweeps_kernel<T>), dim3(nb), dim3(256), 0, st, A);
    return hipGetLastError();
}

template hipError_t launch_small_sweeps<double>(double *, double *const[3], const Geom &, const FaceBox[3], const Phys &,
                                                const int[6], bool, hipStream_t);
template hipError_t launch_small_sweeps<float>(float *, float *const[3], const Geom &, const FaceBox[3], const Phys &,
                                               const int[6], bool, hipStream_t);

}  // namespace ww
