// ww_index.h -- integer index arithmetic of the tiled kernels: exact division
// by a launch constant, and the numbering of the x sweep's 256-face tiles and
// the y/z sweeps' tiles.  Plain C++ (no HIP types), so that the host can
// check it.
//
// Integer work is not free beside the sweeps' floating-point work: 32-bit
// multiplies run at a quarter of the FMA rate, a 64-bit division is a
// sequence of more than a hundred instructions, and the x tiles' row numbers
// took ten of them per wave.  Every tile and face number fits 32 bits
// (a launch of 256-thread blocks has fewer than 2^24 of them, HIP's limit on
// the threads of a grid axis), divisors are known on the host, and addresses
// are a tile base (scalar) plus a 32-bit element offset (per lane).
#pragma once
#include <stdint.h>

#ifdef __HIP__
#include <hip/hip_runtime.h>
#define WW_HD __host__ __device__ __forceinline__
#else
#define WW_HD inline
#endif

namespace ww {

// n / d for 32-bit unsigned n and a launch constant d in 1..2^31 by a
// multiplication (Granlund & Montgomery, "Division by invariant integers
// using multiplication", PLDI 1994, Fig. 4.1).
struct FastDiv {
    uint32_t d, m;
    int s1, s2;
    FastDiv() = default;
    explicit FastDiv(uint32_t div) : d(div)
    {
        int l = 0;
        while ((uint64_t(1) << l) < div) ++l;
        m = (uint32_t)(((uint64_t(1) << 32) * ((uint64_t(1) << l) - div)) / div + 1);
        s1 = l < 1 ? l : 1;
        s2 = l > 1 ? l - 1 : 0;
    }
    WW_HD uint32_t div(uint32_t n) const
    {
        const uint32_t t = (uint32_t)(((uint64_t)m * n) >> 32);
        return (t + ((n - t) >> s1)) >> s2;
    }
};

// x sweep, rows of at least 86 faces: faces are numbered row by row (row =
// transverse position (jj, kk) of the face box, jj fastest; n1 rows per kk),
// a tile is up to 256 consecutive faces from face g0, touching at most four
// rows.  Row s of the tile (s = 0..3) holds tile faces from s nf - fa0 on and
// is staged with its 3 + 2 halo, so face t of row s reads its six cells from
// tile cell t + 5 s on.  A state row is nf + 5 cells long, so the staged
// cells of consecutive rows are consecutive in memory too, except where the
// rows pass to the next plane (row s = sw of the tile, tile cell cw): there
// the index jumps by the rows that the face box leaves out of a plane.
struct XTile {
    uint32_t g0;
    int nf, nface, ncell;      // faces per row; faces and staged cells of the tile
    int fa0;                   // first face within its row
    int jj0, kk0;              // row of face g0 (face-box numbering)
    int n1, sw, cw;            // rows per plane; first row and cell beyond the plane's end
    WW_HD int row_of(int t) const
    {
        const int b1 = nf - fa0;
        return (t >= b1) + (t >= b1 + nf) + (t >= b1 + 2 * nf);
    }
    WW_HD int row_of_cell(int c) const
    {
        const int o1 = nf + 5 - fa0;
        return (c >= o1) + (c >= o1 + nf + 5) + (c >= o1 + 2 * (nf + 5));
    }
    WW_HD int face_x(int t, int s) const { return t + fa0 - s * nf; }
    WW_HD int cell_of(int t, int s) const { return t + 5 * s; }      // of the face's first stencil cell
    // a plane holds one row (inactive axis) or at least five: at most one
    // plane's end in four rows
    WW_HD int jj(int s) const { return n1 == 1 ? 0 : jj0 + s - (s >= sw ? n1 : 0); }
    WW_HD int kk(int s) const { return n1 == 1 ? kk0 + s : kk0 + (s >= sw ? 1 : 0); }
    // state offset of staged cell c from staged cell 0
    WW_HD uint32_t state_rel(int c, uint32_t jump) const { return (uint32_t)c + (c >= cw ? jump : 0u); }
};

WW_HD XTile xtile(uint32_t g0, uint32_t total, const FastDiv &nf, const FastDiv &n1)
{
    XTile X;
    X.g0 = g0;
    X.nf = (int)nf.d;
    X.n1 = (int)n1.d;
    X.nface = (int)(total - g0 < 256u ? total - g0 : 256u);
    const uint32_t row = nf.div(g0);
    X.fa0 = (int)(g0 - row * nf.d);
    const uint32_t k = n1.div(row);
    X.kk0 = (int)k;
    X.jj0 = (int)(row - k * n1.d);
    X.ncell = X.nface + 5 * (X.row_of(X.nface - 1) + 1);
    X.sw = X.n1 - X.jj0;
    X.cw = X.sw * (X.nf + 5) - X.fa0;
    return X;
}

// y/z sweeps: positions of the transverse plane (na along x, then the other
// axis) are numbered row by row; lane pl of a tile that starts at position
// (a0, b0) is q rows further on, at x index a0 + pl - q na.
WW_HD int yz_rows_on(uint32_t a0, int pl, const FastDiv &na, int pw)
{
    const uint32_t a = a0 + (uint32_t)pl;
    if (na.d >= (uint32_t)pw) return a >= na.d ? 1 : 0;
    return (int)na.div(a);
}

}  // namespace ww
