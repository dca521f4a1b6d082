// ww_ghost_dev.h -- ghost zones as images of interior cells.
//
// The ghost zones of a later axis copy those of the earlier ones, so without
// user faces a ghost cell's value is that of the interior cell its coordinates
// map to axis by axis (periodic image or nearest interior cell): no order is
// needed, neither for a fill in one launch nor for a sweep that stages the
// image cells themselves.
#pragma once
#include "ww_index.h"
#include "ww_internal.h"

namespace ww {

__device__ __forceinline__ int ghost_image(int x, int n, int per_lo, int per_hi)
{
    if (x < 0) return per_lo ? x + n : 0;
    if (x >= n) return per_hi ? x - n : n - 1;
    return x;
}

// Three shells of ghost cells, numbered x fastest: the z zones over the padded
// x and y ranges, the y zones over the padded x and interior z range, the x
// zones over the interior y and z ranges.
struct GhostArgs {
    FastDiv px, py;            // padded x and y lengths
    FastDiv nx6, ny;           // 2 gx, interior y length
    FastDiv g6y;               // 2 gy
    uint32_t nz_shell, ny_shell, total;
    int per[6];                // face is periodic
};

inline long ghost_cells(const Geom &G)
{
    const long px = G.n[0] + 2 * G.g[0], py = G.n[1] + 2 * G.g[1];
    return 2L * G.g[2] * px * py + 2L * G.g[1] * px * G.n[2] + 2L * G.g[0] * G.n[1] * G.n[2];
}

// Needs fewer than 2^31 ghost cells.
inline GhostArgs ghost_args(const Geom &G, const int bc[6])
{
    const long px = G.n[0] + 2 * G.g[0], py = G.n[1] + 2 * G.g[1];
    GhostArgs A;
    A.px = FastDiv((uint32_t)px);
    A.py = FastDiv((uint32_t)py);
    A.nx6 = FastDiv((uint32_t)(G.act[0] ? 2 * G.g[0] : 1));
    A.g6y = FastDiv((uint32_t)(G.act[1] ? 2 * G.g[1] : 1));
    A.ny = FastDiv((uint32_t)G.n[1]);
    A.nz_shell = (uint32_t)(2L * G.g[2] * px * py);
    A.ny_shell = (uint32_t)(2L * G.g[1] * px * G.n[2]);
    A.total = (uint32_t)ghost_cells(G);
    for (int f = 0; f < 6; ++f) A.per[f] = bc[f] == 0;
    return A;
}

// Ghost cell t of the box.
template <typename T>
__device__ __forceinline__ void ghost_fill(T *u, const Geom &G, const GhostArgs &A, uint32_t t)
{
    int p[3];
    auto zone = [&](uint32_t g, int ax) { return (int)g < G.g[ax] ? (int)g - G.g[ax] : G.n[ax] + (int)g - G.g[ax]; };
    if (t < A.nz_shell) {
        const uint32_t r = A.px.div(t), g = A.py.div(r);
        p[0] = (int)(t - r * A.px.d) - G.g[0];
        p[1] = (int)(r - g * A.py.d) - G.g[1];
        p[2] = zone(g, 2);
    } else if (t < A.nz_shell + A.ny_shell) {
        const uint32_t q = t - A.nz_shell, r = A.px.div(q), k = A.g6y.div(r);
        p[0] = (int)(q - r * A.px.d) - G.g[0];
        p[1] = zone(r - k * A.g6y.d, 1);
        p[2] = (int)k;
    } else {
        const uint32_t q = t - A.nz_shell - A.ny_shell, r = A.nx6.div(q), k = A.ny.div(r);
        p[0] = zone(q - r * A.nx6.d, 0);
        p[1] = (int)(r - k * A.ny.d);
        p[2] = (int)k;
    }
    long di = G.base, si = G.base;
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        di += (long)p[e] * G.s[e];
        si += (long)ghost_image(p[e], G.n[e], A.per[2 * e], A.per[2 * e + 1]) * G.s[e];
    }
    T w[8];
#pragma unroll
    for (int v = 0; v < 8; ++v) w[v] = u[si + v * G.sv];
#pragma unroll
    for (int v = 0; v < 8; ++v) u[di + v * G.sv] = w[v];
}

}  // namespace ww
