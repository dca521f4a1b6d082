// ww_batch.h -- internal types of the batched (many-patch) stage.
#pragma once
#include "ww_batch_plan.h"
#include "ww_index.h"
#include "ww_internal.h"

namespace ww {

// One patch of the arena: its cells per axis, where its padded state starts
// in the arena, whether its x sweep uses the flattened tile, and the divisors
// of its cell and face numbers.  A multiple of 8 bytes: the kernel reads it
// in 8-byte words.
struct PatchDesc {
    int n[3];
    int xflat;
    long soff;
    FastDiv nx, ny;            // n0, n1 (cells)
    FastDiv na;                // n0 + 2 (y and z faces along x)
    FastDiv nf, n1f;           // n0 + 1, n1 + 2 (x faces per row, rows per plane)
    FastDiv nxp;               // n0 + 6 (cells of a staged row)
};
static_assert(sizeof(PatchDesc) % 8 == 0, "read in 8-byte words");

// Geometry of a padded periodic patch of cell width dl and its face boxes.
WW_HD void patch_geom(const int (&n)[3], double dl, double idl, Geom &G, FaceBox (&F)[3])
{
    int N[3];
    for (int d = 0; d < 3; ++d) {
        G.n[d] = n[d];
        G.act[d] = 1;
        G.g[d] = 3;
        G.dl[d] = dl;
        G.idl[d] = idl;
        N[d] = n[d] + 6;
    }
    G.s[0] = 1;
    G.s[1] = N[0];
    G.s[2] = (long)N[0] * N[1];
    G.sv = (long)N[0] * N[1] * N[2];
    G.base = 3 + 3 * G.s[1] + 3 * G.s[2];
    for (int d = 0; d < 3; ++d) {
        FaceBox &B = F[d];
        for (int e = 0; e < 3; ++e) {
            if (e == d) { B.lo[e] = 0; B.cnt[e] = n[e] + 1; }
            else { B.lo[e] = -1; B.cnt[e] = n[e] + 2; }
        }
        B.s[0] = 1;
        B.s[1] = B.cnt[0];
        B.s[2] = (long)B.cnt[0] * B.cnt[1];
        B.sc = (long)B.cnt[0] * B.cnt[1] * B.cnt[2];
    }
}

// Counts of a stage: the next item, then per split patch the items done per phase.
inline int stage_counters(int nsplit) { return 1 + 3 * nsplit; }
// Stage 0's CFL maximum (bit pattern of a positive double) and bad-cell count
// of a split patch.
struct SplitDt {
    unsigned long long mx;
    int bad;
    int pad_;
};

template <typename T>
struct BatchArgs {
    const PatchDesc *pd;
    const BatchItem *items;
    const SplitDesc *split;
    int nitem, nwhole;
    int32_t *counter;          // the stage's counters (cleared before the stage)
    SplitDt *sdt;              // cleared before stage 0
    const T *u0;               // arena of the step's initial state
    T *us;                     // arena of the stage input
    T *acc;                    // arena of the RK accumulator
    T *out;                    // arena of the stage output
    T *scratch;                // face fluxes of whole patches, slot_elems per block (or per patch if fewer)
    long slot_elems;
    int nslot;
    T *split_scratch;          // face fluxes of split patches
    long split_elems;
    double *dt;                // per-patch time step (written in stage 0)
    int32_t *flag;             // per-patch count of non-physical cells
    double cfl;
    double dl, idl;            // cell width of every patch and axis
    int s;                     // RK stage 0..3
    double bw, cw;             // weights of dt L in acc and in out
    Phys P;
};

bool batch_xflat_ok(int nx, long nrows);

template <typename T>
hipError_t launch_batch_stage(const BatchArgs<T> &a, int ft, int nblocks, hipStream_t st);

template <typename T>
hipError_t batch_occupancy(int ft, int *blocks_per_cu);

// Clear n counters (a kernel, so that it can be captured in a graph).
hipError_t launch_batch_reset(int32_t *counters, int n, hipStream_t st);

}  // namespace ww
