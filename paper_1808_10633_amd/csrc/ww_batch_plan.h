// ww_batch_plan.h -- the work items of a batched stage and their order.
// Plain C++ (no device code), so that it is tested on the CPU.
//
// Resident blocks take the items in list order from a shared counter.  Most
// patches are one item: a block takes the whole patch through the stage, with
// face-flux buffers of its own.  A patch that would keep one block busy beyond
// the others' end is split (split >= 0) into items of three phases, worked on
// by several blocks: columns lo..hi-1 of its y and z sweeps (and in stage 0 a
// share of its CFL maximum), then x tiles lo..hi-1 with the rho, m, E update,
// then shares lo..hi-1 of the B update.  An item waits for the counts of items
// that all come earlier in the list: a block only ever waits for items that
// running blocks hold, so the waits end whatever the number of resident blocks.
#pragma once
#include <algorithm>
#include <functional>
#include <queue>
#include <set>
#include <vector>

namespace ww {

enum { ITEM_YZ = 1, ITEM_X = 2, ITEM_B = 4, ITEM_WHOLE = 7 };
struct BatchItem {
    int patch, mask;
    int lo, hi;
    int split;                 // index of the split patch, or -1
    int slot;                  // its face-flux slot (whole patches: their number among the whole ones)
    int prev;                  // split patch that had the slot before, or -1
    int part;                  // number of the item in its phase
};
// Items of a split patch per phase.
struct SplitDesc {
    int n[3];                  // y and z sweeps, x sweep, B update
    int pad_;
};

// Units of a split patch: columns of its y and z sweeps (64 positions along
// the sweep axis), x tiles (255 faces), shares of the B update (256 columns of
// up to 16 cells).
constexpr int BATCH_THREADS = 256;
inline int batch_columns(const int *n, int d)
{
    return (int)(((long)(n[0] + 2) * (n[3 - d] + 2) + 63) / 64);
}
inline int batch_x_tiles(const int *n)
{
    return (int)(((long)(n[0] + 1) * (n[1] + 2) * (n[2] + 2) - 1 + BATCH_THREADS - 2) / (BATCH_THREADS - 1));
}
inline int batch_b_shares(const int *n)
{
    return (int)(((long)n[0] * n[1] * ((n[2] + 15) / 16) + BATCH_THREADS - 1) / BATCH_THREADS);
}
// Elements (per flux component) of a patch's face buffers.
inline double batch_faces(const int *n, int d)
{
    double f = n[d] + 1.0;
    for (int e = 0; e < 3; ++e) if (e != d) f *= n[e] + 2.0;
    return f;
}
inline double batch_cost(const int *n) { return batch_faces(n, 0) + batch_faces(n, 1) + batch_faces(n, 2); }

struct BatchPlan {
    std::vector<BatchItem> items;
    std::vector<SplitDesc> split;
    std::vector<int> split_patch;   // patch of each split index
    int nwhole = 0;
    int nslot = 0;                  // face-flux buffers of split patches
    long whole_elems = 0;           // elements of a whole patch's buffers (largest)
    long split_elems = 0;           // and of a split patch's
    double share = 0.0;             // the work of a block if it were even
    double span = 0.0;              // the end of the last item by the order's simulation
};

// Costs are in faces swept by one block.  An item's wait, device-wide fences
// and count take a block as long as about 800 faces (1100 patches of 16^3,
// FP32: 1.42 ms a stage as whole patches, 1.58 ms as 12100 items).  No item is
// made smaller than 1024 faces.  These costs, and the margins of batch_plan, come
// from FP32 sets; FP64 uses them too.
constexpr double ITEM_OVERHEAD = 800.0, ITEM_MIN_FACES = 1024.0;

// Plan for `workers` resident blocks.  elems(p): face-flux elements of patch
// p; can_split(p); whole_slots: most blocks of a launch; cap: elements that
// the buffers of whole and split patches together may take.
//
// Patches costing more than `above` even shares of the work are split into
// items of `unit` shares.  The order is that of a simulation in which a free
// block takes the next item of the largest split patch whose waits are over,
// else the next whole patch (largest first), else the item whose wait ends
// first; span is the end of that simulation.
template <typename Elems, typename CanSplit>
BatchPlan batch_plan_try(int npatch, const int *dims, int workers, int whole_slots, long cap, Elems elems,
                         CanSplit can_split, double above, double unit_shares)
{
    BatchPlan P;
    std::vector<int> order(npatch);
    std::vector<double> cost(npatch);
    double total = 0.0;
    for (int p = 0; p < npatch; ++p) {
        order[p] = p;
        cost[p] = batch_cost(dims + 3 * p);
        total += cost[p];
    }
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return cost[a] > cost[b]; });
    const double share = total / workers, unit = std::max(share * unit_shares, ITEM_MIN_FACES);
    P.share = share;
    std::vector<char> is_split(npatch, 0);
    for (int p : order)
        if (cost[p] > above * share && cost[p] > 4.0 * ITEM_MIN_FACES && can_split(p)) {
            is_split[p] = 1;
            P.split_patch.push_back(p);
            P.split_elems = std::max(P.split_elems, elems(p));
        }
    auto sizes = [&]() {
        P.nwhole = npatch - (int)P.split_patch.size();
        P.whole_elems = 0;
        for (int p = 0; p < npatch; ++p)
            if (!is_split[p]) P.whole_elems = std::max(P.whole_elems, elems(p));
        const long left = cap - P.whole_elems * std::min(P.nwhole, whole_slots);
        P.nslot = P.split_patch.empty() ? 0 : (int)std::min((long)P.split_patch.size(), left / P.split_elems);
    };
    sizes();
    if (P.nslot < 1 && !P.split_patch.empty()) {      // no room: whole patches only
        std::fill(is_split.begin(), is_split.end(), 0);
        P.split_patch.clear();
        P.split_elems = 0;
        sizes();
    }
    const int ns = (int)P.split_patch.size();
    // per split patch and phase: units and cost per unit
    struct Phase { int units, items; double cost; };
    std::vector<Phase> ph(3 * (size_t)ns);
    P.split.resize(ns);
    for (int i = 0; i < ns; ++i) {
        const int *n = dims + 3 * P.split_patch[i];
        const int u[3] = { batch_columns(n, 1) + batch_columns(n, 2), batch_x_tiles(n), batch_b_shares(n) };
        const double c[3] = { batch_faces(n, 1) + batch_faces(n, 2), batch_faces(n, 0),
                              0.25 * n[0] * (double)n[1] * n[2] };
        for (int k = 0; k < 3; ++k) {
            const int m = (int)std::min((double)u[k], std::max(1.0, c[k] / unit));
            ph[3 * i + k] = Phase{ u[k], m, c[k] / m + ITEM_OVERHEAD };
            P.split[i].n[k] = m;
        }
        P.split[i].pad_ = 0;
    }
    std::vector<int> phase(ns, 0), next(ns, 0);
    std::vector<double> ends(ns, 0.0);                // end of the current phase's items so far
    typedef std::pair<double, int> Event;
    std::priority_queue<Event, std::vector<Event>, std::greater<Event>> pending;     // (ready time, split)
    std::set<int> ready;                              // split patches whose waits are over
    std::priority_queue<double, std::vector<double>, std::greater<double>> block;    // times blocks are free
    for (int w = 0; w < workers; ++w) block.push(0.0);
    for (int i = 0; i < std::min(ns, P.nslot); ++i) pending.push(Event(0.0, i));
    size_t iw = 0;
    int whole = 0;
    for (;;) {
        double t = block.top();
        while (!pending.empty() && pending.top().first <= t) { ready.insert(pending.top().second); pending.pop(); }
        while (iw < order.size() && is_split[order[iw]]) ++iw;
        int i = -1;
        if (!ready.empty()) i = *ready.begin();
        else if (iw >= order.size()) {
            if (pending.empty()) break;
            t = pending.top().first;
            i = pending.top().second;
            pending.pop();
            ready.insert(i);
        }
        block.pop();
        if (i < 0) {
            const int p = order[iw++];
            P.items.push_back(BatchItem{ p, ITEM_WHOLE, 0, 0, -1, whole++, -1, 0 });
            block.push(t + cost[p]);
            P.span = std::max(P.span, t + cost[p]);
            continue;
        }
        const int k = phase[i], m = next[i]++;
        const Phase &q = ph[3 * i + k];
        P.items.push_back(BatchItem{ P.split_patch[i], 1 << k, (int)((long)q.units * m / q.items),
                                     (int)((long)q.units * (m + 1) / q.items), i, i % P.nslot,
                                     i >= P.nslot ? i - P.nslot : -1, m });
        ends[i] = std::max(ends[i], t + q.cost);
        block.push(t + q.cost);
        P.span = std::max(P.span, t + q.cost);
        if (next[i] == q.items) {
            ready.erase(i);
            next[i] = 0;
            if (++phase[i] < 3) pending.push(Event(ends[i], i));
            else if (i + P.nslot < ns) pending.push(Event(ends[i], i + P.nslot));
        }
    }
    return P;
}

// The plan of the smallest span among whole patches only and four grains of
// splitting.  FP32, whole only / the chosen one, ms a stage: 1024 patches of
// 16-64 cells per axis 17.8 / 10.8, 64 of 32-64 17.4 / 1.9, 256 of 16-64
// 13.4 / 3.0; one 64^3 patch 16 / 0.17.  Where whole patches end within 5 % of
// an even share on half as many blocks (tuned shapes run half to all of
// `workers`) there is nothing to gain: splitting the largest of 4096 patches
// all the same cost 1 %.  And a plan has to promise a tenth over whole patches
// on three quarters or all of the blocks: 1100 equal patches on 1024 blocks,
// promised a gain over 1024 but not over 768, were 5 % slower.
template <typename Elems, typename CanSplit>
BatchPlan batch_plan(int npatch, const int *dims, int workers, int whole_slots, long cap, Elems elems,
                     CanSplit can_split)
{
    auto plan = [&](int w, double above, double unit) {
        return batch_plan_try(npatch, dims, std::max(1, w), whole_slots, cap, elems, can_split, above, unit);
    };
    const BatchPlan whole = plan(workers / 2, 1e300, 1.0);
    if (whole.span <= 1.05 * whole.share) return whole;
    const bool many = npatch > 1 << 17;         // a simulation takes 0.2 us a patch
    double ratio = 1e300;
    for (int q = many ? 4 : 3; q <= 4; ++q) {
        const BatchPlan P = plan(workers * q / 4, 1e300, 1.0);
        ratio = std::min(ratio, P.span / P.share);
    }
    BatchPlan best;
    best.span = 1e300;
    const double grain[4][2] = { { 0.5, 0.25 }, { 1.0, 0.5 }, { 0.5, 0.125 }, { 0.5, 1.0 / 16.0 } };
    for (int g = 0; g < (many ? 1 : 4); ++g) {
        BatchPlan P = plan(workers, grain[g][0], grain[g][1]);
        if (P.span < best.span) best = std::move(P);
    }
    return best.span / best.share < 0.9 * ratio ? best : whole;
}

}  // namespace ww
