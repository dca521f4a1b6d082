"""The work-item list of the batched form (csrc/ww_batch_plan.h), built for the
CPU: every patch is covered exactly once, an item waits only for items earlier
in the list, face buffers are handed on only after their last user, and the
scratch stays within what it was allowed."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1808_10633_amd", "csrc")

PROGRAM = r"""
#include "ww_batch_plan.h"
#include <cstdio>
using namespace ww;
#define CHECK(c) do { if (!(c)) { printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)

static int check_one(const std::vector<int> &dims, int workers, int slots, double capf, int never, int expect, int grain)
{
    const int np = (int)dims.size() / 3;
    auto elems = [&](int p) { return 7 * (long)batch_cost(&dims[3 * p]); };
    long biggest = 0;
    for (int p = 0; p < np; ++p) biggest = std::max(biggest, elems(p));
    const long cap = (long)(capf * biggest * slots);
    auto can = [&](int p) { return !never || p % never != 0; };
    const BatchPlan P = grain < 0 ? batch_plan(np, dims.data(), workers, slots, cap, elems, can)
                                  : batch_plan_try(np, dims.data(), workers, slots, cap, elems, can, grain > 1 ? 1.0 : 0.5,
                                                   1.0 / (2 << grain));
    const int ns = (int)P.split_patch.size();
    if (expect >= 0 && grain < 0) CHECK((ns > 0) == (expect > 0));
    CHECK((int)P.split.size() == ns && P.nwhole == np - ns);
    CHECK(ns == 0 || P.nslot * P.split_elems + std::min(P.nwhole, slots) * P.whole_elems <= cap);
    CHECK(ns == 0 || (P.nslot >= 1 && P.nslot <= ns));
    std::vector<int> whole(np, 0), seen(3 * ns, 0), upto(3 * ns, 0);
    int nw = 0;
    for (const BatchItem &I : P.items) {
        CHECK(I.patch >= 0 && I.patch < np);
        const int *n = &dims[3 * I.patch];
        if (I.split < 0) {
            CHECK(I.mask == ITEM_WHOLE && !whole[I.patch]++ && I.slot == nw++);
            CHECK(elems(I.patch) <= P.whole_elems);
            continue;
        }
        CHECK(I.split < ns && P.split_patch[I.split] == I.patch && elems(I.patch) <= P.split_elems);
        CHECK(!never || I.patch % never != 0);
        CHECK(I.slot >= 0 && I.slot < P.nslot);
        const int k = I.mask == ITEM_YZ ? 0 : I.mask == ITEM_X ? 1 : 2, q = 3 * I.split + k;
        CHECK(I.mask == 1 << k);
        // consecutive, non-empty ranges
        CHECK(I.part == seen[q] && I.lo == upto[q] && I.hi > I.lo);
        upto[q] = I.hi;
        ++seen[q];
        // the phase before is complete in the list
        if (k) CHECK(seen[q - 1] == P.split[I.split].n[k - 1]);
        // and so is the patch that had the face buffers before
        if (I.prev >= 0) {
            CHECK(I.prev < I.split && I.prev % P.nslot == I.slot && I.split - I.prev == P.nslot);
            CHECK(seen[3 * I.prev + 2] == P.split[I.prev].n[2]);
        } else CHECK(I.split < P.nslot);
        const int units = k == 0 ? batch_columns(n, 1) + batch_columns(n, 2) : k == 1 ? batch_x_tiles(n) : batch_b_shares(n);
        CHECK(I.hi <= units);
        if (seen[q] == P.split[I.split].n[k]) CHECK(I.hi == units);
    }
    for (int i = 0; i < ns; ++i) {
        whole[P.split_patch[i]]++;
        for (int k = 0; k < 3; ++k) CHECK(seen[3 * i + k] == P.split[i].n[k]);
    }
    for (int p = 0; p < np; ++p) CHECK(whole[p] == 1);
    CHECK(nw == P.nwhole);
    return 0;
}

// The chosen plan, and every grain (buffers are handed on where the scratch is short).
static int check(const std::vector<int> &dims, int workers, int slots, double capf, int never, int expect)
{
    for (int grain = -1; grain < 4; ++grain)
        if (check_one(dims, workers, slots, capf, never, expect, grain)) { printf("grain %d\n", grain); return 1; }
    return 0;
}

int main()
{
    unsigned long long x = 88172645463325252ull;
    auto rnd = [&](int n) { x ^= x << 13; x ^= x >> 7; x ^= x << 17; return (int)((x >> 20) % n); };
    auto draw = [&](int np, std::vector<int> edges) {
        std::vector<int> d;
        for (int i = 0; i < 3 * np; ++i) d.push_back(edges[rnd((int)edges.size())]);
        return d;
    };
    for (int w : { 1, 3, 512, 768 }) {
        if (check(draw(1, { 64 }), w, 1024, 1.0, 0, w > 3 ? 1 : -1)) return 1;
        if (check(draw(1, { 4 }), w, 1024, 1.0, 0, 0)) return 1;
        if (check(draw(1, { 255, 100 }), w, 1024, 1.0, 0, -1)) return 1;
        if (check(draw(20, { 8, 12, 16, 24 }), w, 1024, 1.0, 0, -1)) return 1;
        if (check(draw(1024, { 16, 24, 32, 48, 64 }), w, 1024, 1.0, 0, -1)) return 1;
        if (check(draw(1100, { 16 }), w, 1024, 1.0, 0, -1)) return 1;        // buffers handed on
        if (check(draw(300, { 16, 24, 33 }), w, 1024, 0.02, 0, -1)) return 1;
        if (check(draw(300, { 16, 24, 33 }), w, 1024, 0.3, 2, -1)) return 1;
        if (check(draw(1024, { 16, 64 }), w, 1024, 1.0, 3, -1)) return 1;
        if (check(draw(9000, { 4, 5, 9, 12 }), w, 1024, 1.0, 0, w >= 512 ? 0 : -1)) return 1;
        std::vector<int> one = draw(2000, { 4, 8 });
        one[300] = one[301] = one[302] = 128;
        if (check(one, w, 1024, 1.0, 0, w >= 512 ? 1 : -1)) return 1;
    }
    for (int it = 0; it < 100; ++it) {
        std::vector<int> e;
        for (int i = 0; i < 4; ++i) e.push_back(4 + rnd(80));
        if (check(draw(1 + rnd(400), e), 1 + rnd(900), 1024, 0.001 * rnd(1000), rnd(5), -1)) return 1;
    }
    printf("ok\n");
    return 0;
}
"""


def test_batch_plan(tmp_path):
    src = tmp_path / "plan.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "plan"
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
