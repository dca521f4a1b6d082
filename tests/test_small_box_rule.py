"""Which boxes run their sweeps in one launch (small_box, csrc/ww_internal.h),
with the tile counts of csrc/ww_small.hip built for the CPU."""
import os
import re
import subprocess

from test_routed_addresses import CLANG, CSRC, HIP_RUNTIME, ROOT

PROGRAM = r"""
#include "ww_small.hip"
#include <cstdio>
using namespace ww;

static bool small(int nx, int ny, int nz, int bc = 0, int weights = 0, int slab = 0)
{
    const int n[3] = { nx, ny, nz };
    wombat_weno_config c{};
    c.nx = nx; c.ny = ny; c.nz = nz;
    c.weights = weights;
    c.slab_planes = slab;
    for (int f = 0; f < 6; ++f) c.bc[f] = bc;
    Geom G{};
    FaceBox F[3]{};
    for (int d = 0; d < 3; ++d) {
        G.n[d] = n[d]; G.act[d] = n[d] > 1; G.g[d] = G.act[d] ? 3 : 0;
        for (int e = 0; e < 3; ++e) F[d].cnt[e] = e == d ? n[e] + 1 : n[e] > 1 ? n[e] + 2 : 1;
        F[d].sc = (long)F[d].cnt[0] * F[d].cnt[1] * F[d].cnt[2];
    }
    return small_box(c, G, F);
}
int ww::sweep_x_fused_min_faces() { return sw::XSEG_MIN; }

#define CHECK(c) do { if (!(c)) { printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)
int main()
{
    // 1-D along x: to 2^17 faces
    CHECK(small(3, 1, 1) && small(4096, 1, 1) && small(131071, 1, 1));
    CHECK(!small(131072, 1, 1) && !small(262144, 1, 1) && !small(1000000, 1, 1));
    // 1-D along y or z: columns of one position
    CHECK(small(1, 4096, 1) && small(1, 1, 4096) && small(1, 65535, 1) && !small(1, 65536, 1));
    // 2-D, 3-D with and without the fused x sweep
    CHECK(small(128, 128, 1) && small(700, 700, 1) && !small(760, 760, 1));
    CHECK(small(32, 32, 32) && small(80, 80, 80) && small(84, 84, 84) && !small(84, 100, 100));
    CHECK(small(97, 61, 43) && small(88, 50, 50) && !small(100, 71, 66) && !small(128, 128, 128));
    // and never with user faces, other weights or slabs
    CHECK(!small(32, 32, 32, 2) && !small(32, 32, 32, 0, 1) && !small(32, 32, 32, 0, 0, 8));
    printf("ok\n");
    return 0;
}
"""


def test_small_box_rule(tmp_path):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(HIP_RUNTIME)
    for f in os.listdir(CSRC):
        if f.endswith(".h") or f == "ww_small.hip":
            # register constraints and occupancy hints of the GPU
            text = re.sub(r"^\s*asm volatile\(.*\);$|__attribute__\(\(amdgpu_\w+\(\d\)\)\)", "",
                          open(os.path.join(CSRC, f)).read(), flags=re.M)
            (tmp_path / f).write_text(text.replace('"../../include/wombat_weno.h"', '"wombat_weno.h"'))
    (tmp_path / "main.cpp").write_text(PROGRAM)
    exe = tmp_path / "rule"
    r = subprocess.run([CLANG, "-std=c++17", "-O1", "-w", "-pthread", "-I", str(tmp_path), "-I", os.path.join(ROOT, "include"),
                        str(tmp_path / "main.cpp"), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
