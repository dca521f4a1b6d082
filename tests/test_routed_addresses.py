"""The learned form's kernels (csrc/ww_router.hip) built for the CPU and run on
boxes whose variables and face components pass 2^32 bytes, and on boxes just
under that, over sparse memory: 256 host threads stand for a block.  The last
tiles' faces, the queued full fluxes and the cells next to troubled faces are
stored at their own places and read from them."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1808_10633_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"

# What the device code needs of the HIP runtime and the GPU, on host threads.
HIP_RUNTIME = r"""
#pragma once
#include <math.h>
#include <pthread.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>
#include <algorithm>
#include <cmath>
#define __HIP__ 1
#define __host__
#define __device__
#define __global__
#define __forceinline__ inline
#define __shared__ static
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))
using std::min;
using std::max;
struct dim3 { unsigned x, y, z; dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {} };
typedef int hipError_t;
typedef void *hipStream_t;
enum { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorInvalidConfiguration = 9 };
inline hipError_t hipGetLastError() { return 0; }
inline hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t) { return 0; }
#define hipLaunchKernelGGL(...) ((void)0)
inline thread_local dim3 threadIdx;
inline dim3 blockIdx, gridDim, blockDim;
inline pthread_barrier_t block_barrier;
inline bool one_thread = false;
inline void __syncthreads() { if (!one_thread) pthread_barrier_wait(&block_barrier); }
inline unsigned long long wave_bits[4];
inline unsigned long long __ballot(bool p)
{
    // every wave calls it: the block's barrier serves
    if (threadIdx.x == 0) wave_bits[threadIdx.y] = 0;
    __syncthreads();
    if (p) __atomic_fetch_or(&wave_bits[threadIdx.y], 1ull << threadIdx.x, __ATOMIC_SEQ_CST);
    __syncthreads();
    const unsigned long long r = wave_bits[threadIdx.y];
    __syncthreads();
    return r;
}
inline int __popcll(unsigned long long x) { return __builtin_popcountll(x); }
inline float __shfl_xor(float x, int) { return x; }       // only in kernels that are not run here
inline int __umul24(int a, int b) { return (a & 0xffffff) * (b & 0xffffff); }
inline unsigned __float_as_uint(float x) { unsigned u; memcpy(&u, &x, 4); return u; }
inline int __float_as_int(float x) { int u; memcpy(&u, &x, 4); return u; }
inline int atomicAdd(int *p, int v) { return __atomic_fetch_add(p, v, __ATOMIC_SEQ_CST); }
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_wave_barrier() ((void)0)
#define __builtin_amdgcn_s_setprio(x) ((void)0)
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_rcp(x) (1.0 / (x))
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_rsq(x) (1.0 / sqrt(x))
#define __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, x, y, z) (c)
"""

PROGRAM = r"""
#include "ww_router.hip"
#include <sys/mman.h>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <map>
#include <set>
#include <thread>
#include <vector>
using namespace ww;

// Sparse zeroed memory: pages exist once written.
template <typename T>
static T *sparse(size_t n)
{
    void *p = mmap(nullptr, n * sizeof(T), PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (p == MAP_FAILED) { printf("mmap of %zu bytes failed\n", n * sizeof(T)); exit(3); }
    return (T *)p;
}
static void block(const std::function<void()> &kernel)
{
    std::vector<std::thread> th;
    pthread_barrier_init(&block_barrier, nullptr, 256);
    for (int i = 0; i < 256; ++i)
        th.emplace_back([&, i] { threadIdx = dim3(i % 64, i / 64); kernel(); });
    for (auto &t : th) t.join();
    pthread_barrier_destroy(&block_barrier);
}

struct Box {
    Geom G;
    FaceBox F[3];
    float *u, *out, *flux[3];
    explicit Box(const int (&n)[3])
    {
        long N[3];
        for (int d = 0; d < 3; ++d) {
            G.n[d] = n[d]; G.act[d] = n[d] > 1; G.g[d] = G.act[d] ? 3 : 0; N[d] = n[d] + 2 * G.g[d];
            G.dl[d] = G.idl[d] = 1.0;
        }
        G.s[0] = 1; G.s[1] = N[0]; G.s[2] = N[0] * N[1]; G.sv = N[0] * N[1] * N[2];
        G.base = G.g[0] + G.g[1] * G.s[1] + G.g[2] * G.s[2];
        for (int d = 0; d < 3; ++d) {
            FaceBox &B = F[d];
            for (int e = 0; e < 3; ++e) {
                if (e == d) { B.lo[e] = 0; B.cnt[e] = n[e] + 1; }
                else if (G.act[e]) { B.lo[e] = -1; B.cnt[e] = n[e] + 2; }
                else { B.lo[e] = 0; B.cnt[e] = 1; }
            }
            B.s[0] = 1; B.s[1] = B.cnt[0]; B.s[2] = (long)B.cnt[0] * B.cnt[1];
            B.sc = B.s[2] * B.cnt[2];
            flux[d] = sparse<float>(NFC * B.sc);
        }
        u = sparse<float>(8 * G.sv);
        out = sparse<float>(8 * G.sv);
    }
    ~Box()
    {
        for (int d = 0; d < 3; ++d) munmap(flux[d], NFC * F[d].sc * 4);
        munmap(u, 8 * G.sv * 4);
        munmap(out, 8 * G.sv * 4);
    }
};
typedef std::vector<int> Pos;

static const float W[8] = { 1.0f, 0.2f, -0.3f, 0.1f, 0.5f, 0.4f, -0.25f, 2.5f };     // uniform state
// Its flux along d in grid components (rho, mx, my, mz, B_d+1, B_d+2, E).
static void flux_of(int d, double (&f)[7])
{
    const double r = W[0], g = 5.0 / 3.0;
    double v[3], b[3], vb = 0, b2 = 0, v2 = 0;
    for (int e = 0; e < 3; ++e) { v[e] = W[1 + e] / r; b[e] = W[4 + e]; vb += v[e] * b[e]; b2 += b[e] * b[e]; v2 += v[e] * v[e]; }
    const double p = (g - 1) * (W[7] - 0.5 * r * v2 - 0.5 * b2), pt = p + 0.5 * b2;
    f[0] = r * v[d];
    for (int e = 0; e < 3; ++e) f[1 + e] = r * v[d] * v[e] - b[d] * b[e] + (e == d ? pt : 0);
    const int t1 = (d + 1) % 3, t2 = (d + 2) % 3;
    f[4] = v[d] * b[t1] - v[t1] * b[d];
    f[5] = v[d] * b[t2] - v[t2] * b[d];
    f[6] = (W[7] + pt) * v[d] - b[d] * vb;
}
// y and z fluxes of the cells of the fused tail: a pattern over the faces.
static float pattern(int h, long i, long j, long k) { return 0.125f * (float)(1 + (h + 3 * i + 5 * j + 7 * k + 1000) % 61); }

#define FAIL(...) do { printf(__VA_ARGS__); printf("\n"); return 1; } while (0)

// One tile of the routed sweep of direction DIR, every third own face
// troubled by the stored mask, then the full fluxes of the queue and (FUSED)
// the cells left to the fix-up.
template <int DIR, bool FUSED, bool FAR>
static int tile_of(const char *name, const int (&n)[3], Box &B, long back)
{
    const FaceBox &F = B.F[DIR];
    long na, nb;
    routed_grid(DIR, F, na, nb);
    const long nt = na * nb, lb = nt - 1 - back, qcap = routed_queue_capacity(DIR, F);
    const bool seg = DIR == 0 && F.cnt[0] >= sw::XSEG_MIN;
    // the tile's faces
    std::vector<Pos> faces;
    std::set<long> own;
    auto add = [&](long i, long j, long k, bool o) {
        faces.push_back(Pos{ (int)i, (int)j, (int)k });
        if (o) own.insert(F.idx(i, j, k));
    };
    if (seg) {
        for (long g = lb * 255; g < F.sc && g < lb * 255 + 256; ++g) {
            const long row = g / F.cnt[0];
            add(g % F.cnt[0], F.lo[1] + row % F.cnt[1], F.lo[2] + row / F.cnt[1], g - lb * 255 < 255 || g == F.sc - 1);
        }
    } else if (DIR == 0) {
        const long ta = lb % na, tb = lb / na;
        for (long row = 4 * ta; row < 4 * ta + 4 && row < (long)F.cnt[1] * F.cnt[2]; ++row)
            for (long i = 64 * tb; i < 64 * tb + 64 && i < F.cnt[0]; ++i)
                add(i, F.lo[1] + row % F.cnt[1], F.lo[2] + row / F.cnt[1], true);
    } else {
        const int b = DIR == 1 ? 2 : 1;
        const long ta = lb / nb, tb = lb % nb, npos = (long)F.cnt[0] * F.cnt[b];
        for (long q = 32 * ta; q < 32 * ta + 32 && q < npos; ++q)
            for (long f = 8 * tb; f < 8 * tb + 8 && f < F.cnt[DIR]; ++f) {
                long p[3];
                p[0] = F.lo[0] + q % F.cnt[0];
                p[b] = F.lo[b] + q / F.cnt[0];
                p[DIR] = f;
                add(p[0], p[1], p[2], true);
            }
    }
    // their cells, uniform; the mask
    unsigned char *mask = sparse<unsigned char>(F.sc);
    unsigned long long *queue = sparse<unsigned long long>(64 * qcap);
    int nown = 0, ntr = 0;
    for (const Pos &p : faces) {
        for (int c = -3; c < 3; ++c) {
            long q[3] = { p[0], p[1], p[2] };
            q[DIR] += c;
            const long id = B.G.base + q[0] * B.G.s[0] + q[1] * B.G.s[1] + q[2] * B.G.s[2];
            for (int v = 0; v < 8; ++v) B.u[id + v * B.G.sv] = W[v];
        }
        const long fi = F.idx(p[0], p[1], p[2]);
        mask[fi] = fi % 3 == 0;
        if (own.count(fi)) { ++nown; ntr += mask[fi]; }
    }
    XFuse<float> xf{};
    xf.out = B.out;
    xf.fy = B.flux[1];
    xf.fz = B.flux[2];
    xf.by = B.F[1];
    xf.bz = B.F[2];
    xf.c = StageCoef{ 0, 0, 0.0, 0.0 };
    std::set<long> cells;
    if (FUSED)
        for (const Pos &p : faces) {
            const int i = p[0], j = p[1], k = p[2], hs[5] = { 0, 1, 2, 3, 6 };
            if (j < 0 || j >= n[1] || k < 0 || k >= n[2]) continue;
            for (int c = i - 1; c <= i; ++c) {
                if (c < 0 || c >= n[0]) continue;
                for (int h : hs)
                    for (int e = 0; e < 2; ++e) {
                        B.flux[1][h * B.F[1].sc + B.F[1].idx(c, j + e, k)] = pattern(h, c, j + e, k);
                        B.flux[2][h * B.F[2].sc + B.F[2].idx(c, j, k + e)] = pattern(h + 2, c, j, k + e);
                    }
            }
        }
    Phys P{ 5.0 / 3.0, 1e-6, 1.5 };
    const sw::XSegArgs XA = sw::xseg_args(F);
    const sw::YZArgs YA = DIR == 2 ? sw::yz_args<2, rt::YZ_PW, rt::YZ_FT>(F, sw::NXCD)
                                   : sw::yz_args<1, rt::YZ_PW, rt::YZ_FT>(F, sw::NXCD);
    const long per = (nt + sw::NXCD - 1) / sw::NXCD;
    if (DIR != 0 || seg) {
        gridDim = dim3((unsigned)(per * sw::NXCD));
        blockIdx = dim3((unsigned)(lb / per + sw::NXCD * (lb % per)), 0, 0);
    } else {
        gridDim = dim3((unsigned)na, (unsigned)nb);
        blockIdx = dim3((unsigned)(lb % na), (unsigned)(lb / na), 0);
    }
    int32_t *nsm = sparse<int32_t>(nt), qcount[64] = {};
    block([&] {
        rt::routed_sweep_kernel<DIR, FUSED, FAR>(B.u, B.flux[DIR], B.G, F, P, nullptr, 0.f, 0, nsm, queue, qcount, qcap, mask, 1,
                                            xf, XA, YA, (uint32_t)nt);
    });
    if (nsm[lb] != nown - ntr) FAIL("%s: %d smooth faces counted, %d", name, nsm[lb], nown - ntr);
    int nq = 0;
    for (int r = 0; r < 64; ++r) nq += qcount[r];
    if (nq != ntr) FAIL("%s: %d faces queued, %d", name, nq, ntr);
    double f[7];
    flux_of(DIR, f);
    auto check_faces = [&](bool troubled) {
        for (const Pos &p : faces) {
            const long fi = F.idx(p[0], p[1], p[2]);
            if (!own.count(fi) || (mask[fi] != 0) != troubled) continue;
            for (int c = 0; c < 7; ++c) {
                if (FUSED && !troubled && c != 4 && c != 5) continue;      // stored where a troubled face is next
                const float got = B.flux[DIR][c * F.sc + fi];
                if (!(fabs(got - f[c]) < 1e-5))
                    FAIL("%s: %s face %d %d %d component %d is %g, not %g", name, troubled ? "troubled" : "smooth", p[0], p[1],
                         p[2], c, got, f[c]);
            }
        }
        return 0;
    };
    if (check_faces(false)) return 1;
    // the queue's regions, one thread each
    one_thread = true;
    gridDim = dim3(1, 64);
    for (int r = 0; r < 64; ++r)
        for (int t = 0; t < 128 && t < qcount[r]; ++t) {
            blockIdx = dim3(0, r);
            threadIdx = dim3(t);
            rt::troubled_kernel<DIR, FAR>(B.u, B.flux[DIR], B.G, F, P, queue, qcount, qcap);
        }
    if (check_faces(true)) return 1;
    if (FUSED) {
        for (int r = 0; r < 64; ++r)
            for (int t = 0; t < 128 && t < qcount[r]; ++t) {
                blockIdx = dim3(0, r);
                threadIdx = dim3(t);
                rt::xfix_queue_kernel<FAR>(B.flux[0], B.G, F, xf, queue, qcount, qcap, mask);
            }
        int done = 0;
        for (const Pos &p : faces) {
            const int i = p[0], j = p[1], k = p[2], hs[5] = { 0, 1, 2, 3, 6 }, hv[5] = { 0, 1, 2, 3, 7 };
            // cells whose two x faces are both this tile's own
            if (i >= n[0] || j < 0 || j >= n[1] || k < 0 || k >= n[2]) continue;
            if (!own.count(F.idx(i, j, k)) || !own.count(F.idx(i + 1, j, k))) continue;
            const long id = B.G.base + i + j * B.G.s[1] + k * B.G.s[2];
            for (int h = 0; h < 5; ++h) {
                const double want = -(pattern(hs[h], i, j + 1, k) - pattern(hs[h], i, j, k)) -
                                    (pattern(hs[h] + 2, i, j, k + 1) - pattern(hs[h] + 2, i, j, k));
                const float got = B.out[id + hv[h] * B.G.sv];
                if (!(fabs(got - want) < 1e-4))
                    FAIL("%s: cell %d %d %d variable %d is %g, not %g", name, i, j, k, hv[h], got, want);
            }
            ++done;
        }
        if (!done) FAIL("%s: no cell checked", name);
    }
    one_thread = false;
    munmap(mask, F.sc);
    munmap(queue, 64 * qcap * 8);
    munmap(nsm, nt * 4);
    return 0;
}

// In the form that the library takes for the box.
template <int DIR, bool FUSED>
static int tile(const char *name, const int (&n)[3], long back)
{
    Box B(n);
    const double bytes = 4.0 * std::max(B.G.sv, B.F[DIR].sc);
    if (far_box(B.G, B.F[DIR])) return tile_of<DIR, FUSED, true>(name, n, B, back);
    if (bytes >= 4294967296.0) FAIL("%s: %.0f bytes a variable at 32-bit offsets", name, bytes);
    return tile_of<DIR, FUSED, false>(name, n, B, back);
}

int main(int argc, char **argv)
{
    const int cube[3] = { 1024, 1024, 1024 }, plane[3] = { 33000, 33000, 1 }, rows[3] = { 60, 4400, 4100 };
    const int near3[3] = { 1012, 1012, 1012 }, near2[3] = { 32750, 32750, 1 };
    int rc = 2;
    // (the cube's last 1026 x faces belong to the row beyond the box: a tile of interior rows)
    const long back = (long)(1025L * 1026 * 1.5) / 255;
    switch (atoi(argv[1])) {
    case 0: rc = tile<0, true>("cube, x with its cells", cube, back); break;
    case 1: rc = tile<1, false>("cube, y", cube, 0); break;
    case 2: rc = tile<2, false>("cube, z", cube, 0); break;
    case 3: rc = tile<0, false>("plane, x", plane, 0); break;
    case 4: rc = tile<1, false>("plane, y", plane, 0); break;
    case 5: rc = tile<0, false>("short rows, x", rows, 0); break;
    case 6: rc = tile<0, true>("under the limit, x with its cells", near3, (long)(1013L * 1014 * 1.5) / 255); break;
    case 7: rc = tile<2, false>("under the limit, z", near3, 0); break;
    case 8: rc = tile<1, false>("under the limit, plane, y", near2, 0); break;
    }
    if (rc == 0) printf("ok\n");
    fflush(stdout);
    return rc;
}
"""
NAMES = ["cube_x_fused", "cube_y", "cube_z", "plane_x", "plane_y", "short_rows_x", "near_x_fused", "near_z", "near_plane_y"]


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("routed")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(HIP_RUNTIME)
    for f in os.listdir(CSRC):
        if f.endswith(".h") or f == "ww_router.hip":
            text = open(os.path.join(CSRC, f)).read()
            # register constraints of the GPU
            text = re.sub(r"^\s*asm volatile\(.*\);$", "", text, flags=re.M)
            (d / f).write_text(text.replace('"../../include/wombat_weno.h"', '"wombat_weno.h"'))
    (d / "main.cpp").write_text(PROGRAM)
    exe = d / "routed"
    r = subprocess.run([CLANG, "-std=c++17", "-O1", "-w", "-pthread", "-I", str(d), "-I", os.path.join(ROOT, "include"),
                        str(d / "main.cpp"), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return str(exe)


@pytest.mark.parametrize("case", range(len(NAMES)), ids=NAMES)
def test_routed_kernels_beyond_32_bit_byte_offsets(program, case):
    r = subprocess.run([program, str(case)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
