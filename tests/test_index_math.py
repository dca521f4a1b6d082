"""The integer index arithmetic of the tiled kernels (csrc/ww_index.h), built
for the CPU: division by a launch constant against the processor's, and the
x and y/z tiles' addresses against the plain index formulas, over boxes of
odd sizes, inactive axes and slabs."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1808_10633_amd", "csrc")

PROGRAM = r"""
#include "ww_index.h"
#include <cstdio>
#include <cstdlib>
using namespace ww;

#define CHECK(c) do { if (!(c)) { printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)

struct Box {                      // the state and a face box, as the library lays them out
    int n[3], act[3], g[3];
    long s[3], base, sv;
    int lo[3], cnt[3];
    long fs[3], fsc;
};

static Box box(const int (&n)[3], int d, int slab)
{
    Box B;
    long N[3];
    for (int e = 0; e < 3; ++e) {
        B.n[e] = n[e]; B.act[e] = n[e] > 1; B.g[e] = B.act[e] ? 3 : 0; N[e] = n[e] + 2 * B.g[e];
    }
    B.s[0] = 1; B.s[1] = N[0]; B.s[2] = N[0] * N[1]; B.sv = N[0] * N[1] * N[2];
    B.base = B.g[0] + B.g[1] * B.s[1] + B.g[2] * B.s[2];
    if (slab) { B.base += 2 * B.s[2]; B.n[2] = slab; }       // planes 2 .. 2 + slab of the box
    for (int e = 0; e < 3; ++e) {
        if (e == d) { B.lo[e] = 0; B.cnt[e] = B.n[e] + 1; }
        else if (B.act[e]) { B.lo[e] = -1; B.cnt[e] = B.n[e] + 2; }
        else { B.lo[e] = 0; B.cnt[e] = 1; }
    }
    B.fs[0] = 1; B.fs[1] = B.cnt[0]; B.fs[2] = (long)B.cnt[0] * B.cnt[1];
    B.fsc = B.fs[2] * B.cnt[2];
    return B;
}
static long sidx(const Box &B, long i, long j, long k) { return B.base + i * B.s[0] + j * B.s[1] + k * B.s[2]; }
static long fidx(const Box &B, long i, long j, long k)
{
    return (i - B.lo[0]) * B.fs[0] + (j - B.lo[1]) * B.fs[1] + (k - B.lo[2]) * B.fs[2];
}

static int divisions()
{
    unsigned long long x = 88172645463325252ull;
    auto rnd = [&] { x ^= x << 13; x ^= x >> 7; x ^= x << 17; return (uint32_t)(x >> 16); };
    for (int it = 0; it < 200000; ++it) {
        uint32_t d = it < 5000 ? it + 1 : rnd() >> (rnd() % 31);
        if (it % 97 == 0) d = 1u << (rnd() % 32);
        if (d < 1 || d > 0x80000000u) d = 1;
        const FastDiv f(d);
        const uint32_t q = 0xffffffffu / d;
        const uint32_t ns[10] = { 0, 1, d - 1, d, d + 1, q * d, q * d - 1, 0xffffffffu, rnd(), rnd() >> 8 };
        for (uint32_t n : ns) CHECK(f.div(n) == n / d);
    }
    return 0;
}

static int xtiles(const int (&n)[3], int slab)
{
    const Box B = box(n, 0, slab), Y = box(n, 1, slab), Z = box(n, 2, slab);
    const FastDiv nf(B.cnt[0]), n1(B.cnt[1]);
    const uint32_t jump = (uint32_t)(B.s[2] - (long)B.cnt[1] * B.s[1]);
    for (int stride = 255; stride <= 256; ++stride)
        for (long g0 = 0; g0 < B.fsc - (stride == 255); g0 += stride) {
            const XTile X = xtile((uint32_t)g0, (uint32_t)B.fsc, nf, n1);
            const long ub = B.base + (X.fa0 - 3) + (B.lo[1] + X.jj0) * B.s[1] + (B.lo[2] + X.kk0) * B.s[2];
            CHECK(X.nface == (B.fsc - g0 < 256 ? B.fsc - g0 : 256));
            CHECK(X.ncell <= 276);
            for (int t = 0; t < X.nface; ++t) {
                const long g = g0 + t, row = g / B.cnt[0], i = g % B.cnt[0];
                const long j = B.lo[1] + row % B.cnt[1], k = B.lo[2] + row / B.cnt[1];
                const int s = X.row_of(t);
                CHECK(s >= 0 && s <= 3 && X.face_x(t, s) == i);
                CHECK(B.lo[1] + X.jj(s) == j && B.lo[2] + X.kk(s) == k);
                CHECK(fidx(B, i, j, k) == g);
                for (int c = 0; c < 6; ++c) {
                    const int tc = X.cell_of(t, s) + c;
                    CHECK(tc < X.ncell);
                    const long id = ub + X.state_rel(tc, jump);
                    CHECK(id == sidx(B, i - 3 + c, j, k) && id >= 0 && id < B.sv);
                    const int sc = X.row_of_cell(tc);
                    CHECK(sc == s && tc + X.fa0 - 3 - sc * (X.nf + 5) == i - 3 + c);
                }
                if (B.act[0] && B.act[1] && B.act[2] && i < B.n[0] && j >= 0 && j < B.n[1] && k >= 0 && k < B.n[2]) {
                    const long x2 = X.nf + 1, w = s >= X.sw;
                    const long fy = 1 + (X.jj0 - 1) * x2 + X.kk0 * Y.fs[2], fz = 1 + X.jj0 * x2 + (X.kk0 - 1) * Z.fs[2];
                    CHECK(fy + i + (s - w) * x2 == fidx(Y, i, j, k));
                    CHECK(fy + x2 + i + (s - w) * x2 == fidx(Y, i, j + 1, k));
                    CHECK(fz + i + s * x2 == fidx(Z, i, j, k));
                    CHECK(fz + Z.fs[2] + i + s * x2 == fidx(Z, i, j, k + 1));
                }
            }
            for (int c = 0; c < X.ncell; ++c) {
                const long id = ub + X.state_rel(c, jump);
                CHECK(id >= 0 && id < B.sv);
            }
        }
    return 0;
}

static int yztiles(const int (&n)[3], int d, int pw, int ft, int slab)
{
    const Box B = box(n, d, slab);
    const int b = d == 1 ? 2 : 1;
    const uint32_t npos = (uint32_t)B.cnt[0] * B.cnt[b];
    const FastDiv na(B.cnt[0]);
    for (uint32_t p0 = 0; p0 < npos; p0 += pw)
        for (int f0 = 0; f0 < B.cnt[d]; f0 += ft) {
            const uint32_t b0 = na.div(p0), a0 = p0 - b0 * na.d;
            const long ub = B.base + B.lo[0] + (long)a0 + (long)(B.lo[b] + (int)b0) * B.s[b] + (long)(f0 - 3) * B.s[d];
            const long fb = (long)a0 + (long)b0 * B.fs[b] + (long)f0 * B.fs[d];
            const int np = (int)(npos - p0 < (uint32_t)pw ? npos - p0 : pw);
            const int rows = ft + 5 < B.n[d] + 6 - f0 ? ft + 5 : B.n[d] + 6 - f0;
            for (int pl = 0; pl < np; ++pl) {
                const int q = yz_rows_on(a0, pl, na, pw);
                long pos[3];
                pos[0] = B.lo[0] + (long)((p0 + pl) % B.cnt[0]);
                pos[b] = B.lo[b] + (long)((p0 + pl) / B.cnt[0]);
                CHECK(B.lo[0] + (int)(a0 + pl - q * na.d) == pos[0] && B.lo[b] + (int)b0 + q == pos[b]);
                for (int r = 0; r < rows; ++r) {
                    pos[d] = f0 - 3 + r;
                    const uint32_t e = (uint32_t)pl + (uint32_t)q * (uint32_t)(B.s[b] - na.d) + (uint32_t)r * (uint32_t)B.s[d];
                    const long id = ub + e;
                    CHECK(id == sidx(B, pos[0], pos[1], pos[2]) && id >= 0 && id < B.sv);
                }
                for (int r = 0; r < ft && f0 + r < B.cnt[d]; ++r) {
                    pos[d] = f0 + r;
                    CHECK(r + 5 < rows);          // the face's six cells are staged
                    const uint32_t e = (uint32_t)pl + (uint32_t)q * (uint32_t)(B.fs[b] - na.d) + (uint32_t)r * (uint32_t)B.fs[d];
                    CHECK(fb + e == fidx(B, pos[0], pos[1], pos[2]) && fb + e < B.fsc);
                }
            }
        }
    return 0;
}

int main()
{
    if (divisions()) return 1;
    const int xs[][3] = { { 85, 3, 3 }, { 86, 7, 5 }, { 97, 12, 10 }, { 255, 3, 4 }, { 256, 5, 3 }, { 300, 1, 1 },
                          { 128, 1, 6 }, { 131, 9, 1 }, { 1000, 3, 3 }, { 100, 24, 30 } };
    for (auto &n : xs) if (xtiles(n, 0) || (n[2] >= 10 && xtiles(n, 5))) { printf("x %d %d %d\n", n[0], n[1], n[2]); return 1; }
    const int ys[][3] = { { 3, 9, 4 }, { 5, 8, 1 }, { 16, 7, 16 }, { 30, 24, 13 }, { 33, 3, 3 }, { 64, 17, 10 }, { 100, 11, 12 },
                          { 61, 30, 9 }, { 3, 40, 3 }, { 1, 20, 11 }, { 1, 9, 1 }, { 1, 1, 14 }, { 129, 5, 1 } };
    for (auto &n : ys)
        for (int d = 1; d <= 2; ++d)
            for (int pw = 32; pw <= 64; pw *= 2)
                if (n[d] > 1 && (yztiles(n, d, pw, 8, 0) || (n[2] >= 9 && yztiles(n, d, pw, 8, 4)))) {
                    printf("dir %d pw %d: %d %d %d\n", d, pw, n[0], n[1], n[2]);
                    return 1;
                }
    printf("ok\n");
    return 0;
}
"""


def test_index_math(tmp_path):
    src = tmp_path / "index.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "index"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=undefined",
                           "-I", CSRC, str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
