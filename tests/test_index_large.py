"""The tiles' index arithmetic (csrc/ww_index.h) on the largest boxes that fit
the card, built for the CPU with checked integer arithmetic: sampled tiles from
the first to the last, the places of their faces and cells against the plain
64-bit formulas, and the reach of the offsets that are held as 32-bit bytes."""
import subprocess

from test_index_math import CSRC, PROGRAM

MAIN = r"""
// Tile of `stride` faces number t; bytes: element size.
static int xsample(const Box &B, const Box &Y, const Box &Z, long t, int stride, long bytes)
{
    const FastDiv nf(B.cnt[0]), n1(B.cnt[1]);
    const uint32_t jump = (uint32_t)(B.s[2] - (long)B.cnt[1] * B.s[1]);
    const long g0 = t * stride;
    const XTile X = xtile((uint32_t)g0, (uint32_t)B.fsc, nf, n1);
    const long ub = B.base + (X.fa0 - 3) + (B.lo[1] + X.jj0) * B.s[1] + (B.lo[2] + X.kk0) * B.s[2];
    for (int f = 0; f < X.nface; ++f) {
        const long g = g0 + f, row = g / B.cnt[0], i = g % B.cnt[0];
        const long j = B.lo[1] + row % B.cnt[1], k = B.lo[2] + row / B.cnt[1];
        const int s = X.row_of(f);
        CHECK(X.face_x(f, s) == i && B.lo[1] + X.jj(s) == j && B.lo[2] + X.kk(s) == k);
        for (int c = 0; c < 6; ++c) {
            const uint32_t rel = X.state_rel(X.cell_of(f, s) + c, jump);
            CHECK(ub + rel == sidx(B, i - 3 + c, j, k));
            CHECK(rel * bytes < 4294967296L);
        }
        if (B.act[1] && B.act[2] && i < B.n[0] && j >= 0 && j < B.n[1] && k >= 0 && k < B.n[2]) {
            const long x2 = X.nf + 1, w = s >= X.sw, ry = i + (s - w) * x2, rz = i + s * x2;
            CHECK(s * x2 < 1 << 24);
            CHECK(1 + (X.jj0 - 1) * x2 + X.kk0 * Y.fs[2] + ry == fidx(Y, i, j, k));
            CHECK(1 + X.jj0 * x2 + (X.kk0 - 1) * Z.fs[2] + rz == fidx(Z, i, j, k));
            CHECK(ry * bytes < 4294967296L && rz * bytes < 4294967296L);
        }
    }
    return 0;
}

static int sample(const int (&n)[3], long bytes)
{
    const Box B = box(n, 0, 0), Y = box(n, 1, 0), Z = box(n, 2, 0);
    for (int stride = 255; stride <= 256; ++stride) {
        const long nt = (B.fsc - (stride == 255) + stride - 1) / stride;
        CHECK(nt < 1L << 24);
        for (long q = 0; q <= 4000; ++q) {
            const long ts[3] = { q, nt - 1 - q, (long)((double)q / 4001 * nt) };
            for (long t : ts)
                if (t >= 0 && t < nt && xsample(B, Y, Z, t, stride, bytes)) return 1;
        }
    }
    return 0;
}

int main()
{
    // FP32 planes: four states and two face boxes, 184 B a cell of 288 GB
    const int planes[][3] = { { 33000, 33000, 1 }, { 39000, 39000, 1 }, { 1 << 20, 1400, 1 }, { 1400, 1 << 20, 1 },
                              { 39000, 1, 39000 } };
    for (auto &n : planes) if (sample(n, 4)) { printf("%d %d %d\n", n[0], n[1], n[2]); return 1; }
    const int boxes[][3] = { { 1024, 1024, 1024 }, { 1 << 20, 11, 9 }, { 100, 3300, 3300 }, { 10000, 10000, 3 }, { 1 << 20, 1, 1 } };
    for (auto &n : boxes) if (sample(n, 8)) { printf("%d %d %d\n", n[0], n[1], n[2]); return 1; }
    printf("ok\n");
    return 0;
}
"""


def test_index_math_of_large_boxes(tmp_path):
    src = tmp_path / "index.cpp"
    src.write_text(PROGRAM[:PROGRAM.index("int main()")] + MAIN)
    exe = tmp_path / "index"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-w", "-fsanitize=undefined",
                           "-fno-sanitize-recover=undefined", "-I", CSRC, str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
