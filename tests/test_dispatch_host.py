"""The launchers' rules (which kernel, which addressing, which columns), compiled
for the host alone and asked for boxes of every kind; nothing runs on a GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FP64, FP32, MIXED, FP16 = range(4)
CG, SC_MP, SC_MC = range(3)
PERIODIC, WALLS = (0, 0, 0), (1, 1, 2)

PROGRAM = r"""
#include <cstdio>
#include "fused.hpp"
using namespace mclbm;
// in: lattice model precision nx ny nz bc0 bc1 bc2 conserve
int main()
{
    int lattice, model, precision;
    KParams P{};
    while (std::scanf("%d %d %d %d %d %d %d %d %d %d", &lattice, &model, &precision, &P.nx, &P.ny, &P.nz, &P.bc[0],
                      &P.bc[1], &P.bc[2], &P.conserve) == 10) {
        P.N = (long long)P.nx * P.ny * P.nz;
        const bool one = lattice == 0 ? rows_preferred(P) : !d3_prefers_two_pass(P, precision, model);
        FusedShape sh{};
        if (lattice == 1 && !fused_shape(P, sh, precision)) fused_odd_shape(P, sh, precision);
        std::printf("%d %d %d %d %d\n", (int)column_pointers(P, lattice == 0, precision, model), (int)one, sh.tx, sh.ty,
                    sh.tz);
    }
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    """Rows of (lattice, model, precision, (nx, ny, nz), bc, conserve) to rows of answers."""
    if not shutil.which("hipcc"):
        pytest.skip("needs hipcc")
    d = tmp_path_factory.mktemp("dispatch")
    src, exe = d / "rules.hip", d / "rules"
    src.write_text(PROGRAM)
    subprocess.run(["hipcc", "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2110_05197_amd", "csrc"),
                    "-o", str(exe), str(src)], check=True, capture_output=True, text=True)

    def run(rows):
        text = "".join("%d %d %d %d %d %d %d %d %d %d\n" % (l, m, p, *box, *bc, c) for l, m, p, box, bc, c in rows)
        out = subprocess.run([str(exe)], input=text, check=True, capture_output=True, text=True).stdout
        return [[float(v) for v in line.split()] for line in out.splitlines()]
    return run


def test_addressing_of_the_one_pass_kernels(ask):
    """Buffer accesses unless the box is one of those that pointers serve better."""
    near = [(1, CG, FP32, (234, 80, 119), PERIODIC, 0), (1, CG, FP32, (141, 72, 164), PERIODIC, 0),
            (1, CG, FP32, (57, 192, 239), WALLS, 0), (1, SC_MC, FP32, (110, 136, 217), WALLS, 0),
            (1, SC_MC, MIXED, (113, 48, 155), PERIODIC, 0), (1, CG, MIXED, (234, 80, 120), WALLS, 1),
            (1, CG, MIXED, (96, 96, 384), WALLS, 0), (1, CG, FP64, (223, 224, 183), WALLS, 0),
            (1, CG, FP64, (208, 336, 331), WALLS, 0), (1, CG, FP64, (192, 192, 192), PERIODIC, 0),
            (1, SC_MP, FP64, (256, 256, 256), PERIODIC, 0), (1, CG, FP16, (160, 160, 160), PERIODIC, 0),
            (1, CG, FP32, (96, 40, 77), WALLS, 0), (1, SC_MP, FP32, (96, 208, 259), WALLS, 0),
            (1, SC_MP, FP32, (96, 96, 96), WALLS, 0), (1, CG, FP32, (96, 96, 96), PERIODIC, 0),
            (0, CG, MIXED, (1900, 1100, 1), PERIODIC, 0), (0, SC_MP, FP32, (1900, 1100, 1), PERIODIC, 0),
            (0, CG, FP64, (1900, 1100, 1), (0, 1, 0), 0), (0, SC_MC, MIXED, (1900, 1100, 1), (0, 1, 0), 0)]
    far = [(1, CG, FP32, (178, 192, 140), PERIODIC, 0), (1, CG, FP16, (96, 72, 90), (0, 1, 0), 0), (1, SC_MC, FP16, (58, 112, 115), WALLS, 0),
           (1, SC_MP, FP16, (200, 120, 90), WALLS, 0), (1, SC_MC, FP16, (96, 192, 210), PERIODIC, 0),
           (1, CG, MIXED, (213, 160, 169), PERIODIC, 1), (1, CG, MIXED, (213, 136, 197), PERIODIC, 0), (1, CG, FP64, (256, 256, 256), PERIODIC, 0),
           (1, SC_MC, FP64, (307, 368, 130), WALLS, 0), (1, CG, FP64, (256, 336, 233), WALLS, 0),
           (1, CG, FP32, (96, 96, 384), WALLS, 0), (1, SC_MC, FP32, (288, 72, 127), (1, 1, 1), 0),
           (1, SC_MP, FP32, (96, 96, 96), PERIODIC, 0), (1, SC_MC, FP32, (96, 136, 201), PERIODIC, 0),
           (0, CG, MIXED, (1900, 1100, 1), (0, 1, 0), 0), (0, CG, FP32, (4096, 4096, 1), PERIODIC, 0),
           (0, CG, FP16, (1900, 1100, 1), (0, 1, 0), 0)]
    answers = [int(a[0]) for a in ask(near + far)]
    assert answers == [0] * len(near) + [1] * len(far)


def test_automatic_choice_of_the_kernel(ask):
    """One pass or two, where both exist, on boxes timed with both kernels: (box,
    one-pass us, two-pass us) on either side of the lines."""
    one = [((1, CG, FP32, (128, 128, 128), PERIODIC, 0), 133, 195), ((1, CG, FP64, (176, 176, 176), PERIODIC, 0), 950, 1100),
           ((1, CG, MIXED, (224, 80, 130), PERIODIC, 0), 224, 264), ((1, SC_MC, FP64, (192, 192, 192), PERIODIC, 0), 1, 2),
           ((1, CG, FP32, (64, 16, 8), PERIODIC, 0), 8, 8), ((0, CG, FP64, (521, 1709, 1), PERIODIC, 0), 69, 77),
           ((0, SC_MC, FP32, (195417, 22, 1), PERIODIC, 0), 68, 100)]
    two = [((1, SC_MP, FP16, (194, 136, 98), PERIODIC, 0), 111, 59), ((1, CG, MIXED, (32, 244, 53), (0, 1, 0), 1), 94, 42),
           ((1, CG, FP32, (32, 172, 101), PERIODIC, 1), 92, 46), ((1, SC_MP, MIXED, (239, 84, 93), WALLS, 0), 128, 85),
           ((1, SC_MP, FP64, (68, 64, 49), PERIODIC, 0), 31, 20), ((1, SC_MC, FP16, (192, 140, 50), WALLS, 0), 115, 67),
           ((1, CG, FP64, (27, 12, 199), PERIODIC, 0), 28, 16), ((1, SC_MP, FP32, (90, 176, 97), PERIODIC, 0), 91, 61),
           ((0, CG, MIXED, (5, 121446, 1), (0, 1, 0), 0), 1029, 32), ((0, CG, FP32, (17, 175932, 1), PERIODIC, 0), 611, 155)]
    answers = [int(a[1]) for a in ask([c[0] for c in one + two])]
    assert answers == [1] * len(one) + [0] * len(two)


def test_march_lengths_are_the_best_of_all(ask):
    """The planes of a chunk, found in about sqrt(nz) steps, against every number
    of chunks: the least rounds * (planes + 3) of 256 blocks a round, fewest chunks
    on a tie, where that is a tenth less than one round's."""
    import random
    import time
    rng = random.Random(5)
    rows = []
    for _ in range(1500):
        box = (rng.randint(2, 500), rng.randint(2, 500), rng.choice([rng.randint(2, 60), rng.randint(60, 3000)]))
        rows.append((1, rng.randint(0, 2), rng.randint(0, 3), box, PERIODIC, 0))
    searched = 0
    for (_, _, prec, (nx, ny, nz), _, _), (_, _, tx, ty, tz) in zip(rows, ask(rows)):
        columns = -(-nx // int(tx)) * -(-ny // int(ty))
        plain = -(-nz // max(1, 256 // columns))
        blocks = columns * -(-nz // plain)
        best, want = plain + 3, plain
        if blocks < (200 if prec == FP32 else 256) and columns * nz >= 256:
            for chunks in range(1, nz + 1):
                t = -(-nz // chunks)
                cost = -(-columns * -(-nz // t) // 256) * (t + 3)
                if cost < best:
                    best, want = cost, t
            if prec != FP16 and 10 * best > 9 * (plain + 3):
                want = plain
        searched += want != plain
        assert tz == want, (nx, ny, nz, prec, tz, want)
    assert searched > 100
    start = time.perf_counter()
    ask([(1, CG, FP32, (2, 4, 260000000), PERIODIC, 0)] * 20)   # a search over nz took seconds a box
    assert time.perf_counter() - start < 2
