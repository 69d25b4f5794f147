"""The tiling of the stencil launches, on the host: a fused norm writes one partial sum a block, so the
bound that sizes the partials has to hold for every tiling that a launch may take."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# make_tiles' blocks against stencil_blocks at the smallest depth (the size of the partials): every even
# width to 900 and the widest, thin and ordinary numbers of rows, every width of the PML
PROGRAM = r"""
#include <cstdio>
#include "tiles.h"
using namespace helm;

static long long tried, strips[31];
static int check(int nx, int ny, int nz, int lox, int tz, int tz_bound) {
    const TileMap M = make_tiles(nx, ny, nz, lox, nx - lox, tz);
    ++tried;
    ++strips[M.strip];
    const int bound = stencil_blocks(nx, ny, nz, tz_bound);
    if (M.total_blocks <= bound) return 0;
    std::printf("%d x %d x %d lox %d tz %d: %d blocks, bound %d\n", nx, ny, nz, lox, tz, M.total_blocks, bound);
    return 1;
}

int main() {
    int bad = 0;
    // total grids whose fused norm has more blocks than the partials' least size of 98304
    bad += check(4096, 20, 744, 5, 2, 2);
    bad += check(2048, 32, 1024, 5, 2, 2);
    bad += check(1024, 20, 1600, 5, 2, 2);
    bad += check(1000, 16, 2048, 5, 2, 2);
    bad += check(620, 16, 4096, 5, 2, 2);
    bad += check(340, 16, 3932, 3, 2, 2);
    bad += check(4096, 16, 4096, 5, 3, 2);
    for (int nx = 2; nx <= 4096; nx = nx < 900 ? nx + 2 : nx < 4000 ? nx + 310 : nx + 4)
        for (int ny = 2; ny <= 4096; ny = ny < 140 ? ny + 1 : ny * 2)
            for (int lox = 1; lox <= 32 && 2 * lox <= nx; ++lox)
                for (int tz : {2, 3, 16})
                    if ((bad += check(nx, ny, 61, lox, tz, 2)) > 20) return 1;
    std::printf("%lld tilings: no strip %lld, 30 columns %lld, 14 %lld, 6 %lld\n", tried, strips[0], strips[30],
                strips[14], strips[6]);
    return bad || !strips[0] || !strips[30] || !strips[14] || !strips[6];
}
"""


def test_partials_hold_every_tiling(tmp_path):
    _run(tmp_path, PROGRAM)


# every row and plane that a march of any tiling forms: the rows and weight nodes it reads with exist
ROWS_PROGRAM = r"""
#include <cstdio>
#include "tiles.h"
using namespace helm;
int main() {
    for (int strip : {0, 30, 14, 6})
        for (int ny = 2; ny <= 200; ++ny) {
            const TileMap M = tile_counts(200, ny, ny, strip, 4);
            // a wavefront's rows y .. y + rows - 1 (edge tiles), y (inner tiles)
            for (int y = 0; y < (strip ? M.neb * M.rows : M.nyt) * kWavesY; y += M.rows) {
                if (y > ny) continue;
                for (int r = 0; r < M.rows; ++r) {
                    const MarchRows m = march_rows(y + r, ny);
                    for (int a : {m.m, m.c, m.p})
                        if (a < 0 || a > ny) return std::printf("strip %d ny %d row %d: reads row %d\n", strip, ny, y + r, a);
                }
            }
        }
    return 0;
}
"""


def _run(tmp_path, program):
    src, exe = tmp_path / "tiles.cpp", tmp_path / "tiles"
    src.write_text(program)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2608_22946_amd", "csrc"),
                           str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout


def test_marches_read_inside_the_grid(tmp_path):
    _run(tmp_path, ROWS_PROGRAM)


@pytest.mark.gpu
def test_norm_of_more_blocks_than_the_least_partials():
    """620 x 16 x 3932 cells at two planes a wavefront: 102284 blocks, where the partials' least size is 98304.
    The norm that one preconditioner call reports is that of the residual of its result (both norms are of
    FP64 residuals that differ by rounding)."""
    import torch
    from paper_2608_22946_amd import helm
    vel = torch.full((3929, 13, 617), 2000.0)
    H = helm.Hierarchy(vel, 10.0, 2 * 3.141592653589793 * 2000.0 / 60.0, 2, precision="fp64", tile_tz=2,
                       tile_split=0, max_outer=1)
    f = H.zeros(0)
    f[1900, 8, 300] = 1e-3
    u, v, its, relres, rc = H.solve_checkpoint(f, 1e-12)
    assert (its, rc) == (1, helm.HELM_NOT_CONVERGED)
    b = H.apply(0, helm.OP_Q, f)
    r = H.residual(0, helm.OP_A, b, v)
    assert abs(float(torch.linalg.vector_norm(r) / torch.linalg.vector_norm(b)) - relres) <= 1e-10 * max(1.0, relres)
