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


# the chunks of the fused restriction hold every coarse plane at the depth that the rule takes
RESTRICT_PROGRAM = r"""
#include <cstdio>
#include "tiles.h"
using namespace helm;
int main() {
    for (int nx : {4, 8, 62, 64, 100, 352, 4096})
        for (int ny : {4, 9, 40, 352, 4096})
            for (int nz = 4; nz <= 400; nz += 2)
                for (int slots : {1, 3, 8}) {
                    const int d = restrict_depth(nx, ny, nz, slots);
                    const TileMap M = restrict_tiles(nx, ny, nz, d);
                    const int chunks = M.total_blocks / (M.nxi * M.nyt);
                    if (d < 1 || d > 32 || M.tz != d || chunks * d < nz / 2 || (chunks - 1) * d >= nz / 2 ||
                        30 * M.nxi < nx / 2 - 1 || kWavesY * M.nyt < ny + 1)
                        return std::printf("%d x %d x %d, %d slots: depth %d, %d chunks\n", nx, ny, nz, slots, d, chunks);
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


def test_restriction_chunks_hold_every_plane(tmp_path):
    _run(tmp_path, RESTRICT_PROGRAM)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape,n_pml", [((20, 12, 28), 4), ((56, 20, 60), 4), ((116, 12, 20), 6), ((16, 8, 92), 4)])
def test_restriction_at_its_own_depth(shape, n_pml, precision):
    """The fused residual + restriction where no depth is fixed, against the FP64 oracle
    (the bars of the stencil kernels)."""
    from tests.test_gpu_parity import Pair, rel, to_np
    from workloads import grf_velocity
    vel = grf_velocity(*shape, seed=81, corr_len=6.0)
    p = Pair(vel, n_pml, precision)
    for level in (0, 1):
        g, z = p.rand(level, 401), p.rand(level, 402)
        for op in (0, 1):
            ref = p.o.restrict(level, p.o.residual(level, op, g.astype(complex), z.astype(complex)))
            err = rel(to_np(p.g.residual_restrict(level, op, p.dev(g), p.dev(z))), ref)
            assert err <= p.tol(1e-12, 1e-6), (level, op, err)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape,n_pml", [((54, 10, 34), 5), ((58, 10, 14), 13), ((62, 6, 10), 29)])
def test_pml_as_wide_as_the_strip(shape, n_pml, precision):
    """Grids whose first column free of stretching is the first one of the inner tiles (strips of 6, 14 and 30
    columns): the fused Jacobi must not form D^-1 in place there, because the column before is stretched."""
    from tests.test_gpu_parity import Pair, rel, to_np
    from workloads import grf_velocity
    p = Pair(grf_velocity(*shape, seed=82, corr_len=6.0), n_pml, precision, tiling=dict(tile_tz=4, tile_split=0))
    g = p.rand(0, 403)
    for op in (0, 1):
        for sweeps in (2, 3):
            ref = p.o.jacobi(0, op, g.astype(complex), sweeps, 0.8)
            err = rel(to_np(p.g.jacobi(0, op, p.dev(g), sweeps, 0.8)), ref)
            assert err <= p.tol(1e-12, 1e-6), (op, sweeps, err)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("m_4h", [5, 6, 7, 8])
def test_vcycle_is_its_steps(m_4h, precision):
    """V^sigma_2h, which forms the bottom combination inside the prolongation and adds its last Jacobi onto the
    iterate, against the same cycle from the entry points of its steps.  The coefficients of the combination are the
    same; only a few sums round differently, so that long bases need no wider bar than the stencils."""
    import torch
    from tests.test_gpu_parity import Pair
    from workloads import grf_velocity
    p = Pair(grf_velocity(20, 12, 16, seed=83, corr_len=4.0), 4, precision, m_4h=m_4h)
    q = p.dev(p.rand(1, 404))
    w = p.g.opt.omega_2h
    y = p.g.jacobi(1, 1, q, 2, w)
    e = p.g.bottom(p.g.residual_restrict(1, 1, q, y))
    p.g.prolong_add(2, e, y)
    y = y + p.g.jacobi(1, 1, p.g.residual(1, 1, q, y), 2, w)
    err = float(torch.linalg.vector_norm(p.g.vcycle(q) - y) / torch.linalg.vector_norm(y))
    assert err <= p.tol(1e-12, 1e-6), err


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
