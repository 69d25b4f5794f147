"""The level stencils on every kind of tile: edge tiles with strips of 30, 14 and 6 columns (one, two
and four rows a wavefront) and none, ragged last groups of rows and chunks of planes, chunks free of
stretching (inner tiles) and not, one launch or two, against the FP64 oracle.

Bars of the stencil kernels: 1e-12 in FP64, 1e-6 in FP32 (relative L2)."""
import numpy as np
import pytest
import torch

from tests.test_gpu_parity import H, Pair, rel, to_np
from workloads import grf_velocity, point_source

pytestmark = pytest.mark.gpu

# total cells = physical + 2 n_pml, all divisible by four; level 1 has half of both
SHAPES = [
    ((56, 12, 36), 4),    # 64 x 20 x 44: strips of 6 columns, four rows a wavefront
    ((76, 24, 28), 4),    # 84 x 32 x 36: 14 columns, two rows
    ((88, 8, 20), 16),    # 120 x 40 x 52: 30 columns, one row
    ((24, 20, 12), 12),   # 48 x 44 x 36: no strip fits
    ((180, 16, 60), 2),   # 184 x 20 x 64: several inner tiles
]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("tiling", [dict(tile_tz=4, tile_split=0), dict(tile_tz=16, tile_split=1)])
@pytest.mark.parametrize("shape,n_pml", SHAPES)
def test_stencils_on_every_tile_kind(shape, n_pml, tiling, precision):
    p = Pair(grf_velocity(*shape, seed=61, corr_len=6.0), n_pml, precision, tiling=tiling)
    bar = p.tol(1e-12, 1e-6)
    for level in (0, 1):
        x, g = p.rand(level, 301, boundary_zero=False), p.rand(level, 302)
        z = p.rand(level, 301)
        for op in (0, 1):
            err = rel(to_np(p.g.apply(level, op, p.dev(x))), p.o.apply(level, op, x.astype(complex)))
            assert err <= bar, ("apply", level, op, err)
            err = rel(to_np(p.g.residual(level, op, p.dev(g), p.dev(z))),
                      p.o.residual(level, op, g.astype(complex), z.astype(complex)))
            assert err <= bar, ("residual", level, op, err)
            err = rel(to_np(p.g.jacobi(level, op, p.dev(g), 2, 0.3)), p.o.jacobi(level, op, g.astype(complex), 2, 0.3))
            assert err <= bar, ("jacobi", level, op, err)
            ref = p.o.restrict(level, p.o.residual(level, op, g.astype(complex), z.astype(complex)))
            err = rel(to_np(p.g.residual_restrict(level, op, p.dev(g), p.dev(z))), ref)
            assert err <= bar, ("residual_restrict", level, op, err)


@pytest.mark.parametrize("shape,n_pml", SHAPES[:3])
def test_fused_norm_residual(shape, n_pml):
    """The outer residual written together with its norm, in FP64: the solves of all tilings agree
    with each other and with the residual of the solution that they return."""
    vel = grf_velocity(*shape, seed=62, corr_len=6.0)
    N = tuple(n + 2 * n_pml for n in shape)
    f = point_source(N, tuple(n // 2 - 1 for n in N), H)
    its = set()
    for tiling in (dict(tile_tz=4, tile_split=0), dict(tile_tz=16, tile_split=1)):
        p = Pair(vel, n_pml, "fp64", tiling=tiling)
        u, v, k, relres, rc = p.g.solve_checkpoint(p.dev(f), 1e-8)
        b = p.g.apply(0, 2, p.dev(f))
        r = p.g.residual(0, 0, b, v)
        assert rc == 0 and relres <= 1e-8
        # both are norms of FP64 residuals that differ by rounding: at most about
        # 2^-52 |A| |A^-1|, and cond(A) is under 4e5 on these grids
        assert abs(float(torch.linalg.vector_norm(r) / torch.linalg.vector_norm(b)) - relres) <= 1e-10
        its.add(k)
    assert len(its) == 1, its
