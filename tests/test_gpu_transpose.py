"""A^T and B^T on every kind of tile of their kernel: edge tiles with both x-PML strips and plain ones,
rows around the ten outputs of a block, chunks of planes free of stretching and not, the largest
coefficient table, against the FP64 oracle.  Bars of the stencil kernels: 1e-12 in FP64, 1e-6 in
FP32 (relative L2)."""
import numpy as np
import pytest

from tests.test_gpu_parity import Pair, rel, to_np
from workloads import grf_velocity, random_table

pytestmark = pytest.mark.gpu

# total cells = physical + 2 n_pml
SHAPES = [
    ((52, 12, 36), 4),     # 60 x 20 x 44: the narrowest grid with edge tiles, 21 rows
    ((48, 10, 30), 4),     # 56 x 18 x 38 rounds to 56 x 20 x 40: no edge tiles
    ((116, 31, 20), 4),    # two inner tiles, 39 + 1 rows
    ((60, 8, 8), 16),      # every row and plane near the PML
    ((24, 16, 100), 20),   # strips wider than an edge tile, several chunks of planes
]


def _fit(shape, n_pml):
    """physical sizes whose totals are multiples of four"""
    return tuple(-(-(n + 2 * n_pml) // 4) * 4 - 2 * n_pml for n in shape)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape,n_pml", SHAPES)
def test_transposed_tiles(shape, n_pml, precision):
    p = Pair(grf_velocity(*_fit(shape, n_pml), seed=71, corr_len=6.0), n_pml, precision,
             tiling=dict(tile_tz=4, tile_split=0))
    for level in (0, 1):
        x = p.rand(level, 311, boundary_zero=False)   # boundary values have no rows
        for op in (5, 6):
            err = rel(to_np(p.g.apply(level, op, p.dev(x))), p.o.apply_t(level, op - 5, x.astype(np.complex128)))
            assert err <= p.tol(1e-12, 1e-6), (level, op, err)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_transposed_largest_table(precision):
    p = Pair(grf_velocity(56, 20, 24, seed=72, corr_len=6.0), 4, precision, table=random_table(73, K=128),
             tiling=dict(tile_tz=4, tile_split=0))
    x = p.rand(0, 312)
    for op in (5, 6):
        err = rel(to_np(p.g.apply(0, op, p.dev(x))), p.o.apply_t(0, op - 5, x.astype(np.complex128)))
        assert err <= p.tol(1e-12, 1e-6), (op, err)
