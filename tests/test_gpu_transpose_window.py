"""A^T and B^T with the widest window of table intervals that a level can stage: a velocity contrast of 24 and the
largest table, on the 4h level, whose window reaches the clamped interval.  In FP64 the window and the rows'
exchange then take more than 64 KB of LDS a block.  Against the FP64 oracle; bars of the stencil kernels: 1e-12 in
FP64, 1e-6 in FP32 (relative L2)."""
import numpy as np
import pytest

from tests.test_gpu_parity import H, Pair, rel, to_np
from workloads import grf_velocity, random_table

pytestmark = pytest.mark.gpu
K = 128


def staged_intervals(omega, level, cmin, cmax):
    """Intervals of the level's window: those of the velocity range and one more each side."""
    def interval(c):
        return min(int(min(omega * H * 2 ** level / (2 * np.pi * c), 0.4) * K / 0.4), K - 1)
    return min(interval(cmin) + 1, K - 1) - max(interval(cmax) - 1, 0) + 1


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_transposed_widest_window(precision):
    g = grf_velocity(56, 40, 48, seed=74, corr_len=6.0).astype(np.float64)
    vel = (500.0 * 24.0 ** ((g - g.min()) / (g.max() - g.min()))).astype(np.float32)
    p = Pair(vel, 4, precision, table=random_table(75, K=K), tiling=dict(tile_tz=4, tile_split=0))
    assert staged_intervals(p.omega, 2, float(vel.min()), float(vel.max())) > 102   # 49152 B + 160 B each: over 64 KB
    for level in (1, 2):
        x = p.rand(level, 312)
        for op in (5, 6):
            err = rel(to_np(p.g.apply(level, op, p.dev(x))), p.o.apply_t(level, op - 5, x.astype(np.complex128)))
            assert err <= p.tol(1e-12, 1e-6), (level, op, err)
