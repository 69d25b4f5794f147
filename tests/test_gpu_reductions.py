"""The reduction kernels and their small dense epilogues at the sizes where their branches change:
one block or several, every number of sums, short (register) and long (LDS) Gram solves, every
column of the Givens update and of the back substitution."""
import numpy as np
import pytest
import torch

from tests.test_gpu_parity import FP32_MAP_GATE, Pair, rel, to_np
from workloads import grf_velocity

pytestmark = pytest.mark.gpu

# a reduction block holds 1024 threads; one block up to 2048 elements, then one element a thread in up
# to 64 blocks, then four elements a thread in up to 256
SIZES = [1, 63, 65, 1023, 1024, 1025, 2048, 2049, 4097, 8193, 65535, 65537, 262145, 300001]


@pytest.mark.parametrize("dtype", [np.complex64, np.complex128])
def test_dots_of_every_count_and_size(dtype):
    """Against numpy in extended precision.  The sums are FP64 with at most
    4 + 6 + 16 + 26 + 64 + 8 additions in a chain (thread, wavefront, waves, a group's blocks,
    groups): under 128 units of 2^-53 of sum |v| |w|."""
    from paper_2608_22946_amd import helm
    rng = np.random.default_rng(5)
    for i, n in enumerate(SIZES):
        for k in range(13):
            if k not in (0, 12) and (k + i) % 3:   # a third of the counts at each size, and both ends
                continue
            V = (rng.standard_normal((k, n)) + 1j * rng.standard_normal((k, n))).astype(dtype)
            w = (rng.standard_normal(n) + 1j * rng.standard_normal(n)).astype(dtype)
            out = helm.vec_dots_static([torch.from_numpy(v).cuda() for v in V], torch.from_numpy(w).cuda())
            o = out.cpu().numpy()
            got = o[0::2] + 1j * o[1::2]
            Vl, wl = V.astype(np.clongdouble), w.astype(np.clongdouble)
            for j in range(k + 1):
                a = Vl[j] if j < k else wl
                ref = np.sum(np.conj(a) * wl)
                assert abs(got[j] - ref) <= 128 * 2.0 ** -53 * float(np.sum(np.abs(a) * np.abs(wl))), (n, k, j)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("m_4h", [1, 2, 3, 4, 5, 8])
def test_bottom_basis_lengths(m_4h, precision):
    """C_4h by its Gram solve: bases of up to five vectors in registers, longer ones in LDS, on a
    4h level of one reduction block (7 x 5 x 6 cells) against the oracle.  Eight monomial vectors
    square a condition number that five do not: their FP64 bar is that of FP32."""
    p = Pair(grf_velocity(20, 12, 16, seed=23, corr_len=4.0), 4, precision, m_4h=m_4h)
    q = p.rand(2, 231)
    err = rel(to_np(p.g.bottom(p.dev(q))), p.o.bottom(q.astype(complex)))
    assert err <= p.tol(1e-9 if m_4h <= 5 else FP32_MAP_GATE, FP32_MAP_GATE if m_4h <= 5 else 1e-2), err
    z = p.g.bottom(p.dev(np.zeros_like(q)))   # no pivot survives
    assert torch.count_nonzero(z) == 0


@pytest.mark.parametrize("m_2h", [1, 2, 7, 12])
def test_coarse_solve_cycle_lengths(m_2h):
    """K_2h with cycles of 1 to 12 columns (the Givens chain and the back substitution of each)."""
    p = Pair(grf_velocity(20, 12, 16, seed=24, corr_len=4.0), 4, "fp64", m_2h=m_2h, c_2h=2)
    r = p.rand(1, 232)
    err = rel(to_np(p.g.coarse_solve(p.dev(r))), p.o.k2h(r.astype(complex)))
    assert err <= 1e-8, err


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("m_4h", [1, 2, 3, 5, 8])
def test_vcycle_basis_lengths(m_4h, precision):
    """V^sigma_2h, whose prolongation forms the bottom solver's combination itself, for each number of
    basis vectors; the bars are those of the bottom solver."""
    p = Pair(grf_velocity(20, 12, 16, seed=25, corr_len=4.0), 4, precision, m_4h=m_4h)
    q = p.rand(1, 233)
    err = rel(to_np(p.g.vcycle(p.dev(q))), p.o.vcycle(q.astype(complex)))
    assert err <= p.tol(1e-9 if m_4h <= 5 else FP32_MAP_GATE, FP32_MAP_GATE if m_4h <= 5 else 1e-2), err
