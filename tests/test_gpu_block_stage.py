"""The per-kernel path's stage in one kernel per block (two-ghost-layer
limiters): small grids split each block's planes over several workgroups, so
the same periodic content on one block and on many has to give the same bits
and the same number of repaired cells, for every split."""
import numpy as np
import pytest

from paper_2303_03026_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def amr():
    from paper_2303_03026_amd import amrvac
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    return amrvac


def tiled(ndim, nx, n, ng, limiter, flux):
    base = (n, n, n if ndim == 3 else 1)
    level, ijk = inputs.uniform_blocks(ndim, base)
    rng = np.random.Generator(np.random.PCG64(23))
    one = rng.uniform(-0.3, 0.3, size=(9,) + (nx,) * ndim)
    one[inputs.RHO] += 1.0
    one[inputs.PR] += 1.0
    # cells to repair: a corner, an edge's middle and one inside
    for at in ((0,) * ndim, (nx - 1,) + (nx // 2,) * (ndim - 1), (nx // 2,) * ndim):
        one[(inputs.PR,) + at] = 1e-3
    prim = np.broadcast_to(one, (len(level),) + one.shape).copy()
    return inputs.Workload("tiled", ndim, nx, base, (0.0,) * 3, (float(n),) * 3, (0,) * 3, (0,) * 3, level, ijk, prim,
                           ng=ng, limiter=limiter, flux=flux, small_pressure=0.01, fix_small_values=1)


def one_stage(amr, w):
    sim = amr.Simulation(w, path=amr.PATH_PLAIN)
    sim.cfl(0)
    before = sim.sync_flags(raise_on_error=False)[1]
    sim.euler_stage()
    fixed = sim.sync_flags(raise_on_error=False)[1] - before
    got = sim.cons(1)
    sim.close()
    return got, fixed


# edges: 16, 36, 100 and 256 columns are 1, 1, 2 and 4 waves a workgroup; the
# middle counts give splits that do not divide the planes
@pytest.mark.parametrize("ng", [2, 3])
@pytest.mark.parametrize("ndim,nx,counts,limiter,flux",
                         [(3, 4, (3, 7, 11), 0, 0), (3, 6, (2, 6, 11), 2, 1), (3, 10, (2, 5, 8), 1, 2),
                          (3, 16, (2, 5, 7), 0, 1), (2, 4, (2, 9), 1, 0), (2, 14, (2, 5), 0, 2)])
def test_the_split_changes_nothing(amr, ng, ndim, nx, counts, limiter, flux):
    if ng == 3 and nx < 6:
        pytest.skip("three ghost layers take blocks of at least 6 cells")
    ref, nref = one_stage(amr, tiled(ndim, nx, 1, ng, limiter, flux))
    assert nref > 0 and np.all(np.isfinite(ref))
    for n in counts:
        got, nfix = one_stage(amr, tiled(ndim, nx, n, ng, limiter, flux))
        assert nfix == nref * n ** ndim, n
        assert np.array_equal(got, np.broadcast_to(ref, got.shape)), n
