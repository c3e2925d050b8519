"""The fused stage of two ghost layers on small and one-block-thick grids:
each limiter and flux against the per-kernel path (whose arithmetic is the
same up to the order of the operations), and what it writes around the
interior: whole rows, so the ghost cells next to the x faces, and nothing
else."""
import numpy as np
import pytest

from paper_2303_03026_amd import inputs

pytestmark = pytest.mark.gpu

GRIDS = {"2d_1x3": (2, (1, 3, 1)), "2d_5x1": (2, (5, 1, 1)), "3d_1x1x1": (3, (1, 1, 1)), "3d_2x1x3": (3, (2, 1, 3))}


@pytest.fixture(scope="module")
def amr():
    from paper_2303_03026_amd import amrvac
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    return amrvac


def workload(name, limiter=0, flux=0):
    ndim, base = GRIDS[name]
    level, ijk = inputs.uniform_blocks(ndim, base)
    rng = np.random.Generator(np.random.PCG64(17))
    prim = rng.uniform(-0.3, 0.3, size=(len(level), 9) + (16,) * ndim)
    prim[:, inputs.RHO] += 1.0
    prim[:, inputs.PR] += 1.0
    prim[:, inputs.BX] += 0.5
    return inputs.Workload(name, ndim, 16, base, (0.0,) * 3, (1.0,) * 3, (0,) * 3, (0,) * 3, level, ijk, prim,
                           limiter=limiter, flux=flux)


@pytest.mark.parametrize("flux", [0, 1, 2], ids=["hll", "hlld", "hllc"])
@pytest.mark.parametrize("limiter", [0, 1, 2], ids=["vanleer", "koren", "cada3"])
@pytest.mark.parametrize("grid", sorted(GRIDS))
def test_one_stage_matches_the_per_kernel_path(amr, grid, limiter, flux):
    w = workload(grid, limiter, flux)
    out = []
    for path in (amr.PATH_PLAIN, amr.PATH_FUSED):
        sim = amr.Simulation(w, path=path)
        sim.cfl(0)
        sim.euler_stage()
        out.append(sim.cons(1))
        sim.close()
    # one stage adds dt L of order one to states of order one, each face flux
    # rounded some 50 times: 1e-13 is about 500 roundings
    assert np.max(np.abs(out[1] - out[0])) <= 1e-13 * np.max(np.abs(out[0]))


@pytest.mark.parametrize("grid", sorted(GRIDS))
def test_only_the_rows_of_the_interior_are_written(amr, grid):
    w = workload(grid)
    sim = amr.Simulation(w, path=amr.PATH_FUSED)
    sim.padded_view(1).fill_(float("nan"))
    sim.torch.cuda.synchronize()
    sim.cfl(0)
    sim.euler_stage()
    got = sim.padded(1)
    sim.close()
    x = np.arange(20)
    inside = (x >= 2) & (x < 18)
    rows = np.ones(got.shape[2:], dtype=bool)
    for ax in range(w.ndim - 1):  # every axis but x
        rows &= inside.reshape([-1 if k == ax else 1 for k in range(w.ndim)])
    assert np.all(np.isnan(got[:, :, ~rows]))
    interior = rows & inside
    assert np.all(np.isfinite(got[:, :, interior]))
