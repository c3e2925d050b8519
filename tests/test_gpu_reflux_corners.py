"""Coarse cells next to finer leaves across faces of two and three directions:
one coarse block in a periodic box of finer ones.  With every such face's flux
corrected, a stage keeps the box's totals."""
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


def one_coarse(ndim, nx, limiter):
    n = 3
    level, ijk = [], []
    for k in range(n if ndim == 3 else 1):
        for j in range(n):
            for i in range(n):
                if (i, j) == (1, 1) and (ndim == 2 or k == 1):
                    level.append(1)
                    ijk.append((i, j, k))
                    continue
                for c in range(2 ** ndim):
                    level.append(2)
                    ijk.append((2 * i + (c & 1), 2 * j + (c >> 1 & 1), 2 * k + (c >> 2) if ndim == 3 else 0))
    level, ijk = np.array(level, np.int32), np.array(ijk, np.int32)
    rng = np.random.Generator(np.random.PCG64(29))
    prim = rng.uniform(-0.3, 0.3, size=(len(level), 9) + (nx,) * ndim)
    prim[:, inputs.RHO] += 1.0
    prim[:, inputs.PR] += 1.0
    return inputs.Workload("one_coarse", ndim, nx, (n, n, n if ndim == 3 else 1), (0.0,) * 3, (1.0,) * 3, (0,) * 3,
                           (0,) * 3, level, ijk, prim, limiter=limiter, ng=3 if limiter >= 3 else 2)


@pytest.mark.parametrize("ndim", [2, 3])
@pytest.mark.parametrize("path,nx,limiter", [("plain", 4, 0), ("plain", 10, 1), ("fused", 16, 0), ("fused", 16, 3)])
def test_totals_are_kept(amr, ndim, path, nx, limiter):
    w = one_coarse(ndim, nx, limiter)
    sim = amr.Simulation(w, path=amr.PATH_PLAIN if path == "plain" else amr.PATH_FUSED)
    sim.cfl(0)
    sim.euler_stage()
    before, after = sim.cons(0), sim.cons(1)
    sim.close()
    vol = 0.5 ** (ndim * (w.level.astype(float) - 1))
    total = lambda u: np.einsum("b,bqc->q", vol, u.reshape(len(vol), 9, -1))  # noqa: E731
    size = total(np.abs(before))
    # roundings: some 50 per face flux and update, each 1.1e-16 of values of
    # the cells' size; a cell left out of a correction changes a total by
    # about 1e-2 of a cell, 1e-6 of the largest box here
    assert np.max(np.abs(after - before)) > 1e-3
    keep = [q for q in range(9) if q != inputs.PSI]  # psi decays
    assert np.all(np.abs(total(after) - total(before))[keep] <= 1e-13 * np.max(size))
