"""HLLD faces whose star states are degenerate (no tangential field, the fast
speed equal to the Alfven speed) beside ordinary ones: an ordinary face must
not depend on which others share its wave.  The per-kernel path lays faces out
in other waves than the fused stage, whose five-cell arithmetic is the same
operation by operation."""
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


def lines(ndim, axis, limiter):
    """Lines along the axis: a random fifth of them uniform with a strong
    field along it and none across, the others random."""
    base = (2, 3, 2 if ndim == 3 else 1)
    level, ijk = inputs.uniform_blocks(ndim, base)
    rng = np.random.Generator(np.random.PCG64(43))
    box = tuple(16 * b for b in base[:ndim][::-1])
    prim = rng.uniform(-0.3, 0.3, size=(9,) + box)
    prim[inputs.RHO] += 1.0
    prim[inputs.PR] += 1.0
    prim[inputs.BX:inputs.BX + 3] += 0.5
    along = ndim - 1 - axis
    pick = rng.random(box[:along] + (1,) + box[along + 1:]) < 0.2
    still = np.zeros(9)
    still[inputs.RHO], still[inputs.PR], still[inputs.BX + axis] = 1.0, 0.25, 2.0
    prim = np.where(pick, still.reshape((9,) + (1,) * ndim), prim)
    return inputs.Workload("lines", ndim, 16, base, (0.0,) * 3, tuple(float(b) for b in base), (0,) * 3, (0,) * 3,
                           level, ijk, inputs.global_to_blocks(prim, ndim, 16).swapaxes(0, 1), limiter=limiter,
                           flux=1, ng=3)


@pytest.mark.parametrize("limiter", [3, 5], ids=["weno5", "mp5"])
@pytest.mark.parametrize("ndim,axis", [(2, 0), (2, 1), (3, 0), (3, 1), (3, 2)])
def test_both_paths_give_the_same_bits(amr, ndim, axis, limiter):
    w = lines(ndim, axis, limiter)
    out = []
    for path in (amr.PATH_PLAIN, amr.PATH_FUSED):
        sim = amr.Simulation(w, path=path)
        sim.cfl(0)
        sim.euler_stage()
        out.append(sim.cons(1))
        sim.close()
    assert np.all(np.isfinite(out[0]))
    assert np.array_equal(out[0], out[1])
