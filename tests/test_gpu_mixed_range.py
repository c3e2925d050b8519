"""FP32 face arithmetic over scales: multiplying density, pressure and B^2 by
one number leaves every speed as it is, so a stage's result only scales, also
where the square of a pressure is outside the range of FP32."""
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


def one_stage(amr, limiter, flux, scale, density=1.0):
    level, ijk = inputs.uniform_blocks(3, (2, 1, 3))
    rng = np.random.Generator(np.random.PCG64(37))
    prim = rng.uniform(-0.5, 0.5, size=(len(level), 9, 16, 16, 16))
    prim[:, inputs.RHO] += 1.0
    prim[:, inputs.PR] += 10.0
    prim[:, inputs.BX:] *= 4.0
    prim[:, inputs.PSI] *= 0.1
    prim[:, inputs.RHO] *= density
    prim[:, [inputs.RHO, inputs.PR]] *= scale
    prim[:, inputs.BX:] *= np.sqrt(scale)
    w = inputs.Workload("scaled", 3, 16, (2, 1, 3), (0.0,) * 3, (1.0,) * 3, (0,) * 3, (0,) * 3, level, ijk, prim,
                        limiter=limiter, flux=flux, ng=3 if limiter >= 3 else 2)
    sim = amr.Simulation(w, path=amr.PATH_FUSED, precision=amr.FP32_MIXED)
    sim.cfl(0)
    sim.euler_stage()
    got = sim.cons(1)
    sim.close()
    got[:, :5] /= scale
    got[:, 5:] /= np.sqrt(scale)
    return got


# van Leer's slope is a product of two differences, which bounds its range
# closer: 2^60, with pressures of 2^64.  So does HLLD's pressure between the
# fast waves, a product of rho c and p: hot gas, whose c is 2^9
@pytest.mark.parametrize("limiter,flux,density,exponents",
                         [(0, 0, 1.0, (60,)), (0, 1, 2.0 ** -14, (60,)), (0, 2, 1.0, (60,)),
                          (2, 0, 1.0, (-84, 84)), (2, 1, 2.0 ** -14, (60,)), (2, 2, 1.0, (-84, 84)),
                          (5, 0, 1.0, (-84, 84)), (5, 1, 2.0 ** -14, (60,)), (5, 2, 1.0, (-84, 84))])
def test_a_stage_scales(amr, limiter, flux, density, exponents):
    want = one_stage(amr, limiter, flux, 1.0, density)
    assert np.all(np.isfinite(want))
    for e in exponents:  # even, so that B scales by a power of two
        got = one_stage(amr, limiter, flux, 2.0 ** e, density)
        for q in range(9):
            # some 50 roundings of FP32 per flux
            assert np.max(np.abs(got[:, q] - want[:, q])) <= 50 * 2.0 ** -24 * np.max(np.abs(want[:, q])), (e, q)
