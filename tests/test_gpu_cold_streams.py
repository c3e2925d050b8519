"""Supersonic faces of cold gas, where the fast speed is lost in rounding
beside the normal velocity: HLLD's and HLLC's star states are not finite
there, and the flux is the upwind side's.  Uniform streams have to stay as
they are, bit for bit; streams of varying density follow the oracle, which
returns the upwind flux before it forms star states."""
import numpy as np
import pytest

from paper_2303_03026_amd import inputs

pytestmark = pytest.mark.gpu

PATHS = [("plain", 8, 0, 2), ("plain", 16, 6, 3), ("fused", 16, 0, 2), ("fused", 16, 1, 3), ("fused", 16, 6, 3)]
FORMS = [p + (0,) for p in PATHS] + [p + (1,) for p in PATHS if p[0] == "fused"]
IDS = ["%s_%d_lim%d_ng%d_%s" % (f[:4] + (("f64", "mixed")[f[4]],)) for f in FORMS]


@pytest.fixture(scope="module")
def amr():
    from paper_2303_03026_amd import amrvac
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    return amrvac


def stream(ndim, form, flux, v):
    """Field-free gas at the pressure floor; with |v| of 8 per direction the
    speed of sound is below half a unit in the velocity's last place."""
    _, nx, limiter, ng, precision = form
    w = inputs.uniform_state(ndim, (2, 3, 2 if ndim == 3 else 1), [1.0, v[0], v[1], v[2], 0, 0, 0, 0, 0], nx=nx)
    w.limiter, w.ng, w.flux, w.gamma = limiter, ng, flux, 2.0
    w.fix_small_values, w.small_pressure = 1, 2.0 ** (-46 if precision else -140)
    return w


def open_sim(amr, w, form):
    return amr.Simulation(w, path=amr.PATH_FUSED if form[0] == "fused" else amr.PATH_PLAIN, precision=form[4])


@pytest.mark.parametrize("flux", [0, 1, 2], ids=["hll", "hlld", "hllc"])
@pytest.mark.parametrize("form", FORMS, ids=IDS)
@pytest.mark.parametrize("ndim", [2, 3])
def test_uniform_stream_bit_identical(amr, ndim, form, flux):
    for sign in (8.0, -8.0):
        sim = open_sim(amr, stream(ndim, form, flux, (sign, -sign, sign)), form)
        u0 = sim.cons()
        sim.advance(2, nstages=3)
        got = sim.cons()
        sim.close()
        assert np.array_equal(got, u0), sign


@pytest.mark.parametrize("flux", [1, 2], ids=["hlld", "hllc"])
@pytest.mark.parametrize("form", FORMS, ids=IDS)
def test_negative_pressure_stream_bit_identical(amr, form, flux):
    """Small values flagged, not replaced."""
    w = stream(3, form, flux, (8.0, -8.0, 8.0))
    w.fix_small_values = 0
    w.prim[:, inputs.PR] = -1.0
    sim = open_sim(amr, w, form)
    u0 = sim.cons()
    sim.cfl(0)
    sim.euler_stage()
    got = sim.cons(1)
    assert sim.sync_flags(raise_on_error=False)[0] & amr.FLAG_SMALL_P
    sim.close()
    assert np.array_equal(got, u0)


@pytest.mark.parametrize("flux", [1, 2], ids=["hlld", "hllc"])
@pytest.mark.parametrize("form", FORMS, ids=IDS)
def test_varying_density_follows_the_oracle(amr, orc, form, flux):
    for sign in (8.0, -8.0):
        w = stream(3, form, flux, (sign, sign, -sign))
        rng = np.random.Generator(np.random.PCG64(31))
        # powers of two: the kinetic energy cancels exactly, the pressure is the floor
        w.prim[:, inputs.RHO] = 2.0 ** rng.integers(0, 3, size=w.prim[:, inputs.RHO].shape)
        sim = open_sim(amr, w, form)
        sim.cfl(0)
        dt, ch, kappa = sim.scalars()
        sim.euler_stage()
        got = sim.cons(1)
        sim.close()
        ref = orc.OracleSim(w)
        ref.euler_stage(dt, ch, kappa)
        want = ref.cons()
        ref.close()
        # some 50 roundings per flux at the path's face precision, of values of
        # the largest flux, which a step moves by at most its own size
        tol = 50 * 2.0 ** (-24 if form[4] else -53)
        for q in range(9):
            assert np.max(np.abs(got[:, q] - want[:, q])) <= tol * np.max(np.abs(want[:, q])), (sign, q)


@pytest.mark.parametrize("form", FORMS, ids=IDS)
def test_contact_speed_on_an_outer_wave(amr, orc, form):
    """HLLD between p = 1/2 and p = -3/2 at gamma = 2: S_M falls on the outer
    wave of the side with negative pressure, whose star state is infinite; the
    flux is the other side's."""
    w = stream(2, form, 1, (0.0, 8.0, 0.0))
    w.fix_small_values = 0
    w.prim[:, inputs.PR] = np.where(np.arange(form[1]) % 2, 0.5, -1.5)
    sim = open_sim(amr, w, form)
    sim.cfl(0)
    dt, ch, kappa = sim.scalars()
    sim.euler_stage()
    got = sim.cons(1)
    sim.close()
    ref = orc.OracleSim(w)
    ref.euler_stage(dt, ch, kappa)
    want = ref.cons()
    ref.close()
    assert np.all(np.isfinite(want))
    tol = 50 * 2.0 ** (-24 if form[4] else -53)
    assert np.max(np.abs(got - want)) <= tol * np.max(np.abs(want))
