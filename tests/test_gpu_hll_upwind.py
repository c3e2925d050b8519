"""HLL (and HLLC where it says so) next to density jumps: the flux of a face whose waves all move one way
is the upwind state's, whichever way that is, so a light cell beside a heavy
one keeps its own accuracy, and a mirrored problem has the mirrored result."""
import numpy as np
import pytest

from paper_2303_03026_amd import inputs

pytestmark = pytest.mark.gpu

# limiters of two ghost layers: their slopes vanish at these layers, so a face's
# light state holds nothing of the heavy one
PATHS = [("plain", 8, 0, 2), ("plain", 16, 2, 2), ("fused", 16, 0, 2), ("fused", 16, 2, 2), ("fused", 16, 1, 3)]
FORMS = [p + (0,) for p in PATHS] + [p + (1,) for p in PATHS if p[0] == "fused"]
IDS = ["%s_%d_lim%d_ng%d_%s" % (f[:4] + (("f64", "mixed")[f[4]],)) for f in FORMS]


@pytest.fixture(scope="module")
def amr():
    from paper_2303_03026_amd import amrvac
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    return amrvac


def workload(form, prim):
    """prim: [9, nz, ny, nx] of a periodic box"""
    _, nx, limiter, ng, _ = form
    base = tuple(n // nx for n in prim.shape[:0:-1])
    level, ijk = inputs.uniform_blocks(3, base)
    return inputs.Workload("layers", 3, nx, base, (0.0,) * 3, tuple(float(b) for b in base), (0,) * 3, (0,) * 3,
                           level, ijk, inputs.global_to_blocks(prim, 3, nx).swapaxes(0, 1), limiter=limiter, ng=ng)


def one_stage(amr, form, w, scalars=None):
    sim = amr.Simulation(w, path=amr.PATH_FUSED if form[0] == "fused" else amr.PATH_PLAIN, precision=form[4])
    if scalars is None:
        sim.cfl(0)
        scalars = sim.scalars()
    else:
        sim.set_scalars(*scalars)
    sim.euler_stage()
    got = sim.cons(1)
    sim.close()
    return got, scalars


def oracle_stage(orc, w, scalars):
    sim = orc.OracleSim(w)
    sim.euler_stage(*scalars)
    want = sim.cons()
    sim.close()
    return want


def layers(nx, axis, speed):
    """Layers of density 1024 and 1 across the axis, moving along it (binary
    fractions, so that the pressures are recovered exactly)."""
    n = 2 * nx
    rng = np.random.Generator(np.random.PCG64(41))
    width = rng.integers(1, 5, size=n)
    rho = np.repeat(np.arange(n) % 2, width)[:n]
    vel = np.repeat(speed + rng.integers(0, 8, size=n) / 64.0, width)[:n]
    shape = [1, 1, 1]
    shape[2 - axis] = n
    box = [nx] * 3
    box[2 - axis] = n
    prim = np.zeros((9,) + tuple(box))
    prim[inputs.RHO] = np.where(rho, 1024.0, 1.0).reshape(shape)
    prim[inputs.VX:inputs.VX + 3] = 0.25
    prim[inputs.VX + axis] = vel.reshape(shape)
    prim[inputs.PR] = 1.0
    for c, b in enumerate((0.25, 0.125, -0.5)):
        prim[inputs.BX + c] = b
    return prim


def mirrored(v, axis, components):
    v = np.flip(v, axis=v.ndim - 1 - axis).copy()
    for c in components:
        v[c + axis] *= -1.0
    return v


def local_sizes(u):
    """Per cell: the sizes its variables are made of."""
    m, b = np.sqrt(np.sum(u[1:4] ** 2, 0)), np.sqrt(np.sum(u[5:8] ** 2, 0))
    return np.stack([u[0], m, m, m, u[4], b, b, b])


# supersonic in both gases; supersonic in the heavy one alone
@pytest.mark.parametrize("speed", [8.0, 1.25])
@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("form", FORMS, ids=IDS)
def test_light_cells_beside_heavy_ones(amr, orc, form, axis, speed):
    nx = form[1]
    prim = layers(nx, axis, speed)
    # some 50 roundings of the path's face precision
    tol = 50 * 2.0 ** (-24 if form[4] else -53)
    got = []
    for p in (prim, mirrored(prim, axis, (inputs.VX, inputs.BX))):
        w = workload(form, p)
        u, scalars = one_stage(amr, form, w)
        base = w.base_blocks
        whole = [inputs.blocks_to_global(a.swapaxes(0, 1), 3, nx, base) for a in (u, oracle_stage(orc, w, scalars))]
        got.append(whole[0])
        size = local_sizes(whole[1])
        bad = np.abs(whole[0] - whole[1])[:8] / size
        assert np.all(bad <= tol), (np.max(bad.reshape(8, -1), 1) / tol)
    back = mirrored(got[1], axis, (1, 5))
    bad = np.abs(got[0] - back)[:8] / local_sizes(got[0])
    assert np.all(bad <= tol), (np.max(bad.reshape(8, -1), 1) / tol)


@pytest.mark.parametrize("flux", [0, 2], ids=["hll", "hllc"])
@pytest.mark.parametrize("form", FORMS, ids=IDS)
def test_no_wave_at_all(amr, orc, form, flux):
    """Negative pressure at rest, flagged and not replaced: both bounds are
    zero and the flux is the left state's."""
    nx = form[1]
    odd = np.arange(nx) % 2
    prim = np.zeros((9, nx, nx, nx))
    prim[inputs.RHO] = np.where(odd, 2.0, 1.0)
    prim[inputs.PR] = np.where(odd, -2.0, -1.0)
    w = workload(form, prim)
    w.flux = flux
    scalars = (2.0 ** -10, 1.0, 0.0)
    got, _ = one_stage(amr, form, w, scalars)
    want = oracle_stage(orc, w, scalars)
    assert np.all(np.isfinite(want)) and np.max(np.abs(want[:, 1])) > 1e-3
    assert np.max(np.abs(got - want)) <= 50 * 2.0 ** (-24 if form[4] else -53) * np.max(np.abs(want))
