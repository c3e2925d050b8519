"""Regrid plans on a hierarchy too deep for the dense slot arrays (twelve
levels): what refinement towards a corner builds, coarsening takes back, and
every leaf set on the way tiles the domain with one level between
neighbours."""
import numpy as np
import pytest

from paper_2303_03026_amd import amrvac, inputs


def as_set(level, ijk):
    return {(int(l), *map(int, p)) for l, p in zip(level, ijk)}


@pytest.mark.parametrize("ndim,levels", [(2, 12), (3, 9)])
def test_refining_and_coarsening_a_corner(ndim, levels):
    base = (4, 4, 4 if ndim == 3 else 1)
    level, ijk = inputs.uniform_blocks(ndim, base)
    w = inputs.Workload("corner", ndim, 16, base, (0.0,) * 3, (1.0,) * 3, (1,) * 3, (1,) * 3, level, ijk,
                        np.zeros((1, 9) + (16,) * ndim))
    first = as_set(level, ijk)
    deep = 2.0 ** (levels - 1)
    for _ in range(levels - 1):
        flags = np.where((ijk[:, :ndim] == 0).all(axis=1), 1, 0)
        level, ijk = amrvac.regrid_plan(w, flags, max_level=levels, level=level, ijk=ijk)
        assert len(as_set(level, ijk)) == len(level)
        # (exact: every term is a multiple of 2^(-ndim (levels - 1)))
        assert np.sum(0.5 ** (ndim * (level.astype(float) - 1))) == 4.0 ** ndim
        same = amrvac.regrid_plan(w, np.zeros(len(level), int), max_level=levels, level=level, ijk=ijk)
        assert as_set(*same) == as_set(level, ijk)
        # two touching leaves, as boxes in cells of the finest level
        size = (deep / 2.0 ** (level - 1)).astype(np.int64)
        lo = ijk[:, :ndim].astype(np.int64) * size[:, None]
        hi = lo + size[:, None]
        touch = np.ones((len(level), len(level)), bool)
        for d in range(ndim):
            touch &= (lo[:, None, d] <= hi[None, :, d]) & (lo[None, :, d] <= hi[:, None, d])
        assert np.max(np.abs(level[:, None] - level[None, :])[touch]) <= 1
    assert level.max() == levels
    for _ in range(levels):
        level, ijk = amrvac.regrid_plan(w, np.full(len(level), -1), max_level=levels, level=level, ijk=ijk)
    assert as_set(level, ijk) == first
