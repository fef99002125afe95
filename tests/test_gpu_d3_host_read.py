"""lb3_moments and lb3_get_populations of fields large enough for the pinned
ring and its helper threads, against the plain copies that a small domain
takes: the large domain is the small one repeated along its periodic z axis, so
every layer holds the same bits (round to nearest: stochastic bits depend on
the node).  Sizes with whole and ragged last chunks; and
overlapping output arrays, which are written in order."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz,reps", [(64, 64, 16, 4), (64, 64, 16, 8), (67, 61, 15, 5),
                                           (97, 83, 5, 21)])
@pytest.mark.parametrize("storage,lattice", [("f64", "d3q19"), ("f16", "d3q27")])
def test_large_reads_match_small_ones(nx, ny, nz, reps, storage, lattice):
    from paper_2006_12910_amd import lb
    rng = np.random.default_rng(nx)
    init = tuple(a + 0.02 * rng.standard_normal((nz, ny, nx)) for a in (1.0, 0.0, 0.0, 0.0))
    kw = dict(tau=0.8, storage=storage, lattice=lattice, rounding="nearest",
              g=(1e-5, 2e-6, -3e-6))
    a = lb.Domain3(nx, ny, nz, init=init, **kw)
    b = lb.Domain3(nx, ny, nz * reps, init=tuple(np.tile(v, (reps, 1, 1)) for v in init), **kw)
    for steps in (3, 2):  # the second read reuses the ring
        a.step(steps)
        b.step(steps)
        small, large = a.moments(), b.moments()
        assert 32 * nx * ny * nz < 8 << 20 <= 32 * nx * ny * nz * reps
        for s, v in zip(small, large):
            assert np.array_equal(np.tile(s, (reps, 1, 1)), v)
        fs, fl = a.populations(), b.populations()
        assert np.array_equal(np.tile(fs.reshape(-1, nz, ny, nx), (1, reps, 1, 1)).ravel(), fl.ravel())
    r, u = np.empty_like(large[0]), np.empty_like(large[0])
    p = lambda v: v.ctypes.data_as(C.POINTER(C.c_double))
    assert lb.library().lb3_moments(b._h, p(r), p(u), p(u), p(u)) == 0
    assert np.array_equal(r, large[0]) and np.array_equal(u, large[3])
    a.close()
    b.close()
