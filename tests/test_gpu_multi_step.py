"""Several steps per launch (lb_step on domains without particles and pressure
faces) against single steps (LB_OPT_TWO_STEP off): the same nodes, collisions
and roundings in both, so the states are bit-identical.  Sizes around the
edges of the regions (one tile, ragged last tiles, a lattice that is smaller
than the rim it wraps into), step counts with every split into odd parts and a
single last step, alone and in a batch of uneven domains."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

OPTIONS = [
    ("f64", dict(bc_y="wall")), ("f64", dict(kT=1e-4)),
    ("f32", dict(kT=1e-4)), ("f32", dict(bc_x="wall", bc_y="wall", kT=1e-4, solids=True)),
    ("f32", dict(bc_y="wall", power_law=dict(n=0.5, K=0.01))), ("f32", dict(collision="trt")),
    ("f16", dict(rounding="stochastic", solids=True)), ("f16", dict(kT=1e-4, bc_y="wall")),
    ("bf16", dict(rounding="stochastic", collision="trt", bc_x="wall")),
]


def _domain(lb, nx, ny, storage, kw, two, seed):
    kw = dict(kw)
    rng = np.random.default_rng(seed)
    if kw.pop("solids", False):
        kw["obstacles"] = rng.random((ny, nx)) < 0.1
    init = (1 + 0.01 * rng.standard_normal((ny, nx)), 0.02 * rng.standard_normal((ny, nx)),
            0.02 * rng.standard_normal((ny, nx)))
    d = lb.Domain(nx, ny, tau=0.8, g=(1e-5, -2e-6), storage=storage, seed=7, domain_id=seed,
                  init=init, **kw)
    d.set_option(lb.OPT_TWO_STEP, two)
    return d


@pytest.mark.parametrize("nx,ny", [(3, 3), (5, 17), (16, 8), (24, 24), (33, 31), (64, 32),
                                   (101, 51), (300, 260), (1031, 770)])
@pytest.mark.parametrize("storage,kw", OPTIONS)
def test_multi_step_is_bit_identical_to_single_steps(nx, ny, storage, kw):
    from paper_2006_12910_amd import lb
    a, b = (_domain(lb, nx, ny, storage, kw, two, 3) for two in (1, 0))
    for n in (1, 2, 3, 10, 17, 19):
        a.step(n)
        b.step(n)
        assert np.array_equal(a.populations(), b.populations()), n
    assert a.time == b.time == 52 and a.mass() == b.mass()
    a.close()
    b.close()


@pytest.mark.parametrize("sizes", [[(5, 17), (33, 31), (101, 51), (300, 260), (64, 32)],
                                   [(1031, 770), (900, 1200)]])  # three steps a launch, and five
@pytest.mark.parametrize("storage,kw", OPTIONS)
def test_multi_step_batch_is_bit_identical_to_single_domains(storage, kw, sizes):
    from paper_2006_12910_amd import lb
    a, b = ([_domain(lb, nx, ny, storage, kw, two, 3 + i) for i, (nx, ny) in enumerate(sizes)]
            for two in (1, 0))
    batch = lb.Batch(a)
    for n in (2, 11, 17):
        batch.step(n)
    for d, s in zip(a, b):
        s.step(30)
        assert np.array_equal(d.populations(), s.populations())
        assert d.time == s.time == 30
    batch.close()
    for d in a + b:
        d.close()
