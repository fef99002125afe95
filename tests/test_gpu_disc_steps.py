"""Several steps per launch with one particle (its coupling on chip, beside the
tiles) against single steps (LB_OPT_TWO_STEP off): the same nodes, links, sums
and roundings in the same order, so the populations and the particle are
bit-identical.  Domains as small as the region and ragged ones; discs of the
smallest and the largest radius that take the path, moving across a periodic
corner, next to a wall and among obstacles with repulsion; step counts with
every split; alone and in a batch with and without discs; and a domain and a
radius that keep single steps."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

NOISE = dict(kT=1e-4)
CASES = [  # nx, ny, storage, domain arguments, disc
    (48, 33, "f32", NOISE, dict(x=1.3, y=0.4, radius=5.0, ux=-0.21, uy=-0.13)),
    (64, 32, "f16", dict(rounding="stochastic"), dict(x=40.0, y=16.0, radius=8.0, ux=0.3, omega=0.01)),
    (32, 32, "f64", NOISE, dict(x=31.9, y=31.9, radius=4.2, ux=0.2, uy=0.24)),
    (101, 77, "f64", dict(collision="trt", lj=(1e-3, 2.5, 0.5), walls=True, solids=True),
     dict(x=50.3, y=12.2, radius=3.7, uy=-0.2, density_ratio=1.5)),
    (300, 200, "bf16", NOISE, dict(x=299.6, y=100.5, radius=8.0, ux=0.15, omega=-0.02)),
    (130, 66, "f32", dict(power_law=dict(n=0.5, K=0.01), walls=True), dict(x=65.0, y=20.0, radius=2.0,
                                                                           ux=0.15, favg=True)),
    (257, 129, "f32", dict(lj=(1e-3, 2.5, 0.5), solids=True, **NOISE),
     dict(x=128.5, y=64.5, radius=6.5, ux=-0.3, uy=0.3, favg=True)),
    (128, 96, "f32", dict(), dict(x=64.0, y=48.0, radius=3.0, fixed=True, omega=0.02)),
    # beside a wall: the particle's region reaches past it to the far side
    (96, 60, "f32", dict(lj=(1e-3, 2.5, 0.5), walls=True, **NOISE), dict(x=3.0, y=5.5, radius=3.0, ux=0.1)),
    # single steps in both: too small a domain, too large a disc
    (31, 40, "f32", NOISE, dict(x=20.0, y=20.0, radius=5.0, ux=0.2)),
    (128, 96, "f32", NOISE, dict(x=64.0, y=48.0, radius=8.2, ux=0.2)),
]


def _domain(lb, nx, ny, storage, kw, disc, two, seed=3):
    kw = dict(kw)
    rng = np.random.default_rng(nx + seed)
    if kw.pop("walls", False):
        kw["bc_y"] = "wall"
    if kw.pop("solids", False):
        m = rng.random((ny, nx)) < 0.04
        yy, xx = np.mgrid[:ny, :nx]
        m &= np.hypot(xx - disc["x"], yy - disc["y"]) > disc["radius"] + 4
        kw["obstacles"] = m
    init = (1 + 0.01 * rng.standard_normal((ny, nx)), 0.02 * rng.standard_normal((ny, nx)),
            0.02 * rng.standard_normal((ny, nx)))
    disc = dict(disc) if disc else None
    favg = disc.pop("favg", False) if disc else False
    d = lb.Domain(nx, ny, tau=0.8, g=(1e-5, -2e-6), storage=storage, seed=7, domain_id=seed,
                  init=init, max_particles=1 if disc else 0, **kw)
    d.set_option(lb.OPT_TWO_STEP, two)
    if favg:
        d.set_option(lb.OPT_FORCE_AVERAGE, 1)
    if disc:
        d.add_particles([disc])
    return d


def _same(a, b):
    assert np.array_equal(a.populations(), b.populations())
    assert bytes(a.particle_state()[0]) == bytes(b.particle_state()[0])
    assert a.time == b.time and a.mass() == b.mass()


@pytest.mark.parametrize("nx,ny,storage,kw,disc", CASES)
def test_disc_steps_are_bit_identical_to_single_steps(nx, ny, storage, kw, disc):
    from paper_2006_12910_amd import lb
    a, b = (_domain(lb, nx, ny, storage, kw, disc, two) for two in (1, 0))
    for n in (1, 3, 2, 7, 18, 4):
        a.step(n)
        b.step(n)
        _same(a, b)
    a.close()
    b.close()


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
def test_disc_steps_batch_is_bit_identical_to_single_domains(storage):
    from paper_2006_12910_amd import lb
    disc = dict(x=30.0, y=30.5, radius=5.0, ux=0.1, uy=-0.2)
    specs = [(64, 64, disc), (33, 31, None), (150, 99, dict(disc, x=149.0, y=1.0)), (200, 64, None),
             (70, 44, dict(disc, radius=8.0))]
    a, b = ([_domain(lb, nx, ny, storage, NOISE, q, two, seed=i) for i, (nx, ny, q) in enumerate(specs)]
            for two in (1, 0))
    batch = lb.Batch(a)
    for n in (2, 9, 16):
        batch.step(n)
    for d, s in zip(a, b):
        s.step(27)
        _same(d, s)
    batch.close()
    for d in a + b:
        d.close()
