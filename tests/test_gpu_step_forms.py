"""Forms of the launches of several steps that the other tests of them leave
out, bit for bit against single steps: up to nine steps a launch and the large
region with seven; stochastic rounding of FP32 storage; every
specialisation of the power-law exponent, alone, beside a disc and in a batch;
grids of 64 workgroups, whose last launch moves the step counter on, and of
one more; single steps over the small region; and the power law with solids in
the two-step 3D sweep."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _domain(lb, nx, ny, storage, kw, two, seed=3, disc=None):
    kw = dict(kw)
    rng = np.random.default_rng(nx + seed)
    if kw.pop("solids", False):
        m = rng.random((ny, nx)) < 0.1
        if disc:
            yy, xx = np.mgrid[:ny, :nx]
            m &= np.hypot(xx - disc["x"], yy - disc["y"]) > disc["radius"] + 4
        kw["obstacles"] = m
    init = (1 + 0.01 * rng.standard_normal((ny, nx)), 0.02 * rng.standard_normal((ny, nx)),
            0.02 * rng.standard_normal((ny, nx)))
    d = lb.Domain(nx, ny, tau=0.8, g=(1e-5, -2e-6), storage=storage, seed=7, domain_id=seed, init=init,
                  max_particles=1 if disc else 0, **kw)
    d.set_option(lb.OPT_TWO_STEP, two)
    if disc:
        d.add_particles([disc])
    return d


def _compare(lb, nx, ny, storage, kw, calls, disc=None):
    a, b = (_domain(lb, nx, ny, storage, kw, two, disc=disc) for two in (1, 0))
    for n in calls:
        a.step(n)
        b.step(n)
        assert np.array_equal(a.populations(), b.populations()), n
    assert a.time == b.time == sum(calls) and a.mass() == b.mass()
    if disc:
        assert bytes(a.particle_state()[0]) == bytes(b.particle_state()[0])
    a.close()
    b.close()


@pytest.mark.parametrize("nx,ny,storage,kw", [
    (256, 256, "f32", dict()), (256, 256, "f32", dict(solids=True)), (256, 256, "f64", dict(kT=1e-4)),
    (400, 400, "f16", dict(rounding="stochastic")), (400, 400, "f16", dict(rounding="stochastic", solids=True)),
    (400, 400, "bf16", dict(solids=True)), (724, 700, "f16", dict(rounding="stochastic", solids=True)),
    (724, 700, "f32", dict(bc_y="wall", kT=1e-4)), (1400, 900, "f32", dict(solids=True, collision="trt"))])
def test_long_launches(nx, ny, storage, kw):
    from paper_2006_12910_amd import lb
    _compare(lb, nx, ny, storage, kw, (9, 18, 1, 7, 22))


@pytest.mark.parametrize("nx,ny", [(24, 24), (257, 131), (724, 700)])
@pytest.mark.parametrize("solids", [False, True])
def test_stochastic_rounding_of_fp32(nx, ny, solids):
    from paper_2006_12910_amd import lb
    _compare(lb, nx, ny, "f32", dict(rounding="stochastic", solids=solids), (5, 13, 1))


POWERS = [0.5, 0.75, 1.5, 1.3, 1.0, 0.6]


@pytest.mark.parametrize("n", POWERS)
@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("collision", ["bgk", "trt"])
def test_power_law_exponents(n, storage, collision):
    from paper_2006_12910_amd import lb
    kw = dict(bc_y="wall", power_law=dict(n=n, K=0.01), collision=collision)
    disc = dict(x=40.0, y=30.5, radius=4.0, ux=0.1, density_ratio=1.5)
    _compare(lb, 101, 61, storage, kw, (7, 10))
    _compare(lb, 300, 260, storage, dict(kw, solids=True), (11,))
    _compare(lb, 101, 61, storage, kw, (6, 4), disc=disc)


@pytest.mark.parametrize("n", POWERS)
def test_power_law_exponents_in_a_batch(n):
    from paper_2006_12910_amd import lb
    kw = dict(bc_y="wall", power_law=dict(n=n, K=0.01))
    sizes = [(48, 33), (300, 90), (128, 64)]
    a, b = ([_domain(lb, nx, ny, "f32", kw, two, seed=i) for i, (nx, ny) in enumerate(sizes)]
            for two in (1, 0))
    batch = lb.Batch(a)
    for c in (4, 9):
        batch.step(c)
    for d, s in zip(a, b):
        s.step(13)
        assert np.array_equal(d.populations(), s.populations())
    batch.close()
    for d in a + b:
        d.close()


# single steps: tiles of 32 x 16, of 26 x 10 and 20 x 4 with four and seven steps
@pytest.mark.parametrize("nx,ny", [(256, 128), (257, 128), (26 * 8, 10 * 8), (26 * 13, 10 * 5), (20 * 8, 4 * 8),
                                   (20 * 13, 4 * 5), (512, 256), (724, 700), (1031, 1000)])
@pytest.mark.parametrize("storage", ["f64", "f16"])
def test_step_counter_around_64_workgroups(nx, ny, storage):
    from paper_2006_12910_amd import lb
    _compare(lb, nx, ny, storage, dict(solids=True), (1, 1, 4, 7, 2, 1, 3))


@pytest.mark.parametrize("shape", [(256, 160, 64), (256, 159, 66)])
@pytest.mark.parametrize("lattice,extra", [
    ("d3q27", dict(power_law=dict(n=0.5, K=0.01))), ("d3q27", dict(power_law=dict(n=1.3, K=0.01))),
    ("d3q19", dict(power_law=dict(n=0.5, K=0.01), collision="trt"))])
def test_two_step_3d_power_law_with_solids(shape, lattice, extra):
    from paper_2006_12910_amd import lb
    nx, ny, nz = shape
    rng = np.random.default_rng(nx + ny)
    s = (nz, ny, nx)
    kw = dict(tau=0.8, storage="f32", lattice=lattice, g=(1e-5, 2e-6, -3e-6), obstacles=rng.random(s) < 0.1,
              init=(1 + 0.01 * rng.standard_normal(s),) + tuple(0.02 * rng.standard_normal(s)
                                                              for _ in range(3)), **extra)
    a, b = lb.Domain3(*shape, **kw), lb.Domain3(*shape, **kw)
    a.step(8)  # two pairs of two-step launches
    for _ in range(8):
        b.step(1)
    assert np.array_equal(a.populations(), b.populations())
    assert a.time == b.time == 8 and a.mass() == b.mass()
    a.close()
    b.close()
