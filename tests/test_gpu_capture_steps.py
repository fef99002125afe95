"""lb_step under a caller's graph capture, for domains that may take several
steps a launch: every replay advances the state as the eager call does, with
the library's eager work between the replays; also where the plan is single
steps (FP16 with noise on a lattice that fills the chip)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = [(128, 64, "f64", dict(bc_y="wall"), False), (300, 260, "f32", dict(kT=1e-5), False),
         (1031, 770, "f16", dict(rounding="stochastic"), False), (128, 96, "f32", dict(kT=1e-5), True),
         (2048, 2048, "f16", dict(kT=1e-5, rounding="stochastic"), False)]


@pytest.mark.parametrize("nx,ny,storage,kw,disc", CASES)
@pytest.mark.parametrize("n", [1, 5, 8])
def test_replays_of_captured_steps(nx, ny, storage, kw, disc, n):
    import torch
    from paper_2006_12910_amd import lb
    rng = np.random.default_rng(1)
    init = (1 + 0.01 * rng.standard_normal((ny, nx)), 0.02 * rng.standard_normal((ny, nx)),
            0.02 * rng.standard_normal((ny, nx)))
    s = torch.cuda.Stream()
    a, b = (lb.Domain(nx, ny, tau=0.8, g=(1e-5, 0.0), storage=storage, seed=5, init=init, stream=s,
                      max_particles=1 if disc else 0, **kw) for _ in range(2))
    if disc:
        for d in (a, b):
            d.add_particles([dict(x=nx / 2, y=ny / 2, radius=5.0, ux=0.05)])
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=s):
        a.step(n)
    for _ in range(3):
        with torch.cuda.stream(s):
            graph.replay()
        torch.cuda.synchronize()
        b.step(n)
        fa, fb = a.moments(), b.moments()  # by the device's step counter
        for v, w in zip(fa, fb):
            assert np.array_equal(v, w)
    assert b.time == 3 * n
    a.close()
    b.close()
