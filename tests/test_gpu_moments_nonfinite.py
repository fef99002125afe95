"""Moments of a node that holds a non-finite population: neither its density nor
its velocity is finite, whichever population it is; the other nodes keep
theirs."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("i", range(9))
def test_no_finite_velocity_of_a_non_finite_node(storage, value, i):
    import torch
    from paper_2006_12910_amd import lb
    nx, ny = 37, 21
    rng = np.random.default_rng(i)
    d = lb.Domain(nx, ny, tau=0.8, storage=storage, g=(1e-5, 2e-6),
                  init=(1.0, 0.02 * rng.standard_normal((ny, nx)), 0.02 * rng.standard_normal((ny, nx))))
    ref = d.moments()
    f = d.populations()
    f[i, 10, 11] = value
    d.set_populations(f)
    dev = [v.cpu().numpy() for v in d.moments_device()]
    torch.cuda.synchronize()
    for got in (d.moments(), dev):
        for v, w in zip(got, ref):
            assert not np.isfinite(v[10, 11])
            v, w = v.copy(), w.copy()
            v[10, 11] = w[10, 11] = 0.0
            assert np.array_equal(v, w)
    d.close()
