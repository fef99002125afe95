"""lb_autotune reports the time per step that the domain runs at afterwards,
with several steps a launch (without and with a disc) and without."""
import time

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("disc", [False, True])
@pytest.mark.parametrize("two", [1, 0])
def test_autotune_reports_what_the_domain_runs_at(disc, two):
    import torch
    from paper_2006_12910_amd import lb
    d = lb.Domain(512, 512, tau=1.0, kT=1e-4, storage="f32", max_particles=1 if disc else 0)
    d.set_option(lb.OPT_TWO_STEP, two)
    if disc:
        d.add_particles([dict(x=200.0, y=256.0, radius=5.0)])
    ms = d.autotune(steps=240)
    assert d.get_option(lb.OPT_TWO_STEP) == two
    best = 1e9
    for _ in range(5):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        d.step(240)
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t0) / 240 * 1e3)
    assert 0.7 * best < ms < 1.3 * best, (ms, best)
    d.close()
