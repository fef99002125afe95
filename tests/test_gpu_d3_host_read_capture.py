"""A thread that reads a 3D domain's fields for the first time (which makes its
pinned ring), and destroys the domain, while another thread captures a graph in
the global mode: neither disturbs the other."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_read_and_destroy_beside_a_capture():
    import torch
    from paper_2006_12910_amd import lb
    a, b = (lb.Domain3(96, 96, 96, tau=0.8, storage="f32", g=(1e-5, 0.0, 0.0)) for _ in range(2))
    for d in (a, b):
        d.step(3)
    want = b.moments()
    x = torch.zeros(1000, device="cuda")
    torch.cuda.synchronize()
    got, graph = [], torch.cuda.CUDAGraph()

    def read():
        got.append(a.moments())
        got.append(a.moments())
        a.close()

    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        x.add_(1)
        t = threading.Thread(target=read)
        t.start()
        t.join()
        x.add_(1)
    assert len(got) == 2
    for m in got:
        for v, w in zip(m, want):
            assert np.array_equal(v, w)
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert x.cpu().eq(2.0 * (k + 1)).all()
    b.close()
