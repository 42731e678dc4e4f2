"""Solves on a stream that is being captured into a graph are refused and
leave no trace: nothing of theirs is in the graph, and the handle's next solve
is right also when its sweep shape changed just before."""
import numpy as np
import pytest

from synthetic.workloads import SourceSpec, random_small_problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
dsn = pytest.importorskip("paper_1910_11335_amd")


def test_solve_under_capture_is_refused_and_leaves_the_handle_right():
    p = random_small_problem(23, n=(11, 34, 26), sn=4, L=1, G=2, n_mat=3, fixup=1)
    s = SourceSpec(position=(-2.3, 7.0, 9.0), spectrum=np.array([1.0, 0.4]))
    kw = dict(fixed_iters=[3, 2])
    ref_h = dsn.Problem(p, "fp32")
    ref_h.set_sweep_shape(1, 64)
    ref = ref_h.solve([s], **kw)["phi_total"].clone()
    ref_h.close()
    h = dsn.Problem(p, "fp32")
    h.set_sweep_shape(1, 64)
    for rep in range(3):
        assert torch.equal(h.solve([s], **kw)["phi_total"], ref)
        h.set_sweep_shape(1, 64, 0, 2 if rep % 2 == 0 else 0)
        out = torch.empty((1, p.G, p.V), dtype=torch.float64, device="cuda")
        x = torch.ones(8, device="cuda")
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph):
            y = x + 1
            with pytest.raises(dsn.DsnError) as err:
                h.solve([s], out=out, **kw)
            assert err.value.status == dsn.dsn.DSN_ERR_DEVICE
            with pytest.raises(dsn.DsnError):
                h.solve([s], out=out, tol=1e-4)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, x + 1)
        assert torch.equal(h.solve([s], **kw)["phi_total"], ref), rep
    h.close()
